// Grouped bf16 GEMM, persistent workgroups, 256 x 256 tiles with 64-wide k-stages: the main
// kernel for layers whose output width is a multiple of 256.
//
// Same contract as the other grouped GEMMs (one launch multiplies every tenant segment of a
// mixed batch by that tenant's own weights, Sec. 6.3):
//      C[rows, :] = epi( A[rows, :] * W_g^T + b_g )        for every m-tile of segment g
//
// Measured facts about gfx950 that shape it
//   * An L2 channel answers one request per clock: 128 bytes if the request covers a whole
//     cache line, 64 if it covers half of one (33 TB/s against 17-20 TB/s for direct-to-LDS
//     copies that hit in L2).  Stores follow the same rule: a wavefront store that touches
//     64 different lines costs 64 requests however few bytes it carries.
//   * What the matrix cores sustain on random operands is a matter of power: fragments out of LDS, 64 x 128 a
//     wavefront, v_mfma_f32_16x16x32_bf16 1 860 TFLOP/s, v_mfma_f32_32x32x16_bf16 1 660 (out of registers 2 120 and 1 860).
//   * LDS reads run at 256 B/clk.
// Hence
//   * 256 x 256 tiles: the fewest operand bytes per FLOP the register file allows, held either by
//     8 wavefronts x 128 accumulator registers (two wavefronts per SIMD) or by 4 wavefronts x 256
//     accumulators in the AGPR half of a 512-register budget (one per SIMD); see Geo below;
//   * k-stages of 64 bf16 = 128 bytes per row: the eight lanes that copy a row fetch one
//     whole cache line, every operand request is a full line;
//   * all 160 KB of LDS are a ring of 2 activation and 3 weight stages of 32 KB; weight
//     copies (mostly L2 misses: a weight panel is shared only by the m-tiles of one
//     tenant) run further ahead than activation copies (mostly hits).  A wavefront issues a
//     stage's activation copies before its weight copies, so with in-order completion "all but
//     the newest weight stage have landed" is exactly the condition for the next stage;
//   * products on the 16 x 16 x 32 instruction, with each fragment read again for the next k-step as soon as it has been used for
//     the last time: one set of fragment registers, and a barrier a stage that stands where a wavefront has its last fragments.
//     65 536 rows of one weight set (d = 768, f = 3072), 32 x 32 x 16 products with two sets of fragments and these: QKV and output
//     projection together 329 us -> 313, FFN1 with GELU 344 -> 319, FFN2 with fp32 residuals 318 -> 290; 64 tenants' 32 768
//     rows, FFN1 239 -> 219, FFN2 224 -> 193;
//   * a compute unit takes 66 bytes per clock through its L1: a stage's copies are spread over its
//     MFMAs, since a wavefront that issues them faster than that stands still with its products
//     (all sixteen behind the sixteen MFMAs of one k-step, as before: second FFN GEMM of 65 536 rows
//     329 us -> 307 with four wavefronts; of 64 tenants' 32 768 rows 209 -> 190; the launches with
//     eight wavefronts 0 to 1.5 % faster);
//   * one workgroup per compute unit walks over its share of the tiles.  Copies for the
//     next tile are issued while the current one finishes;
//   * operand roles are swapped (weights are the MFMA's first operand, in a permuted row
//     order): a lane ends up with one row of C and 16 consecutive columns per four MFMA tiles;
//     bias is folded into the accumulator initialisation.  For the stores each wavefront
//     transposes its results through the part of the two idle ring slots that only its
//     own copies overwrite (no barrier), so that 16 consecutive lanes write 256 contiguous
//     bytes of a row: full-line requests again.  Units of 16 rows in turn, one written while the one before it
//     is read (eight wavefronts; in blocks of 32 rows with a wait between, FFN1 of 65 536 rows 1.5 % longer).
// What bounds it now: under the launches the clock is 1.9 GHz (2.4 under a copy, 1.7 under the vendor's 8192^3), so what a launch
// takes is its energy; a stage of products takes 2 640 clocks for 2 048 of matrix instructions, waits of 50 to 100 among them.
#include "hmi_kernels.h"

#include "gelu.h"
#include "lds_copy.h"
#include "wave.h"

namespace hmi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kXcds = 8;
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int WTN = 128, TN = 8;                             // a wavefront's 128 columns: eight MFMA tiles
// The workgroup is NW = 8 or 4 wavefronts, NW/2 x 2 over the tile: wavefront tiles of 64 x 128 (two per SIMD,
// 128 accumulator registers each) or 128 x 128 (one per SIMD with 256 accumulators in the AGPR half of a
// 512-register budget: a third less fragment traffic per MFMA and one instruction stream per matrix pipe,
// but nothing to run while that one wavefront waits, so it pays only where the main loop is long).
template <int NW>
struct Geo {
  static constexpr int NTH = 64 * NW;
  static constexpr int WTM = BM / (NW / 2), TM = WTM / 16;  // wavefront tile rows, MFMA tiles
  static constexpr int FWB = NW == 4 ? 2 : 1;               // register buffers of weight fragments (see HMI_ROWS)
  static constexpr int RH = WTM / 64;                       // output-row ids a lane keeps per tile
  static constexpr int LD = BM / 8 / NW;                    // one-KB copies (8 rows x 128 B) per wavefront, operand and stage: 4 or 8
  static constexpr int WAVE_SLICE = LD * 1024;              // the part of a stage slot that one wavefront's copies fill
};
constexpr int ROW_BYTES = BK * 2;                            // 128: one cache line per row and stage
constexpr int A_STAGES = 2, W_STAGES = 3;
constexpr int STAGE_BYTES = BM * ROW_BYTES;                  // 32 KB, same for both operands
constexpr int W_RING = A_STAGES * STAGE_BYTES;               // byte offset of the weight ring
constexpr int LDS_BYTES = W_RING + W_STAGES * STAGE_BYTES;   // 163840 = all of it

__device__ __forceinline__ float bf2f(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 p = {(__bf16)lo, (__bf16)hi};                       // round to nearest even
  return __builtin_bit_cast(uint32_t, p);
}

// LDS chunk swizzles (a row is 8 chunks of 16 bytes, two rows per 256-byte bank line).  A fragment read takes one chunk of 16
// rows for each quarter of the lanes: consecutive activation rows, weight rows in the order perm_w.  Either way the 16 lanes
// served together hit 16 distinct chunks.
__device__ __forceinline__ int swz_a(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int swz_w(int row) { return ((row >> 1) & 1) | (((row >> 4) & 3) << 1); }
// MFMA first-operand position i (0..15) of MFMA tile j <- weight row perm_w(i) + 64 (j / 4) + 4 (j % 4) of the wavefront's 128,
// chosen so that output register r of tile j and lane quarter q is column 64 (j / 4) + 16 q + 4 (j % 4) + r.
__device__ __forceinline__ int perm_w(int i) { return (i >> 2) * 16 + (i & 3); }

// Results leave with the non-temporal hint: nothing in this launch reads them again, and every line of L2 they do not
// take stays with the operand panels that other workgroups of the XCD are about to ask for (measured: 1-2 % fewer
// bytes fetched, GEMM time -0.7 to -1 % on the FFN, encoder and shared-layer workloads).
#define HMI_STORE_OUT(PTR, V) __builtin_nontemporal_store((V), (PTR))


// What a lane needs to know about a tile: where its copies come from and where the bias is.
constexpr int kMBlock = 8;   // m-tiles per block of a long segment's tile order

template <int NW>
struct TileRegs {
  int n0, row0, rows;
  const char* Wb;                  // first weight row of the tile: tenant's matrix + n0 rows
  const uint16_t* bias;
  uint32_t a_off[Geo<NW>::LD];     // byte offsets of this lane's activation copy sources at k = 0, plus 3072 - 1024 j
  int out_row[Geo<NW>::RH];        // where row (wavefront's first row + 64 h + lane) of the tile goes in C (row clamped to the tile)
};

// (the same for all lanes, so that it goes to a scalar register)
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int NW>
__device__ __forceinline__ void load_tile(const GemmArgs& g, const Route& rt, int w, int wave, int lane, TileRegs<NW>& tr) {
  constexpr int WTM = Geo<NW>::WTM, RH = Geo<NW>::RH, LD = Geo<NW>::LD;
  // Tile order: segment by segment; inside a segment n-tile by n-tile with the segment's
  // m-tiles innermost, so that the tiles which share a weight panel (and the few that
  // share an activation panel) run next to each other and the panel is fetched from HBM once.
  const int nt_n = g.n_out / BN;
  const int mt_any = w / nt_n;                               // some m-tile of the segment w falls in
  const int seg = uniform(rt.tile_seg[g.which_tiles][mt_any]);
  const int s0 = uniform(rt.seg_tok_off[seg]), s1 = uniform(rt.seg_tok_off[seg + 1]);
  const int mt_first = mt_any - (uniform(rt.tile_row0[g.which_tiles][mt_any]) - s0) / BM;
  const int mt_cnt = (s1 - s0 + BM - 1) / BM;
  const int q = w - mt_first * nt_n;
  // A long segment goes block by block of kMBlock m-tiles (the last block may be shorter): an activation panel's
  // n-tiles are then at most kMBlock tiles apart, close enough to run in the same round of the XCD's workgroups.
  const int b = q / (kMBlock * nt_n);
  const int bm = b < mt_cnt / kMBlock ? kMBlock : mt_cnt - b * kMBlock;
  const int rem = q - b * (kMBlock * nt_n);
  tr.n0 = (rem / bm) * BN;
  tr.row0 = s0 + (b * kMBlock + rem % bm) * BM;
  tr.rows = min(BM, s1 - tr.row0);
  const size_t slot_base = (size_t)uniform(rt.seg_slot[seg]) * g.slot_stride;
  tr.Wb = g.pool + slot_base + g.w_off + (size_t)tr.n0 * (size_t)(g.k * 2);
  tr.bias = reinterpret_cast<const uint16_t*>(g.pool + slot_base + g.b_off);
#pragma unroll
  for (int h = 0; h < RH; ++h) tr.out_row[h] = rt.row_src[tr.row0 + min((wave >> 1) * WTM + h * 64 + lane, tr.rows - 1)];
  // lane l fills LDS position (row l/8, chunk l%8) of an 8-row block with the global chunk
  // position ^ swizzle(row): the eight lanes of a row cover its whole 128-byte line.
#pragma unroll
  for (int j = 0; j < LD; ++j) {
    const int row = (wave * LD + j) * 8 + (lane >> 3);
    const int src = rt.row_src[tr.row0 + min(row, tr.rows - 1)];
    tr.a_off[j] = (uint32_t)src * (uint32_t)(g.lda * 2) + (((lane & 7) ^ swz_a(row)) << 4) + (3072 - (j & 3) * 1024);
  }
}


// The last workgroup of an XCD to finish puts the XCD's counters back to zero for the next launch.
__device__ __forceinline__ void finish_workgroup(const Route& rt, int xcd, int n_local) {
  if (threadIdx.x == 0) {
    int* done = rt.gemm_sched + 8 + xcd;
    if (atomicAdd(done, 1) == n_local - 1) {
      __hip_atomic_store(rt.gemm_sched + xcd, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

template <int NW, int EPI, bool OUT_F32, bool RESID_F32, bool HAS_C2>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4)))
void gemm_bf16_p256_kernel(GemmArgs g, Route rt, int total, int per_xcd) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int WTM = Geo<NW>::WTM, TM = Geo<NW>::TM, FWB = Geo<NW>::FWB, LD = Geo<NW>::LD, WAVE_SLICE = Geo<NW>::WAVE_SLICE;

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int KT = g.k / BK;
  const buffer_t a_buf = buffer_at(reinterpret_cast<const char*>(g.A) - 3072);

  // ---- this workgroup's tiles: XCD x (workgroups are dealt to XCDs round robin) owns the
  // contiguous range [x per_xcd, (x+1) per_xcd).  A workgroup's first two tiles are fixed
  // (its index inside the XCD, plus one round); from the third on it claims the next
  // unclaimed tile of the range, so that workgroups that drew cheap (short) tiles take more.
  // Wavefront 0 claims the tile after next at the start of a tile and passes the answer to
  // the other wavefronts through a mailbox in global memory (LDS has no byte to spare).
  const int n_local = gridDim.x / kXcds;
  const int xcd = blockIdx.x % kXcds;
  const int w_base = xcd * per_xcd;
  const int w_end = min(w_base + per_xcd, total);
  int* const claim_ctr = rt.gemm_sched + xcd;
  int* const mailbox = rt.gemm_sched + 16 + blockIdx.x;
  int w = w_base + blockIdx.x / kXcds;
  int w_next = w + n_local;
  if (w >= w_end) { finish_workgroup(rt, xcd, n_local); return; }
  const bool claimer = wave == 0 && lane == 0;
  int claimed = 0, mail = 0;
  if (claimer) claimed = atomicAdd(claim_ctr, 1);
  int budget = per_xcd;           // no workgroup can own more tiles than its XCD has: bounds the loop whatever the claims say

  TileRegs<NW> cur, nxt;
  load_tile(g, rt, w, wave, lane, cur);
  load_tile(g, rt, w_next < w_end ? w_next : w, wave, lane, nxt);

  // weight copies: the lane part of the source offset (plus 3072 - 1024 j) is the same for every tile
  uint32_t b_off[LD];
#pragma unroll
  for (int j = 0; j < LD; ++j) {
    const int row = (wave * LD + j) * 8 + (lane >> 3);
    b_off[j] = (uint32_t)row * (uint32_t)(g.k * 2) + (((lane & 7) ^ swz_w(row)) << 4) + (3072 - (j & 3) * 1024);
  }

  // ---- fragment read offsets inside a stage slot for the two k-steps of a stage
  // (k-step ks reads chunk (4 ks + lq) ^ swizzle: that is the k-step 0 offset with ks << 6 XORed in)
  int fx_base, fw_base;
  {
    const int rx = wm * WTM + l16;                       // + 16 i: swizzle unchanged
    const int rw = wn * WTN + perm_w(l16);               // + 64 (j / 4) + 4 (j % 4): swizzle unchanged
    fx_base = rx * ROW_BYTES + ((lq ^ swz_a(rx)) << 4);
    fw_base = W_RING + rw * ROW_BYTES + ((lq ^ swz_w(rw)) << 4);
  }

  // Ring bookkeeping (uniform): a_rd / w_rd are the byte offsets of the slots that hold the stage being multiplied.
  // Activation stage s+2 goes into that slot once stage s is done, weight stage s+2 into the slot before it; a stage index
  // of KT or more means a stage of the next tile (for the last tile: an in-bounds re-read of its own first stages that
  // nobody consumes).  Needs KT >= 3, so that the copies never reach the tile after next.
  int a_rd = 0, w_rd = 0;
  // Copies FROM .. FROM + COUNT - 1 of a wavefront's slice (1 KB each), from buffer SRC (uniform, of which the offset SOFF is), by
  // buffer loads: a global load to LDS counts among the LDS operations too, out of order, so that any wait for a fragment would
  // be one for all of them.  Four in a row share one LDS base (one M0 write); the instruction offset j KB that separates them
  // applies to the global address too, so the lane offsets carry 3072 - j KB and the buffers begin 3072 bytes early.
#define HMI_COPY(SRC, SOFF, VOFF, SLOT_OFF, FROM, COUNT)                                          \
  {                                                                                               \
    _Pragma("unroll") for (int j_ = (FROM); j_ < (FROM) + (COUNT); ++j_) {                        \
      lds_ptr_t dst_ = (lds_ptr_t)(smem + (SLOT_OFF) + wave * WAVE_SLICE + (j_ / 4) * 4096);      \
      if ((j_ & 3) == 0) copy_to_lds<0>(SRC, dst_, (VOFF)[j_], SOFF);                             \
      else if ((j_ & 3) == 1) copy_to_lds<1024>(SRC, dst_, (VOFF)[j_], SOFF);                     \
      else if ((j_ & 3) == 2) copy_to_lds<2048>(SRC, dst_, (VOFF)[j_], SOFF);                     \
      else copy_to_lds<3072>(SRC, dst_, (VOFF)[j_], SOFF);                                        \
    }                                                                                             \
  }
  static_assert(LD % 4 == 0, "HMI_COPY addresses the copies in groups of four");

  bf16x8 fx[TM], fw[FWB][TN];
  f32x4 acc[TM][TN];

  // MFMA fragments of k-step KS of the stage in slots A_SLOT / W_SLOT
#define HMI_READ_X(I, A_SLOT, KS)                                                                 \
  fx[I] = *reinterpret_cast<const bf16x8*>(smem + (A_SLOT) + (fx_base ^ ((KS) << 6)) + (I) * 16 * ROW_BYTES);
#define HMI_READ_W(B, J, W_SLOT, KS)                                                              \
  fw[B][J] = *reinterpret_cast<const bf16x8*>(smem + (W_SLOT) + (fw_base ^ ((KS) << 6)) + ((J) >> 2) * 64 * ROW_BYTES + ((J) & 3) * 4 * ROW_BYTES);

  // The products of MFMA rows R0 .. R1 - 1 of the k-step whose fragments are in fx and fw[B], in this order, and between them
  //   * the reads of k-step KS of slots A_SLOT / W_SLOT, whose fragments take the place of this one's as soon as each has been
  //     used for the last time (RD = 1): activations behind their row, weights behind the last row's products, which are eight
  //     MFMAs and the other wavefront's ahead of their next use.  With one wavefront per SIMD that is too short: weights have a
  //     second buffer there (fw[NB]) and are read two a row from row 1 on;
  //   * COPIES copies, evenly: COPY(c) is the c-th.  With two wavefronts per SIMD those of k-step 1's rows (the activations, which
  //     have to be there a stage later) between the first third of the products: dense QKV and output projection of 65 536
  //     rows 307 -> 288 us together.
#define HMI_ROWS(B, NB, R0, R1, RD, A_SLOT, W_SLOT, KS, COPIES, COPY)                             \
  _Pragma("unroll") for (int i = (R0); i < (R1); ++i)                                             \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) {                                              \
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[B][j], fx[i], acc[i][j], 0, 0, 0);   \
      if (RD) {                                                                                   \
        if (FWB == 1 && i == TM - 1) HMI_READ_W(0, j, W_SLOT, KS)                                 \
        if (FWB == 2 && i >= 1 && i <= TN / 2 && (j == 2 || j == 5)) HMI_READ_W((NB) % FWB, ((i - 1) * 2 + (j == 5)) % TN, W_SLOT, KS) \
        if (j == TN - 1) HMI_READ_X(i, A_SLOT, KS)                                                \
      }                                                                                           \
      {                                                                                           \
        constexpr int N_ = ((R1) - (R0)) * TN / (NW == 8 && (KS) == 0 ? 3 : 1);                   \
        const int at_ = (i - (R0)) * TN + j, c0_ = (2 * at_ * (COPIES) + N_) / (2 * N_), c1_ = (2 * (at_ + 1) * (COPIES) + N_) / (2 * N_); \
        if (c1_ > c0_ && c0_ < (COPIES)) COPY(c0_)                                                \
      }                                                                                           \
      __builtin_amdgcn_sched_barrier(0);                                                          \
    }

  // accumulators of a tile start at its bias: lane quarter q of the MFMA tiles 4 h .. 4 h + 3 holds columns
  // n0 + wn * 128 + 64 h + 16 q + (0..15), the same for all rows.
#define HMI_INIT_ACC(TR)                                                                          \
  _Pragma("unroll") for (int h = 0; h < TN / 4; ++h) {                                            \
    const int col0_ = (TR).n0 + wn * WTN + h * 64 + 16 * lq;                                      \
    const u32x4 b0_ = *reinterpret_cast<const u32x4*>((TR).bias + col0_);                         \
    const u32x4 b1_ = *reinterpret_cast<const u32x4*>((TR).bias + col0_ + 8);                     \
    _Pragma("unroll") for (int q = 0; q < 2; ++q) {                                               \
      acc[0][4 * h + q] = f32x4{bf2f(b0_[2 * q] & 0xffffu), bf2f(b0_[2 * q] >> 16), bf2f(b0_[2 * q + 1] & 0xffffu), bf2f(b0_[2 * q + 1] >> 16)}; \
      acc[0][4 * h + 2 + q] = f32x4{bf2f(b1_[2 * q] & 0xffffu), bf2f(b1_[2 * q] >> 16), bf2f(b1_[2 * q + 1] & 0xffffu), bf2f(b1_[2 * q + 1] >> 16)}; \
    }                                                                                             \
  }                                                                                               \
  _Pragma("unroll") for (int i = 1; i < TM; ++i)                                                  \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) acc[i][j] = acc[0][j];

  // One stage: two k-steps of 32, and a barrier behind the first row of the second one's products, where this wavefront has all
  // of the stage in registers.  A wavefront's L1 takes 66 bytes a clock for the whole compute unit, a 1 KB copy every 16 clocks,
  // and a wavefront that issues them faster stands still with its MFMAs: the copies are spread.  The weights of stage s + 2 go
  // between the products of the first k-step (into the slot of stage s - 1), the activations of stage s + 2 between those of
  // the second one, behind the barrier that frees the slot of stage s.
  // MODE says where they come from:
  //   0: the current tile (s <= KT-4)
  //   1: (s = KT-3) the current tile; the tile claimed for the round after next goes into the mailbox
  //   2: (s = KT-2) the next tile's stage 0; its weights only behind the barrier, so that nothing is in flight in front of it
  //      and the mailbox store is done
  //   3: (s = KT-1) the next tile's weight stage 1; no activations: the freed slots serve the epilogue first
#define HMI_COPY_W(C) HMI_COPY(w_buf_, w_at_, b_off, W_RING + wf_, C, 1)
#define HMI_COPY_A(C) HMI_COPY(a_buf, (s + 2) * ROW_BYTES, cur.a_off, fa_, C, 1)
#define HMI_COPY_AW(C) { if ((C) < LD) { HMI_COPY(a_buf, 0, nxt.a_off, fa_, (C) % LD, 1) } else { HMI_COPY(w_buf_, 0, b_off, W_RING + wf_, (C) % LD, 1) } }
#define HMI_COPY_NONE(C) {}
#define HMI_ITER(MODE)                                                                            \
  {                                                                                               \
    const int wf_ = w_rd == 0 ? (W_STAGES - 1) * STAGE_BYTES : w_rd - STAGE_BYTES;   /* the slot of stage s - 1, and of s + 2 */ \
    const buffer_t w_buf_ = buffer_at(((MODE) < 2 ? cur.Wb : nxt.Wb) - 3072);                     \
    const int w_at_ = (MODE) < 2 ? (s + 2) * ROW_BYTES : ROW_BYTES;                               \
    constexpr int WC = (MODE) == 2 ? 0 : LD;                                                      \
    if (wave_active) {                                                                            \
      HMI_ROWS(0, 1, 0, TM, 1, a_rd, w_rd, 1, WC, HMI_COPY_W)                                     \
      HMI_ROWS(FWB - 1, 0, 0, 1, 0, 0, 0, 0, 0, HMI_COPY_NONE)                                    \
    } else {                                                                                      \
      HMI_COPY(w_buf_, w_at_, b_off, W_RING + wf_, 0, WC)                                         \
    }                                                                                             \
    HMI_WAIT_LGKMCNT0();          /* this wavefront no longer reads stage s from LDS */           \
    if ((MODE) == 2) HMI_WAIT_VMCNT(0);              /* its copies of stage s+1 (both operands) have landed: nothing newer, */ \
    else HMI_WAIT_VMCNT(LD);                          /* or the weights of stage s+2 */            \
    __builtin_amdgcn_s_barrier(); /* ... everybody's, and nobody reads stage s any more */        \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    if ((MODE) == 1 && claimer) __hip_atomic_store(mailbox, claimed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); \
    if ((MODE) == 2) mail = __hip_atomic_load(mailbox, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  \
    const int fa_ = a_rd, fw_ = w_rd;                                                             \
    a_rd ^= STAGE_BYTES;                                                                          \
    w_rd = w_rd == (W_STAGES - 1) * STAGE_BYTES ? 0 : w_rd + STAGE_BYTES;                         \
    if ((MODE) == 3) {                                                                            \
      patch_a = fa_; patch_w = fw_;                                                               \
      if (wave_active) { HMI_ROWS(FWB - 1, 0, 1, TM, 0, 0, 0, 0, 0, HMI_COPY_NONE) }              \
    } else {                                                                                      \
      if (wave_active) {                                                                          \
        HMI_READ_X(0, a_rd, 0)                                                                    \
        if ((MODE) == 2) HMI_ROWS(FWB - 1, 0, 1, TM, 1, a_rd, w_rd, 0, 2 * LD, HMI_COPY_AW)       \
        else HMI_ROWS(FWB - 1, 0, 1, TM, 1, a_rd, w_rd, 0, LD, HMI_COPY_A)                        \
      } else {                                                                                    \
        if ((MODE) == 2) { HMI_COPY(a_buf, 0, nxt.a_off, fa_, 0, LD) HMI_COPY(w_buf_, 0, b_off, W_RING + wf_, 0, LD) } \
        else HMI_COPY(a_buf, (s + 2) * ROW_BYTES, cur.a_off, fa_, 0, LD)                          \
      }                                                                                           \
    }                                                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                            \
  }

  // ---- prologue of the first tile: stages 0 and 1 in the order in which the steady state issues them
  HMI_INIT_ACC(cur)
  {
    const buffer_t w_buf = buffer_at(cur.Wb - 3072);
    HMI_COPY(w_buf, 0, b_off, W_RING, 0, LD)
    HMI_COPY(a_buf, 0, cur.a_off, 0, 0, LD)
    HMI_COPY(w_buf, ROW_BYTES, b_off, W_RING + STAGE_BYTES, 0, LD)
    HMI_COPY(a_buf, ROW_BYTES, cur.a_off, STAGE_BYTES, 0, LD)
  }
  HMI_WAIT_VMCNT(2 * LD);
  __builtin_amdgcn_s_barrier();
  bool wave_active = wm * WTM < cur.rows;
  int patch_a = 0, patch_w = 0;

  for (;;) {
    // ================= main loop of the current tile =================
    {
      int s = 0;
      if (wave_active) {                                       // the first k-step's fragments
#pragma unroll
        for (int j = 0; j < TN; ++j) HMI_READ_W(0, j, w_rd, 0)
#pragma unroll
        for (int i = 0; i < TM; ++i) HMI_READ_X(i, a_rd, 0)
      }
      for (; s < KT - 3; ++s) HMI_ITER(0)
      HMI_ITER(1)
      HMI_ITER(2)
      HMI_ITER(3)
    }

    // ================= epilogue of the current tile =================
    // Results cross LDS so that whole lines of C are read and written (straight from the accumulators, 64 bytes of a row at a
    // time, launches took 6 to 10 % longer): units of 16 rows, 256 bytes of each (all 128 columns as bf16, or 64 of them as fp32),
    // a patch of 4 KB a unit, of which a wavefront has as many as its own slices of the two slots hold that stage KT-1
    // occupied.  A row keeps its 16-byte chunk c at chunk position c ^ row; read back, 16 lanes hold a row, 4 rows a step.
    // While a unit is read the next one is written and later ones' residuals are on their way.  Results that get a residual added
    // cross the patch in fp32 even if they are stored as bf16, so that they are rounded once, after the addition.
    // Rows past the end of a short tile are copies of its last row, results and residuals too, and are stored where that is
    // (same data to the same address: harmless).
    if (wave_active) {
      constexpr bool RESID = EPI == EPI_BIAS_RESID, STAGE_F32 = OUT_F32 || RESID;
      constexpr int PASSES = STAGE_F32 ? 2 : 1, UNITS = TM * PASSES;
      constexpr int AHEAD = RESID ? 2 : 1;                   // units whose residuals are asked for ahead (3 and 4 spill: 4 % longer)
      const int c = lane & 15, rq = lane >> 4;
      unsigned char* const slice_a = smem + patch_a + wave * WAVE_SLICE;
      unsigned char* const slice_w = smem + W_RING + patch_w + wave * WAVE_SLICE;
      const int put_at = l16 * 256 + (((STAGE_F32 ? lq * 4 : lq * 2) ^ l16) << 4), get_at = rq * 256 + ((c ^ rq) << 4);
      const int col = cur.n0 + wn * WTN + c * (STAGE_F32 ? 4 : 8);
      uint32_t orow[TM][4];
      f32x4 rv32[RESID && RESID_F32 ? AHEAD + 1 : 1][4];
      u32x2 rv16[RESID && !RESID_F32 ? AHEAD + 1 : 1][4];
#define HMI_PATCH(U) (NW == 8 ? ((U) & 1 ? slice_w : slice_a) : ((U) & 2 ? slice_w : slice_a) + ((U) & 1) * 4096)
#define HMI_UNIT_ROWS(U)                                                                          \
  if ((U) % PASSES == 0) {                                                                        \
    _Pragma("unroll") for (int it = 0; it < 4; ++it)                                              \
      orow[(U) / PASSES][it] = (uint32_t)__shfl(cur.out_row[(U) / PASSES >> 2], ((U) / PASSES & 3) * 16 + it * 4 + rq, 64); \
  }
#define HMI_UNIT_RESID(U)                                                                         \
  _Pragma("unroll") for (int it = 0; it < 4; ++it) {                                              \
    const size_t at_ = (size_t)orow[(U) / PASSES][it] * g.ldr + col + (U) % PASSES * 64;          \
    if constexpr (RESID_F32) rv32[(U) % (AHEAD + 1)][it] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.resid) + at_); \
    else rv16[(U) % (AHEAD + 1)][it] = *reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(g.resid) + at_); \
  }
#define HMI_UNIT_PUT(U)                                                                           \
  _Pragma("unroll") for (int jt = 0; jt < 4; ++jt) {                                              \
    if constexpr (STAGE_F32) {                                                                    \
      *reinterpret_cast<f32x4*>(HMI_PATCH(U) + (put_at ^ (jt << 4))) = acc[(U) / PASSES][(U) % PASSES * 4 + jt]; \
    } else {                                                                                      \
      u32x4 h_;                                                                                   \
      _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                             \
        float v0 = acc[U][2 * jt + (e >> 1)][2 * (e & 1)], v1 = acc[U][2 * jt + (e >> 1)][2 * (e & 1) + 1]; \
        if (EPI == EPI_BIAS_GELU) { v0 = gelu_poly(v0); v1 = gelu_poly(v1); }                     \
        else if (EPI == EPI_BIAS_RELU) { v0 = fmaxf(v0, 0.0f); v1 = fmaxf(v1, 0.0f); }            \
        h_[e] = pack_bf16(v0, v1);                                                                \
      }                                                                                           \
      *reinterpret_cast<u32x4*>(HMI_PATCH(U) + (put_at ^ ((((jt >> 1) << 3) | (jt & 1)) << 4))) = h_; \
    }                                                                                             \
  }
      static_assert(EPI == EPI_BIAS_RESID || !OUT_F32, "fp32 results are sums with residuals");
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        HMI_UNIT_ROWS(u)
        if constexpr (RESID) HMI_UNIT_RESID(u)
      }
      if (NW == 4) {       // the rows still to come stay where the MFMAs left them (the AGPR half) until their turn
#pragma unroll
        for (int i2 = 1; i2 < TM; ++i2)
#pragma unroll
          for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i2][j]));
      }
      HMI_UNIT_PUT(0)
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        const int i = u / PASSES;
        if (wm * WTM + i * 16 >= cur.rows) break;
        u32x4 got[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) got[it] = *reinterpret_cast<const u32x4*>(HMI_PATCH(u) + (get_at ^ (it << 6)) + it * 1024);
        if (NW == 4) {
#pragma unroll
          for (int i2 = (u + 1) / PASSES + 1; i2 < TM; ++i2)
#pragma unroll
            for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i2][j]));
        }
        if (u + 1 < UNITS) HMI_UNIT_PUT(u + 1)
        if (u + AHEAD < UNITS) {
          HMI_UNIT_ROWS(u + AHEAD)
          if constexpr (RESID) HMI_UNIT_RESID(u + AHEAD)
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const size_t off = (size_t)orow[i][it] * g.ldc + col + u % PASSES * 64;
          if constexpr (STAGE_F32) {
            f32x4 v = __builtin_bit_cast(f32x4, got[it]);
            if constexpr (RESID && RESID_F32) v += rv32[u % (AHEAD + 1)][it];
            else if constexpr (RESID) {
              const u32x2 r = rv16[u % (AHEAD + 1)][it];
              v += f32x4{bf2f(r[0] & 0xffffu), bf2f(r[0] >> 16), bf2f(r[1] & 0xffffu), bf2f(r[1] >> 16)};
            }
            const u32x2 hh = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            if (OUT_F32) HMI_STORE_OUT(reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + off), v);
            else HMI_STORE_OUT(reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.C) + off), hh);
            if (HAS_C2) HMI_STORE_OUT(reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.C2) + off), hh);
          } else {
            HMI_STORE_OUT(reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C) + off), got[it]);
            if (HAS_C2) HMI_STORE_OUT(reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C2) + off), got[it]);
          }
        }
      }
#undef HMI_PATCH
#undef HMI_UNIT_ROWS
#undef HMI_UNIT_RESID
#undef HMI_UNIT_PUT
    }

    // ================= move on to the next tile =================
    w = w_next;
    if (w >= w_end || --budget <= 0) break;
    w_next = w_base + 2 * n_local + __builtin_amdgcn_readfirstlane(mail);
    if (claimer) claimed = atomicAdd(claim_ctr, 1);
    cur = nxt;
    wave_active = wm * WTM < cur.rows;
    HMI_INIT_ACC(cur)
    // the copies that were held back at the last stage (the new tile's activation stage 1) go into the slot the epilogue
    // just used, as its weight stage 2 will in its first stage; a wavefront's copies fill only its own slice of a slot,
    // which is its own staging patch: no barrier
    HMI_COPY(a_buf, ROW_BYTES, cur.a_off, patch_a, 0, LD)
    load_tile(g, rt, w_next < w_end ? w_next : w, wave, lane, nxt);
  }
  HMI_WAIT_VMCNT(0);   // none of this workgroup's copies may outlive it
  finish_workgroup(rt, xcd, n_local);
}

template <int NW, int EPI, bool OUT_F32, bool RESID_F32, bool HAS_C2>
void launch_one(const GemmArgs& g, const Route& rt, hipStream_t s) {
  auto kern = gemm_bf16_p256_kernel<NW, EPI, OUT_F32, RESID_F32, HAS_C2>;
  const int n_cu = rt.n_cu >= kXcds ? rt.n_cu : 256;
  const int nt_n = g.n_out / BN;
  const long long total = (long long)g.n_mtiles * nt_n;
  if (total <= 0) return;
  const int per_xcd = (int)((total + kXcds - 1) / kXcds);
  const int local = per_xcd < n_cu / kXcds ? per_xcd : n_cu / kXcds;   // workgroups per XCD: at most one per compute unit
  hipLaunchKernelGGL(kern, dim3(local * kXcds), dim3(Geo<NW>::NTH), LDS_BYTES, s, g, rt, (int)total, per_xcd);
}

template <int NW, int EPI, bool OUT_F32, bool RESID_F32, bool HAS_C2>
void allow_lds() {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_bf16_p256_kernel<NW, EPI, OUT_F32, RESID_F32, HAS_C2>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
}

// Which geometry a launch gets (measured on the FFN and encoder workloads): launches that add a residual (output
// projection, second FFN GEMM) run with four wavefronts, 3-6 % faster there (no spills in their fp32 epilogue, a
// long main loop in the second FFN GEMM); bias-only and activation launches keep eight, whose two wavefronts per
// SIMD overlap each other's epilogue latencies (the first FFN GEMM is 11 % slower with four).
#ifndef WP
#define WP 8
#endif
#ifndef WR
#define WR 4
#endif
constexpr int kWavesPlain = WP, kWavesResid = WR;
}  // namespace

// every instantiation launch_gemm_bf16_p256 can pick
void init_gemm_bf16_p256_kernels() {
  allow_lds<kWavesPlain, EPI_BIAS, false, false, true>();   allow_lds<kWavesPlain, EPI_BIAS, false, false, false>();
  allow_lds<kWavesPlain, EPI_BIAS_GELU, false, false, false>();
  allow_lds<kWavesPlain, EPI_BIAS_RELU, false, false, false>();
  allow_lds<kWavesResid, EPI_BIAS_RESID, true, true, true>();   allow_lds<kWavesResid, EPI_BIAS_RESID, true, true, false>();
  allow_lds<kWavesResid, EPI_BIAS_RESID, true, false, true>();  allow_lds<kWavesResid, EPI_BIAS_RESID, true, false, false>();
  allow_lds<kWavesResid, EPI_BIAS_RESID, false, true, false>(); allow_lds<kWavesResid, EPI_BIAS_RESID, false, false, false>();
}

// Preconditions (checked by the caller): n_out % 256 == 0, k % 64 == 0, k >= 192,
// which_tiles names a list of 256-row m-tiles, all operands 16-byte aligned,
// byte offsets of A rows and of W rows inside a slot below 4 GB.
void launch_gemm_bf16_p256(const GemmArgs& g, const Route& rt, hipStream_t s) {
  const bool c2 = g.C2 != nullptr;
  switch (g.epi) {
    case EPI_BIAS:
      return c2 ? launch_one<kWavesPlain, EPI_BIAS, false, false, true>(g, rt, s) : launch_one<kWavesPlain, EPI_BIAS, false, false, false>(g, rt, s);
    case EPI_BIAS_GELU:
      return launch_one<kWavesPlain, EPI_BIAS_GELU, false, false, false>(g, rt, s);
    case EPI_BIAS_RELU:
      return launch_one<kWavesPlain, EPI_BIAS_RELU, false, false, false>(g, rt, s);
    default:
      if (g.out_f32) {
        if (g.resid_f32) return c2 ? launch_one<kWavesResid, EPI_BIAS_RESID, true, true, true>(g, rt, s) : launch_one<kWavesResid, EPI_BIAS_RESID, true, true, false>(g, rt, s);
        return c2 ? launch_one<kWavesResid, EPI_BIAS_RESID, true, false, true>(g, rt, s) : launch_one<kWavesResid, EPI_BIAS_RESID, true, false, false>(g, rt, s);
      }
      if (g.resid_f32) return launch_one<kWavesResid, EPI_BIAS_RESID, false, true, false>(g, rt, s);
      return launch_one<kWavesResid, EPI_BIAS_RESID, false, false, false>(g, rt, s);
  }
}

}  // namespace hmi
