// The paper's bottleneck adapter over a mixed-tenant batch (Sec. 3.2.2, batched as in
// Sec. 6.3), one kernel:  Y = X + Up_t(ReLU(Down_t(X))),  Down_t: d -> 64,  Up_t: 64 -> d,
// bf16 storage, fp32 accumulation, Y rounded once.
//
// With a 64-wide bottleneck the block moves 4 d bytes per token for 256 d flops per token:
// far below the machine balance, so the kernel is organised around the HBM stream and not
// around the MFMA pipes.  A workgroup (8 wavefronts, one per compute unit) walks a
// contiguous range of 32-row units of the tenant-sorted batch.  A unit's rows are copied
// straight into LDS (full 128-byte lines, rows gathered through row_src), both
// projections run out of LDS and registers, the result replaces the rows in LDS, and the
// same rows stream back out with 16-byte stores: X is read once and Y written once.
// Two row buffers alternate, so the copies of the unit after next run under this unit's
// arithmetic; wavefronts 0-3 issue the copies and wavefronts 4-7 the stores, which keeps
// each wavefront's memory counter to one kind of access (loads return in order among
// loads only).
//
// The tenant's two matrices live in registers for as long as the units stay in one
// segment: at load time they are laid out in MFMA operand order (pack_adapter_operand
// below), so a reload is a handful of 1 KB coalesced reads.
//
//   Down:  wavefront (cb, kq) multiplies the unit by column block cb of Down over its
//          quarter kq of d (k-steps 2 kq and 2 kq + 1 of every eight); the four partial sums per element meet in LDS (fixed order of
//          addition), where bias and ReLU are applied and the 32 x 64 result is rounded to
//          bf16 once, as the two-kernel path does between its GEMMs.
//   Up:    wavefront w owns output columns [w d/8, (w+1) d/8); it adds bias and the
//          unit's own rows from LDS and writes the rounded sum back in place.
//
// Inside a shared layer the block is followed by the layer's LayerNorm over (residual stream + Y): a workgroup has whole
// rows of Y in LDS, so it does that too (LN_* below), with the arithmetic of the vector LayerNorm kernel, to the bit: a wavefront
// takes rows w, w + 8, .. of the unit, as far as there are any.  Y itself is then never written.  Half of a unit's residual
// rows are asked for a unit ahead, the others behind the down-projection.
// Measured: 65 536 rows of d = 768 with an fp32 residual 55 + 75 us as two kernels, 120 as one.
//
// In small launches (a unit a workgroup, ONE below) it is a chain of latencies on top of the 0.2 MB of matrices, which take a
// compute unit 1.4 us.  The chain is kept short: each wavefront finds its unit by itself, from the segments' ends; everything
// is asked for before anything is waited for; sums over a wavefront stay in registers.  141 rows of two tenants with LayerNorm
// 13.4 -> 8.3 us, a decode step's 7 rows 13.3 -> 9.2 and 256 rows of 137 tenants 15.8 -> 12.6 (their 27 MB come from HBM),
// 2 664 rows 15.5 -> 11.8.
#include "hmi_kernels.h"

#include "wave.h"

namespace hmi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

constexpr int kXcds = 8;
constexpr int RT = 32;            // rows of a unit at most
constexpr int RANK = 64;          // bottleneck width
constexpr int NTH = 512;
constexpr int MAX_UNITS = 64;     // units one workgroup may be handed
constexpr int MAX_SEGS = 256;     // tenants of a launch whose units are counted exactly (four per lane)
constexpr int PART_BYTES = 4 * RT * RANK * 4;   // four partial sums of the 32 x 64 bottleneck, fp32
constexpr int MID_BYTES = RT * RANK * 2;
constexpr int RS_BYTES = MAX_UNITS * RT * 4;
constexpr int DESC_BYTES = (MAX_UNITS * 4 + 4) * 4;

__device__ __forceinline__ float bf2f(uint32_t u16) { return __uint_as_float(u16 << 16); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// A tenant's matrices.  In a decode step a tenant has a row or two: its 0.2 MB are read by one workgroup, once, and only push
// the shared layers' weights out of the L2s (with the hint a step through six shared layers is 3 % shorter); over a full batch
// the workgroups that hold the tenant's other rows read them again, from L2, and there the plain load is the faster one.
template <bool ONCE>
__device__ __forceinline__ bf16x8 load_w(const bf16x8* p) {
  if (ONCE) return __builtin_nontemporal_load(p);
  return *p;
}

// What happens to the finished rows of a unit.
enum Out : int { OUT_STREAM, LN_RESID_BF16, LN_RESID_F32 };

// Four columns of a residual row as they are loaded, and as fp32.
template <bool F32> struct Four { typedef u16x4 type; };
template <> struct Four<true> { typedef f32x4 type; };
__device__ __forceinline__ f32x4 to_f32(u16x4 h) { return f32x4{bf2f(h[0]), bf2f(h[1]), bf2f(h[2]), bf2f(h[3])}; }
__device__ __forceinline__ f32x4 to_f32(f32x4 v) { return v; }

template <int NV, bool ONE>
struct Shape {
  static constexpr int CH = NV * 32;          // 16-byte chunks of a row (d = 256 NV)
  static constexpr int ROWB = CH * 16;
  static constexpr int BUF = RT * ROWB;
  static constexpr int KS = NV * 16;          // 16-wide k-steps over d
  static constexpr int KSW = KS / 4;          // ... per wavefront of the down-projection
  static constexpr int NJ = RT * CH / 256;    // copies (stores) per lane and unit
  static constexpr int OFF_PART = (ONE ? 1 : 2) * BUF;
  static constexpr int OFF_MID = OFF_PART + PART_BYTES;
  static constexpr int OFF_RS = OFF_MID + MID_BYTES;
  static constexpr int OFF_DESC = OFF_RS + (ONE ? RT * 4 : RS_BYTES);
  static constexpr int OFF_NORM = OFF_DESC + (ONE ? 0 : DESC_BYTES);   // LayerNorm gain, then shift, as stored
  static constexpr int OFF_BIAS = OFF_NORM + 2 * ROWB;     // the tenant's up-projection bias
  static constexpr int LDS = OFF_BIAS + ROWB;
  static_assert(LDS <= 163840, "LDS");
};

// LDS layouts (all XOR swizzles act on 16-byte chunk indices, so that the 16 lanes that
// the LDS serves together hit 16 different chunks of its 256-byte bank line):
//   row buffer   row r, position p holds the row's chunk p ^ (r & 15)
//   partial sum  [kq][row r][16 chunks of 4 fp32], chunk q at position q ^ (r & 15)
//   bottleneck   row r is 128 bytes (64 bf16), chunk c at position c ^ ((r >> 1) & 7)
// ONCE: the tenants' matrices are loaded with the non-temporal hint (load_w above); OUT_STREAM: so are the result's stores.
// Both are compile-time: a run-time choice between a hinted and a plain access to one address is merged into the plain one.
// ONE: a workgroup is one unit (a launch of at most as many units as compute units).  It is straight code then, in
// which the compiler waits for each load where it is needed; in the loop of the general form, where waits hold for all turns, the
// matrices have to be there before the first one.
template <int NV, bool ONCE, int OUT, bool ONE>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(2, 2)))
void adapter_bf16_kernel(AdapterArgs a, Route rt) {
  using S = Shape<NV, ONE>;
  constexpr bool LN = OUT != OUT_STREAM;
  typedef typename Four<OUT == LN_RESID_F32>::type four_t;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int j = lane & 31, h = lane >> 5;           // MFMA: token row of the unit, k-half
  int* desc = reinterpret_cast<int*>(smem + S::OFF_DESC);
  int* rs = reinterpret_cast<int*>(smem + S::OFF_RS);

  // ---- which units are mine and where their rows live.  Every wavefront finds out by itself (a barrier less in a chain of
  //      them); the first one writes it down.
  int m = 1, first_row, first_rows, cur_slot;
  if (ONE) {
    // Workgroups are dealt to the XCDs round robin; an XCD's take neighbouring units, so that a tenant's matrices are fetched into one
    // L2 and not into all eight (2 664 rows of 37 requests 14.1 us -> 11.8; in the general form, where a workgroup has several units
    // and mostly several tenants, launches got 1 to 5 % longer).
    const int xcd = blockIdx.x % kXcds, n_wgs = gridDim.x;
    const int wg = xcd * (n_wgs / kXcds) + min(xcd, n_wgs % kXcds) + (int)blockIdx.x / kXcds;
    // unit wg of the segments' units in order: a lane counts those of four segments
    int cut[5], units = 0;
#pragma unroll
    for (int e = 0; e < 5; ++e) cut[e] = rt.seg_tok_off[min(4 * lane + e, a.n_segs)];
#pragma unroll
    for (int e = 0; e < 4; ++e) units += (cut[e + 1] - cut[e] + a.unit_rows - 1) >> a.unit_shift;
    const int upto = wave_incl_scan(units), b = wg;
    const int l0 = __builtin_ctzll(__ballot(upto > b));       // (the launch has exactly as many workgroups as there are units)
    int u = b - (upto - units), seg = 4 * lane, row0 = 0, rows = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = (cut[e + 1] - cut[e] + a.unit_rows - 1) >> a.unit_shift;
      if (u >= 0 && u < n) { seg = 4 * lane + e; row0 = cut[e] + (u << a.unit_shift); rows = min(a.unit_rows, cut[e + 1] - row0); }
      u -= n;
    }
    first_row = __builtin_amdgcn_readlane(row0, l0);
    first_rows = __builtin_amdgcn_readlane(rows, l0);
    cur_slot = rt.seg_slot[__builtin_amdgcn_readlane(seg, l0)];
  } else {
    const int* const tile_seg = rt.tile_seg[a.which_tiles];
    const int* const tile_row0 = rt.tile_row0[a.which_tiles];
    const int u_begin = blockIdx.x * a.units_each + min((int)blockIdx.x, a.units_more);
    const int n_units = a.units_each + ((int)blockIdx.x < a.units_more);
    int row0 = 0, rows = 0, slot = 0;
    if (lane < n_units) {
      const int u = u_begin + lane, t = u >> 2, seg = tile_seg[t];
      row0 = tile_row0[t] + (u & 3) * RT;
      rows = min(RT, rt.seg_tok_off[seg + 1] - row0);
      slot = rt.seg_slot[seg];
    }
    const unsigned long long mask = __ballot(rows > 0);
    if (mask == 0) return;
    m = __popcll(mask);
    if (wave == 0 && rows > 0) {
      const int pos = __popcll(mask & ((1ull << lane) - 1ull));
      desc[pos * 4 + 0] = row0; desc[pos * 4 + 1] = rows; desc[pos * 4 + 2] = slot;
    }
    const int l0 = __builtin_ctzll(mask);
    first_row = __builtin_amdgcn_readlane(row0, l0);
    first_rows = __builtin_amdgcn_readlane(rows, l0);
    cur_slot = __builtin_amdgcn_readlane(slot, l0);
  }
  const int cb = wave & 1, kq = wave >> 1;    // down-projection role
  bf16x8 wd[S::KSW], wu[NV][4];
  u32x4 bu = {};     // up-projection bias of my 32 NV columns, packed: eight of them in each of the first 4 NV lanes
  u32x2 bd;          // down-projection bias of my four bottleneck columns, packed

  // copies unit ui into row buffer b (wavefronts 0-3; a lane moves NJ chunks of 16 bytes)
  const char* X = reinterpret_cast<const char*>(a.X);
  char* Y = reinterpret_cast<char*>(a.Y);
  // A lane's NJ = 4 NV chunks of a unit: chunk jj * 256 + t8 with t8 = tid mod 256.  256 NV
  // chunks are exactly 8 rows, so chunk (NV g + r3) * 256 + t8 lies in row 8 g + ro[r3] at a
  // row position that does not depend on g; sw[r3] is that position swizzled for g even.
  int t8, ro[NV], sw[NV];
  auto place = [&]() {
    t8 = tid & 255;
#pragma unroll
    for (int r3 = 0; r3 < NV; ++r3) {
      const int c = r3 * 256 + t8;
      ro[r3] = c / S::CH;
      sw[r3] = ((c % S::CH) ^ ro[r3]) << 4;
    }
  };
  place();
#define HMI_ISSUE_COPIES(UI, B)                                                                    \
  {                                                                                                \
    _Pragma("unroll") for (int g_ = 0; g_ < 4; ++g_)                                               \
      _Pragma("unroll") for (int r3 = 0; r3 < NV; ++r3) {                                          \
        const char* src_ = X + (size_t)rs[(UI) * RT + 8 * g_ + ro[r3]] * S::ROWB + (sw[r3] ^ ((g_ & 1) << 7)); \
        lds_ptr_t dst_ = (lds_ptr_t)(smem + (B) * S::BUF + ((g_ * NV + r3) * 256 + wave * 64) * 16); \
        __builtin_amdgcn_global_load_lds((glb_ptr_t)src_, dst_, 16, 0, 0);                         \
      }                                                                                            \
  }

#define HMI_LOAD_WD(SLOT)                                                                          \
  {                                                                                                \
    const bf16x8* pwd = reinterpret_cast<const bf16x8*>(a.pool + (size_t)(SLOT) * a.slot_stride + a.wd_off) + \
                        ((cb * S::KS + 2 * kq) * 64 + lane);                                       \
    _Pragma("unroll") for (int s = 0; s < S::KSW; ++s)                                             \
      wd[s] = load_w<ONCE>(pwd + ((s >> 1) * 8 + (s & 1)) * 64);   /* k-step 8 (s / 2) + 2 kq + s % 2 */ \
  }
#define HMI_LOAD_BD(SLOT)                                                                          \
  bd = *reinterpret_cast<const u32x2*>(a.pool + (size_t)(SLOT) * a.slot_stride + a.bd_off + (tid & 15) * 8);
#define HMI_LOAD_WU(SLOT)                                                                          \
  {                                                                                                \
    const char* base = a.pool + (size_t)(SLOT) * a.slot_stride;                                    \
    const bf16x8* pwu = reinterpret_cast<const bf16x8*>(base + a.wu_off) + (wave * NV * 4 * 64 + lane); \
    _Pragma("unroll") for (int c = 0; c < NV; ++c)                                                 \
      _Pragma("unroll") for (int s = 0; s < 4; ++s) wu[c][s] = load_w<ONCE>(pwu + (c * 4 + s) * 64); \
    if (lane < 4 * NV) bu = *reinterpret_cast<const u32x4*>(base + a.bu_off + (wave * 4 * NV + lane) * 16); \
  }

  // A compute unit takes 66 bytes a clock, and a unit's matrices are most of its bytes (1.4 us of them): they are asked for as
  // early as may be, in the order in which they are needed (loads return in order): Down, the first unit's rows (through
  // registers, so that nothing behind them has to be waited for with them), its residual rows, Up.
  const int my_src = rt.row_src[first_row + min(lane & 31, first_rows - 1)];
  auto row_of = [&](int idx) {             // of unit idx / 32: surplus rows of a short unit repeat its last row
    const int u = idx >> 5, r = idx & 31;
    return rt.row_src[desc[u * 4] + min(r, desc[u * 4 + 1] - 1)];
  };
  int src = 0;                             // row tid of the workgroup's units
  if (!ONE) {
    HMI_BARRIER();                         // desc
    if (tid < m * RT) src = row_of(tid);
  }
  HMI_LOAD_WD(cur_slot)
  __builtin_amdgcn_sched_barrier(0);
  u32x4 x0[2 * NV];
#pragma unroll
  for (int jj = 0; jj < 2 * NV; ++jj) {
    const int c = jj * NTH + tid, row = c / S::CH;
    const int from = __shfl(my_src, row, 64);
    if (row < first_rows) x0[jj] = *reinterpret_cast<const u32x4*>(X + (size_t)from * S::ROWB + (c % S::CH) * 16);
  }
  u32x4 norm = {};
  if (LN && tid < 2 * S::CH) norm = reinterpret_cast<const u32x4*>(tid < S::CH ? a.ln_g : a.ln_b)[tid < S::CH ? tid : tid - S::CH];
  __builtin_amdgcn_sched_barrier(0);
  // The residual rows that this wavefront normalises: rows wave + 8 q of a unit, as far as it has them, columns 256 v + 4 lane
  // .. (q = 0, 1 are asked for a unit ahead, the others behind the down-projection; all four ahead do not fit the registers)
  four_t res[LN ? 4 : 1][LN ? NV : 1];
#define HMI_LOAD_RESID_ROW(Q, ROW)                                                                 \
  {                                                                                                \
    const size_t row_ = (size_t)__builtin_amdgcn_readfirstlane(ROW) * (S::CH * 8);                 \
    _Pragma("unroll") for (int v = 0; v < NV; ++v) {                                               \
      if (OUT == LN_RESID_F32) res[Q][v] = *reinterpret_cast<const four_t*>(static_cast<const float*>(a.resid) + row_ + v * 256 + lane * 4); \
      else res[Q][v] = *reinterpret_cast<const four_t*>(static_cast<const uint16_t*>(a.resid) + row_ + v * 256 + lane * 4); \
    }                                                                                              \
  }
#define HMI_LOAD_RESID(UI, Q0, ROWS)                                                               \
  _Pragma("unroll") for (int q = (Q0); q < (Q0) + 2; ++q)                                          \
    if (wave + 8 * q < (ROWS)) HMI_LOAD_RESID_ROW(q, rs[(UI) * RT + wave + 8 * q])
  if (LN) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (wave + 8 * q < first_rows) HMI_LOAD_RESID_ROW(q, __builtin_amdgcn_readlane(my_src, wave + 8 * q))
  }
  HMI_LOAD_BD(cur_slot)
  HMI_LOAD_WU(cur_slot)
  __builtin_amdgcn_sched_barrier(0);
  // the units' row numbers and the LayerNorm's parameters to LDS, then the first unit's rows
  if (ONE && wave == 0 && lane < RT) rs[lane] = my_src;
  if (!ONE && tid < m * RT) rs[tid] = src;
  if (LN && tid < 2 * S::CH) reinterpret_cast<u32x4*>(smem + S::OFF_NORM)[tid] = norm;
#pragma unroll
  for (int jj = 0; jj < 2 * NV; ++jj) {
    const int c = jj * NTH + tid, row = c / S::CH;
    if (row < first_rows) *reinterpret_cast<u32x4*>(smem + row * S::ROWB + (((c % S::CH) ^ (row & 15)) << 4)) = x0[jj];
  }
  HMI_BARRIER();
  if (!ONE) {
    if (wave < 4 && m > 1) HMI_ISSUE_COPIES(1, 1)
    if (m * RT > NTH) {
      for (int idx = NTH + tid; idx < m * RT; idx += NTH) rs[idx] = row_of(idx);   // read behind the loop's first barrier at the earliest
    }
#pragma unroll
    for (int s = 0; s < S::KSW; ++s) asm volatile("" :: "v"(wd[s]));       // (waited for here)
#pragma unroll
    for (int c = 0; c < NV; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) asm volatile("" :: "v"(wu[c][s]));
    asm volatile("" :: "v"(bu), "v"(bd));
  }

  for (int i = 0; i < m; ++i) {
    const int b = i & 1;
    unsigned char* buf = smem + b * S::BUF;
    if (LN) {   // the addresses made from the thread's number are made anew for each unit: there are no registers to keep them in
      asm volatile("" : "+v"(tid));
      lane = tid & 63; j = lane & 31; h = lane >> 5;
      place();
    }
    const int rows = ONE ? first_rows : desc[i * 4 + 1];
    // the tenant of the next unit, if it is another one: its matrices replace this unit's as
    // soon as each has been used for the last time, so that the reads run under the rest of the unit
    const int next_slot = i + 1 < m ? desc[(i + 1) * 4 + 2] : cur_slot;
    const bool reload = next_slot != cur_slot;   // same for the whole workgroup
    // ---- Down: partial[kq] = X[32, my quarter of d] * Down[cb block, same quarter]^T
    {
      // my k-steps are 8 a + 2 kq + e (a = 0 .. KS/8 - 1, e = 0, 1): the row chunks 16 a + 4 kq + 2 e + h,
      // whose swizzled position inside the 256-byte group a is the same for every a
      f32x16 acc = {};
      const unsigned char* xr = buf + j * S::ROWB;
      const unsigned char* x0 = xr + (((4 * kq + h) ^ (j & 15)) << 4);
      const unsigned char* x1 = xr + (((4 * kq + 2 + h) ^ (j & 15)) << 4);
#pragma unroll
      for (int s = 0; s < S::KSW; ++s) {
        const bf16x8 xf = *reinterpret_cast<const bf16x8*>(((s & 1) ? x1 : x0) + (s >> 1) * 256);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wd[s], xf, acc, 0, 0, 0);
      }
      unsigned char* pr = smem + S::OFF_PART + kq * (RT * RANK * 4) + j * (RANK * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int q = cb * 8 + h * 4 + e;
        *reinterpret_cast<f32x4*>(pr + ((q ^ (j & 15)) << 4)) = f32x4{acc[4 * e], acc[4 * e + 1], acc[4 * e + 2], acc[4 * e + 3]};
      }
    }
    if (reload) HMI_LOAD_WD(next_slot)
    if (LN) { HMI_LOAD_RESID(i, 2, rows) }
    HMI_BARRIER();
    // ---- bottleneck: sum of the four quarters + bias, ReLU, one rounding to bf16
    {
      const int row = tid >> 4, q = tid & 15;
      const unsigned char* pr = smem + S::OFF_PART + row * (RANK * 4) + ((q ^ (row & 15)) << 4);
      f32x4 v = *reinterpret_cast<const f32x4*>(pr);
#pragma unroll
      for (int k = 1; k < 4; ++k) v += *reinterpret_cast<const f32x4*>(pr + k * (RT * RANK * 4));
      v += f32x4{bf2f(bd[0] & 0xFFFFu), bf2f(bd[0] >> 16), bf2f(bd[1] & 0xFFFFu), bf2f(bd[1] >> 16)};
      u32x2 o;
      o[0] = pack_bf16(fmaxf(v[0], 0.0f), fmaxf(v[1], 0.0f));
      o[1] = pack_bf16(fmaxf(v[2], 0.0f), fmaxf(v[3], 0.0f));
      *reinterpret_cast<u32x2*>(smem + S::OFF_MID + row * 128 + (((q >> 1) ^ ((row >> 1) & 7)) << 4) + (q & 1) * 8) = o;
    }
    if (reload) HMI_LOAD_BD(next_slot)
    HMI_BARRIER();
    // ---- Up: my d/8 output columns, added to the unit's rows in place
    {
      u32x4* const my_bias = reinterpret_cast<u32x4*>(smem + S::OFF_BIAS) + wave * 4 * NV;   // only this wavefront's
      if (lane < 4 * NV) my_bias[lane] = bu;
      bf16x8 mf[4];
      const unsigned char* mr = smem + S::OFF_MID + j * 128;
#pragma unroll
      for (int s = 0; s < 4; ++s) mf[s] = *reinterpret_cast<const bf16x8*>(mr + (((2 * s + h) ^ ((j >> 1) & 7)) << 4));
      unsigned char* xr = buf + j * S::ROWB;
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        f32x16 acc;
        const u32x4 b0 = my_bias[c * 4 + h * 2], b1 = my_bias[c * 4 + h * 2 + 1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] = bf2f(b0[e] & 0xFFFFu); acc[2 * e + 1] = bf2f(b0[e] >> 16);
          acc[8 + 2 * e] = bf2f(b1[e] & 0xFFFFu); acc[8 + 2 * e + 1] = bf2f(b1[e] >> 16);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wu[c][s], mf[s], acc, 0, 0, 0);
        const int p0 = (wave * NV + c) * 4 + 2 * h;
        u32x4* x0 = reinterpret_cast<u32x4*>(xr + ((p0 ^ (j & 15)) << 4));
        u32x4* x1 = reinterpret_cast<u32x4*>(xr + (((p0 + 1) ^ (j & 15)) << 4));
        const u32x4 v0 = *x0, v1 = *x1;
        u32x4 o0, o1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o0[e] = pack_bf16(acc[2 * e] + bf2f(v0[e] & 0xFFFFu), acc[2 * e + 1] + bf2f(v0[e] >> 16));
          o1[e] = pack_bf16(acc[8 + 2 * e] + bf2f(v1[e] & 0xFFFFu), acc[8 + 2 * e + 1] + bf2f(v1[e] >> 16));
        }
        *x0 = o0; *x1 = o1;
      }
    }
    if (reload) HMI_LOAD_WU(next_slot)
    cur_slot = next_slot;
    HMI_BARRIER();
    if (LN) {
      // ---- LayerNorm of (residual + adapted row), rounded as the separate kernels would pass it on
#pragma unroll
      for (int q0 = 0; q0 < 4; q0 += 2) {
        if (q0 && wave + 8 * q0 >= rows) break;
        f32x4 v[2][NV];
        float sum[2], var[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = wave + 8 * (q0 + q);
          sum[q] = 0.0f;
#pragma unroll
          for (int c = 0; c < NV; ++c) {
            const u16x4 y = *reinterpret_cast<const u16x4*>(buf + r * S::ROWB + (((c * 32 + (lane >> 1)) ^ (r & 15)) << 4) + (lane & 1) * 8);
            v[q][c] = to_f32(res[q0 + q][c]) + to_f32(y);
            sum[q] += v[q][c][0] + v[q][c][1] + v[q][c][2] + v[q][c][3];
          }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) sum[q] = wave_sum(sum[q]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          sum[q] /= (float)(NV * 256);                                 // the mean
          var[q] = 0.0f;
#pragma unroll
          for (int c = 0; c < NV; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float z = v[q][c][e] - sum[q]; var[q] += z * z; }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) var[q] = wave_sum(var[q]);
        // the next unit's rows and its tenant's matrices, before this unit's stores are in the way
        if (!ONE && q0 == 0) HMI_WAIT_VMCNT(0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = wave + 8 * (q0 + q);
          if (r < rows) {
            const float rstd = 1.0f / sqrtf(var[q] / (float)(NV * 256) + a.eps);
            const size_t at = (size_t)__builtin_amdgcn_readfirstlane(rs[i * RT + r]) * (S::CH * 8) + lane * 4;
#pragma unroll
            for (int c = 0; c < NV; ++c) {
              const u16x4* norm = reinterpret_cast<const u16x4*>(smem + S::OFF_NORM) + c * 64 + lane;
              const f32x4 gg = to_f32(norm[0]), bb = to_f32(norm[NV * 64]);
              f32x4 y;
#pragma unroll
              for (int e = 0; e < 4; ++e) y[e] = (v[q][c][e] - sum[q]) * rstd * gg[e] + bb[e];
              *reinterpret_cast<f32x4*>(a.x32 + at + c * 256) = a.x32_is_sum ? v[q][c] : y;
              *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(a.Y) + at + c * 256) = u32x2{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i + 1 < m) { HMI_LOAD_RESID(i + 1, 0, desc[(i + 1) * 4 + 1]) }
      __builtin_amdgcn_sched_barrier(0);
    } else
    // ---- wavefronts 4-7 stream the finished rows out; wavefronts 0-3 make sure the next
    //      unit's rows have landed.  After the barrier the buffer is free for unit i + 2.
    if (wave >= 4) {
      if (!ONE) HMI_WAIT_VMCNT(0);        // (the next tenant's matrices, as above)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x4 v[NV];
        int orow[NV];
#pragma unroll
        for (int r3 = 0; r3 < NV; ++r3) {
          v[r3] = *reinterpret_cast<const u32x4*>(buf + ((g * NV + r3) * 256 + t8) * 16);
          orow[r3] = rs[i * RT + 8 * g + ro[r3]];
        }
#pragma unroll
        for (int r3 = 0; r3 < NV; ++r3)
          if (8 * g + ro[r3] < rows) {
            u32x4* dst = reinterpret_cast<u32x4*>(Y + (size_t)orow[r3] * S::ROWB + (sw[r3] ^ ((g & 1) << 7)));
            // a result that goes to the caller leaves without taking lines of L2 (4.7 -> 5.0 TB/s)
            __builtin_nontemporal_store(v[r3], dst);
          }
      }
    } else if (i + 1 < m) {
      HMI_WAIT_VMCNT(0);
    }
    HMI_BARRIER();
    if (wave < 4 && i + 2 < m) HMI_ISSUE_COPIES(i + 2, b)
  }
#undef HMI_ISSUE_COPIES
#undef HMI_LOAD_WD
#undef HMI_LOAD_BD
#undef HMI_LOAD_WU
#undef HMI_LOAD_RESID
#undef HMI_LOAD_RESID_ROW
}

template <int NV, bool ONE>
decltype(&adapter_bf16_kernel<NV, false, OUT_STREAM, ONE>) pick(const AdapterArgs& a) {
  if (a.stream_out) return adapter_bf16_kernel<NV, false, OUT_STREAM, ONE>;
  if (a.resid_f32) return a.weights_once ? adapter_bf16_kernel<NV, true, LN_RESID_F32, ONE> : adapter_bf16_kernel<NV, false, LN_RESID_F32, ONE>;
  return a.weights_once ? adapter_bf16_kernel<NV, true, LN_RESID_BF16, ONE> : adapter_bf16_kernel<NV, false, LN_RESID_BF16, ONE>;
}

// log2 of the rows of the units that a launch of one unit a workgroup is cut into, or 0: the general form.
int unit_shift(const AdapterArgs& a, int n_cu) {
  // While there is a compute unit for each, the units are as small as may be: what one costs is then the traffic of its rows
  // through one of them, besides its matrices' (two requests of 101 and 40 rows with LayerNorm: 12.4 us in units of 32 rows, up
  // to 0.49 MB each, 8.3 in units of 8), and they are counted exactly (a decode step of 256 rows, the most popular tenant with 34
  // of them: 14.5 us with four units for each 128-row tile, most of them empty, 12.6 with these).  The general form does not
  // count: it has four units for every 128-row tile, and a step of 257 tenants with a row each takes 18.2 us, of 256 15.1.
  // Without LayerNorm a unit's own rows are little work and units of 16 rows only read the matrices twice: where 8-row units are
  // too many, units of 32 (two batches: 2 789 rows of d = 512, 15.3 us in units of 16, 14.1 in units of 32; 3 473 of d = 256
  // 12.3 and 11.7).
  if (a.n_segs <= MAX_SEGS)
    for (int k = 0; k < 3; ++k)   // (two workgroups a compute unit, where rows are narrow enough, load the matrices twice: 8 586 rows of d = 256 5 % slower)
      if (a.units[k] <= n_cu && !(a.stream_out && k == 1)) return 3 + k;
  return 0;
}

template <int NV>
void launch_nv(const AdapterArgs& a, const Route& rt, hipStream_t s) {
  const int n_cu = rt.n_cu >= 1 ? rt.n_cu : 256;
  if (a.n_tiles128 <= 0) return;
  AdapterArgs b = a;
  if (const int shift = unit_shift(a, n_cu)) {
    b.unit_shift = shift;
    b.unit_rows = 1 << shift;
    hipLaunchKernelGGL((pick<NV, true>(a)), dim3(a.units[shift - 3]), dim3(NTH), (Shape<NV, true>::LDS), s, b, rt);
    return;
  }
  const long long U = (long long)a.n_tiles128 * 4;
  long long grid = U < n_cu ? U : n_cu;                               // one workgroup per compute unit ...
  const long long need = (U + MAX_UNITS - 1) / MAX_UNITS;            // ... unless that hands a workgroup
  if (grid < need) grid = need;                                       //     more units than it can list
  b.units_each = (int)(U / grid);
  b.units_more = (int)(U % grid);
  hipLaunchKernelGGL((pick<NV, false>(a)), dim3((unsigned)grid), dim3(NTH), (Shape<NV, false>::LDS), s, b, rt);
}

template <int NV, bool ONE>
void allow_lds() {
  for (auto kern : {adapter_bf16_kernel<NV, false, OUT_STREAM, ONE>, adapter_bf16_kernel<NV, false, LN_RESID_BF16, ONE>,
                    adapter_bf16_kernel<NV, true, LN_RESID_BF16, ONE>, adapter_bf16_kernel<NV, false, LN_RESID_F32, ONE>,
                    adapter_bf16_kernel<NV, true, LN_RESID_F32, ONE>})
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, Shape<NV, ONE>::LDS);
}

}  // namespace

void init_adapter_bf16_kernels() {
  allow_lds<1, false>(); allow_lds<2, false>(); allow_lds<3, false>();
  allow_lds<1, true>(); allow_lds<2, true>(); allow_lds<3, true>();
}

// Operand order: 1 KB blocks, one per (32-row block, 16-wide k-step), k-steps innermost.
// Lane l of a block holds the 8 elements [16 s + 8 (l / 32), +8) of the block's row
// perm(l % 32), where perm places the rows so that output register r of lane half hh of
// the 32x32x16 MFMA is the block's row 16 hh + r.
void pack_adapter_operand(void* dst, const void* src, int rows, int cols) {
  uint16_t* o = static_cast<uint16_t*>(dst);
  const uint16_t* in = static_cast<const uint16_t*>(src);
  const int ks = cols / 16;
  for (int rb = 0; rb < rows / 32; ++rb)
    for (int s = 0; s < ks; ++s)
      for (int l = 0; l < 64; ++l) {
        const int i = l & 31;
        const int row = rb * 32 + ((i >> 2) & 1) * 16 + (i >> 3) * 4 + (i & 3);
        const uint16_t* from = in + (size_t)row * cols + s * 16 + 8 * (l >> 5);
        uint16_t* to = o + (((size_t)rb * ks + s) * 64 + l) * 8;
        for (int e = 0; e < 8; ++e) to[e] = from[e];
      }
}

bool adapter_bf16_supported(int d, int rank) { return rank == RANK && d % 256 == 0 && d >= 256 && d <= 768; }

// Preconditions (checked by the caller): adapter_bf16_supported(d, rank); which_tiles names
// the list of 128-row m-tiles and n_tiles128 its length; both matrices of every slot in
// the batch are in MFMA operand order; X, resid and x32 are 16-byte aligned [N, d] arrays, and so is Y where ln_g is set.  Y may
// be X (a unit's rows are in LDS before they are written, and no other unit has them), else they do not overlap.
void launch_adapter_bf16(const AdapterArgs& a, const Route& rt, hipStream_t s) {
  switch (a.d / 256) {
    case 1: return launch_nv<1>(a, rt, s);
    case 2: return launch_nv<2>(a, rt, s);
    default: return launch_nv<3>(a, rt, s);
  }
}

}  // namespace hmi

// The rule alone, for the tests: rows of a unit (8, 16, 32), or 0 for the general form.  units8, units16, units32: units of that
// many rows, summed over the batch's tenants.
extern "C" int32_t hmi_internal_adapter_unit(int32_t tenants, int32_t units8, int32_t units16, int32_t units32, int32_t with_norm, int32_t n_cu) {
  hmi::AdapterArgs a{};
  a.n_segs = tenants; a.stream_out = !with_norm;
  a.units[0] = units8; a.units[1] = units16; a.units[2] = units32;
  const int shift = hmi::unit_shift(a, n_cu);
  return shift ? 1 << shift : 0;
}
