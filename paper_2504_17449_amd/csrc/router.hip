// Tenant-segmented router: orders a batch's requests by tenant id (stable), finds the segments of equal tenant and
// their offsets, and emits the m-tile work lists and the sorted-row -> original-row map the grouped GEMMs consume.
//
// This is the GPU form of "stack the parameters of the adapters per request" in the paper's parallel adapter
// inference (Sec. 6.3): instead of copying a tenant's parameters next to every request, requests are grouped so that
// one segment shares one weight image.
//
// It is latency and nothing else: a few thousand numbers, but every step waits for the one before, and a barrier of
// sixteen wavefronts costs several hundred clocks.  So
//   * a workgroup has as many wavefronts as the batch needs (one up to 64 requests, four up to 256, eight up to 512,
//     sixteen beyond, with one or two requests per lane);
//   * the sort is an LSD radix sort with digits of at most 6 bits and two barriers a pass: a wavefront ranks its elements
//     among equal digits by ballots and writes its own counts; every wavefront then adds up all counts itself, one digit
//     per lane, and scans them by shuffles;
//   * a prefix sum over the workgroup is a shuffle scan, one barrier, and the same scan over the wavefronts' totals;
//   * large batches get several workgroups, each of which does all of this (from its own reads of the inputs) and then
//     writes its share of the row map; only the first writes anything else.
// Measured per launch, before (sixteen wavefronts, five barriers a pass, one workgroup) and now: one request of 40 rows
// 10.5 us -> 5.6, 256 decode rows 14.2 -> 7.1, 37 requests of 2 664 rows 11.4 -> 7, 512 of 65 536 rows 16.8 -> 9.0, 1 024 of
// 65 536 rows over 10 000 ids 24.4 -> 13.1; 2 us of each are the reads of the inputs over the host link.
#include "hmi_kernels.h"

#include "wave.h"

namespace hmi {
namespace {

constexpr int kMaxWorkgroups = 8;

// Exclusive prefix sums of two values per element over the workgroup's elements in order (round, wavefront, lane), and
// their totals.  One barrier; `tots` must not be in use by an earlier call (each call gets its own).
template <int W, int C>
__device__ __forceinline__ void block_exscan2(const int (&a)[C], const int (&b)[C], int (*tots)[2], int (&ea)[C], int (&eb)[C],
                                              int& total_a, int& total_b) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int ia[C], ib[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    ia[c] = wave_incl_scan(a[c]);
    ib[c] = wave_incl_scan(b[c]);
    if (lane == 63) { tots[c * W + w][0] = ia[c]; tots[c * W + w][1] = ib[c]; }
  }
  __syncthreads();
  const int ta = lane < W * C ? tots[lane][0] : 0, tb = lane < W * C ? tots[lane][1] : 0;
  const int sa = wave_incl_scan(ta), sb = wave_incl_scan(tb);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    ea[c] = __builtin_amdgcn_readlane(sa - ta, c * W + w) + ia[c] - a[c];
    eb[c] = __builtin_amdgcn_readlane(sb - tb, c * W + w) + ib[c] - b[c];
  }
  total_a = __builtin_amdgcn_readlane(sa, 63);
  total_b = __builtin_amdgcn_readlane(sb, 63);
}

// W wavefronts, C requests per lane (R <= 64 W C)
template <int W, int C>
__global__ __launch_bounds__(64 * W) void router_kernel(Route rt, int R, int key_bits) {
  constexpr int NT = 64 * W, E = NT * C;
  __shared__ int key_s[E];              // sorted tenant ids
  __shared__ int perm_s[E];             // sorted position -> request
  __shared__ int slot_s[E];             // request -> HBM slot
  __shared__ int tok_s[E + 1];          // request -> first original row
  __shared__ int stok_s[E + 1];         // sorted position -> first sorted row
  __shared__ int segtok_s[E + 1];       // segment -> first sorted row
  __shared__ int cnt[W * C][64];        // per round and wavefront: elements of each digit
  __shared__ int tots[3][W * C][2];
  int* const tb0 = key_s;               // segment -> its first tile in list 0 / list 1 (written when the keys and slots are done with)
  int* const tb1 = slot_s;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool main_wg = blockIdx.x == 0;

  // ---- inputs: they may live in host memory (a round trip over the host link per dependent read), so each is read
  //      exactly once, here, all reads in flight together.  tok_off = exclusive scan of seq_lens in arrival order.
  int k_[C], v_[C], len[C], slot[C], zero[C], kv_slot[C], kv_pos[C];
  const bool kv = main_wg && rt.kv_slot_in;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = c * NT + tid;
    const bool in = i < R;
    len[c] = in ? rt.seq_lens[i] : 0;
    k_[c] = in ? rt.tenant_ids[i] : 0;
    slot[c] = in ? rt.req_slot[i] : 0;
    kv_slot[c] = kv && in ? rt.kv_slot_in[i] : 0;
    kv_pos[c] = kv && in ? rt.kv_pos_in[i] : 0;
    v_[c] = i;
    zero[c] = 0;
  }
  int tok[C], unused[C], N, unused_total;
  block_exscan2<W, C>(len, zero, tots[0], tok, unused, N, unused_total);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = c * NT + tid;
    if (i < R) {
      tok_s[i] = tok[c]; slot_s[i] = slot[c];
      if (main_wg) { rt.tok_off[i] = tok[c]; rt.req_tenant[i] = k_[c]; }
      if (kv) { rt.kv_slot[i] = kv_slot[c]; rt.kv_pos[i] = kv_pos[c]; }
    }
  }
  if (tid == 0) { tok_s[R] = N; if (main_wg) rt.tok_off[R] = N; }
  if (main_wg && rt.dense_seg_tok_off) {
    const int Gd = (N + kDenseSegRows - 1) / kDenseSegRows;
    for (int g = tid; g <= Gd; g += NT) rt.dense_seg_tok_off[g] = min(g * kDenseSegRows, N);
    if (tid == 0) rt.dense_n_segments[0] = Gd;
  }

  // ---- stable LSD radix sort of (tenant id, request) by tenant id, all passes equally wide (64 tenants: one pass,
  //      1 000: two, 10 000: three)
  const int passes = (key_bits + 5) / 6;
  const int db = (key_bits + passes - 1) / passes;                       // bits per digit
  for (int shift = 0; shift < passes * db; shift += db) {
    int digit[C], rank[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const bool valid = c * NT + tid < R;
      digit[c] = (k_[c] >> shift) & ((1 << db) - 1);
      unsigned long long mask = __ballot(valid);
#pragma unroll
      for (int b = 0; b < 6; ++b) {
        const bool bit = (digit[c] >> b) & 1;
        const unsigned long long bal = __ballot(valid && bit);
        if (b < db) mask &= bit ? bal : ~bal;
      }
      rank[c] = __popcll(mask & ((1ull << lane) - 1ull));
      cnt[c * W + w][lane] = 0;
      if (valid && rank[c] == 0) cnt[c * W + w][digit[c]] = __popcll(mask);
    }
    __syncthreads();
    // lane = digit: where the elements of this digit begin for this wavefront
    int run = 0, base[C];
#pragma unroll
    for (int j = 0; j < W * C; ++j) {
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (j == c * W + w) base[c] = run;
      run += cnt[j][lane];
    }
    const int before = wave_incl_scan(run) - run;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int pos = __shfl(before + base[c], digit[c], 64) + rank[c];
      if (c * NT + tid < R) { key_s[pos] = k_[c]; perm_s[pos] = v_[c]; }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int i = c * NT + tid;
      if (i < R) { k_[c] = key_s[i]; v_[c] = perm_s[i]; }
    }
  }

  // ---- segments (maximal runs of one tenant) and sorted-token offsets
  int head[C], slen[C], g_[C], st[C], G, unused_n;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int p = c * NT + tid;
    const bool in = p < R;
    head[c] = in && (p == 0 || k_[c] != key_s[p - 1]);
    slen[c] = in ? tok_s[v_[c] + 1] - tok_s[v_[c]] : 0;
  }
  block_exscan2<W, C>(head, slen, tots[1], g_, st, G, unused_n);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int p = c * NT + tid;
    if (p < R) {
      stok_s[p] = st[c];
      if (main_wg) rt.perm[p] = v_[c];
      if (head[c]) {
        segtok_s[g_[c]] = st[c];
        if (main_wg) {
          rt.seg_tenant[g_[c]] = k_[c];
          rt.seg_slot[g_[c]] = slot_s[v_[c]];
          rt.seg_req_off[g_[c]] = p;
          rt.seg_tok_off[g_[c]] = st[c];
        }
      }
    }
  }
  if (tid == 0) {
    segtok_s[G] = N;
    stok_s[R] = N;
    if (main_wg) { rt.seg_req_off[G] = R; rt.seg_tok_off[G] = N; rt.n_segments[0] = G; }
  }
  __syncthreads();

  // ---- m-tile work lists for both tile heights: tiles never straddle a segment
  if (main_wg) {
    const int tm0 = rt.tile_m[0], tm1 = rt.tile_m[1];
    int nt0[C], nt1[C], b0[C], b1[C], n0, n1;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int g = c * NT + tid;
      const int rows = g < G ? segtok_s[g + 1] - segtok_s[g] : 0;
      nt0[c] = tm0 > 0 ? (rows + tm0 - 1) / tm0 : 0;
      nt1[c] = tm1 > 0 ? (rows + tm1 - 1) / tm1 : 0;
    }
    block_exscan2<W, C>(nt0, nt1, tots[2], b0, b1, n0, n1);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int g = c * NT + tid;
      if (g < G) { tb0[g] = b0[c]; tb1[g] = b1[c]; }
    }
    if (tid == 0) {
      if (tm0 > 0) rt.n_tiles[0][0] = n0;
      if (tm1 > 0) rt.n_tiles[1][0] = n1;
    }
    __syncthreads();
    // one thread per tile, whatever the sizes of the segments (a single tenant's batch is one segment of hundreds of
    // tiles): the tile's segment is the last one whose first tile is not behind it
    for (int k = 0; k < 2; ++k) {
      const int* tb = k == 0 ? tb0 : tb1;
      const int tm = k == 0 ? tm0 : tm1, n = k == 0 ? n0 : n1;
      for (int t = tid; t < n; t += NT) {
        int lo = 0, hi = G - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (tb[mid] <= t) lo = mid; else hi = mid - 1;
        }
        rt.tile_seg[k][t] = lo;
        rt.tile_row0[k][t] = segtok_s[lo] + (t - tb[lo]) * tm;
      }
    }
  }

  // ---- sorted row -> original row.  Wavefront x of all workgroups takes the sorted positions x, x + (their number), ...,
  //      64 at a time, a lane each.  A lane writes the rows of a short request itself; over the long ones the wavefront
  //      walks together, with the numbers broadcast from their lane's registers.
  constexpr int kShort = 8;
  const int waves = W * gridDim.x, x = blockIdx.x * W + w;
  for (int base = 0; base < R; base += waves * 64) {
    const int myp = base + lane * waves + x;
    int src0 = 0, dst0 = 0, n_rows = 0;
    if (myp < R) { src0 = tok_s[perm_s[myp]]; dst0 = stok_s[myp]; n_rows = stok_s[myp + 1] - dst0; }
    if (n_rows <= kShort)
      for (int i = 0; i < n_rows; ++i) rt.row_src[dst0 + i] = src0 + i;
    for (unsigned long long todo = __ballot(n_rows > kShort); todo; todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);
      const int s0 = __builtin_amdgcn_readlane(src0, l), d0 = __builtin_amdgcn_readlane(dst0, l);
      const int n = __builtin_amdgcn_readlane(n_rows, l);
      for (int i = lane; i < n; i += 64) rt.row_src[d0 + i] = s0 + i;
    }
  }
}

template <int W, int C>
void launch_w(const Route& rt, int R, int N, hipStream_t s) {
  // one workgroup per 512 rows of each wavefront: below that the stores are no longer than the rest of its work
  const int wgs = N / (W * 512) < 1 ? 1 : N / (W * 512) > kMaxWorkgroups ? kMaxWorkgroups : N / (W * 512);
  hipLaunchKernelGGL((router_kernel<W, C>), dim3(wgs), dim3(64 * W), 0, s, rt, R, rt.key_bits);
}

}  // namespace

void launch_router(const Route& rt, int R, int N, hipStream_t s) {
  if (R <= 64) return launch_w<1, 1>(rt, R, N, s);
  if (R <= 256) return launch_w<4, 1>(rt, R, N, s);
  if (R <= 512) return launch_w<8, 1>(rt, R, N, s);
  if (R <= 1024) return launch_w<16, 1>(rt, R, N, s);
  launch_w<16, 2>(rt, R, N, s);
}

}  // namespace hmi
