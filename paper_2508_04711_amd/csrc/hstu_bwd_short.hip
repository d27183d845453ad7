// bf16 backward pass of batches of short sequences, dq, dk and dv in one kernel (see hstu_mfma.h for
// the common parts).
#include "hstu_mfma.h"

namespace hstu {

namespace {

// =============================================================================================
// A group of whole sequences of together at most 128 rows needs nothing from outside: Q, K, V and dO
// are read once, and dQ, dK and dV come from one computation of the scores.  (Two passes read the four
// inputs twice and are bound by that: on 8192 sequences of 16..64 rows dk/dv and dq move 3.7 GB.)
//
// Four waves, wave w owns keys 32w..32w+31 of the group (K and V rows in registers); Q and dO of the
// group lie in LDS.  Against each 32-row block of queries that its keys are seen by a wave works out
// S = Q K^T, dP = dO V^T, P and dS, and keeps the two as bf16 operands (8 registers each per block); then
// dV^T = dO^T P and dK^T = Q^T dS over all blocks, one accumulator after the other.  Last, dS and K take
// the place of Q and dO in LDS, and wave w owns queries 32w..32w+31: dQ^T = K^T dS^T, both operands
// through transposing reads (dS lies key by key).  With one accumulator alive at a time the kernel fits
// 256 registers at d = 128 (three spill, in the code for sequences of more than 128 rows) and 168 at d = 64, so that
// two and three workgroups share a CU, some computing while the others' loads and stores are under way.
//
// Bound by memory: the seven tensors once.  8192 sequences of 16..64 rows, H = 4, d = 128 (2.35 GB): 848 us
// for schedule, dk/dv and dq pass (4.3 GB) -> 537 us, 4.4 TB/s; 1024 of 120..128 rows 386 -> 220; at d = 64, 4096
// of 64..128 rows 530 -> 360; small ones, where launches count: 256 of 64..128 rows, H = 2, d = 64 36 -> 23.
// (With silu' of all blocks kept in fp32 instead, so that dV needs no P kept, the registers do not suffice.)
//
// There is no schedule: a workgroup takes the groups whose first row lies in its share of the rows, one
// head, and works them out from the offsets (64 sequences per look, one per lane).
// A sequence of more than 128 rows (the host sends batches whose max_len says there are none, but
// lengths above max_len are still computed) is left to workgroups of their own at the end of the grid: see
// long_sequences.
// =============================================================================================

constexpr int GT = 128;  // rows of a group
constexpr int NBLK = GT / 32;

// Per-lane LDS addresses of the operand reads.
template <int D>
struct ShortWave {
  RowAddr<D> ra;
  ColAddr<D> ca;
};

// `lane` as a value the compiler knows nothing about: what is computed from it is computed there, where
// it would otherwise be kept in registers (of which there are none to spare) from before the scores on.
__device__ __forceinline__ int opaque(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

// P and dS of the wave's keys against the four 32-query blocks from position pos0 on, rounded to bf16
// (zeros where nothing is seen).  Bit i of the result: block i is seen.  WP / WDS: which of the two is wanted.
template <int D, bool WP, bool WDS>
__device__ __forceinline__ int scores(const ShortWave<D>& w, const char* qt, const char* gt, const bf16x8 (&kreg)[D / 16],
                                      const bf16x8 (&vreg)[D / 16], bf16x8 (&pk)[NBLK][2], bf16x8 (&ds)[NBLK][2],
                                      const Window& win, int pos0, int hh, float c1, float alpha) {
  int seen = 0;
#pragma unroll
  for (int i = 0; i < NBLK; ++i) {
    const int b = pos0 + 32 * i;
    if (b > win.hi_max || b + 31 < win.lo_min) {
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int e = 0; e < 8; ++e) pk[i][y][e] = ds[i][y][e] = (__bf16)0.f;
      continue;
    }
    seen |= 1 << i;
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) s = mfma(w.ra.read(qt, i, ks), kreg[ks], s);
    if constexpr (WDS) {
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) dp = mfma(w.ra.read(gt, i, ks), vreg[ks], dp);
    }
    const bool mask = win.masks(b);
    const VisWindow vis = win.vis(b, hh);
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      // stage by stage over eight elements, so that no instruction waits for its predecessor's result
      float t[8], g[8], p[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = s[8 * y + j] * c1;
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = __builtin_amdgcn_exp2f(t[j]);
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = 1.0f + t[j];
#pragma unroll
      for (int j = 0; j < 8; ++j) g[j] = __builtin_amdgcn_rcpf(t[j]);
#pragma unroll
      for (int j = 0; j < 8; ++j) p[j] = s[8 * y + j] * g[j];
      if constexpr (WDS) {
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = __builtin_fmaf(-p[j], g[j], p[j]);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = __builtin_fmaf(alpha, t[j], g[j]);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = dp[8 * y + j] * t[j];
      }
      if (mask) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool v = vis(8 * y + j);
          p[j] = v ? p[j] : 0.f;
          t[j] = v ? t[j] : 0.f;
        }
      }
      if constexpr (WP) pk[i][y] = pack8(p);
      if constexpr (WDS) ds[i][y] = pack8(t);
    }
  }
  return seen;
}

// acc += rows^T b over the blocks seen: dV^T += dO^T P, dK^T += Q^T dS.
template <int D>
__device__ __forceinline__ void contract(const ShortWave<D>& w, const char* tile, const bf16x8 (&b)[NBLK][2],
                                         f32x16 (&acc)[D / 32], int seen) {
#pragma unroll
  for (int i = 0; i < NBLK; ++i) {
    if (!(seen & (1 << i))) continue;
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
      acc[c] = mfma(w.ca.read(tile, 2 * i, c), b[i][0], acc[c]);
      acc[c] = mfma(w.ca.read(tile, 2 * i + 1, c), b[i][1], acc[c]);
    }
  }
}

// dS and K rows of the wave's 32 keys into LDS: dS as [key][128 queries], K as [key][D].
template <int D>
__device__ __forceinline__ void hand_over(char* dst, char* kt, const bf16x8 (&kreg)[D / 16], const bf16x8 (&ds)[NBLK][2],
                                          int lane, int wave) {
  lane = opaque(lane);
  const int hh = lane >> 5, row = wave * 32 + (lane & 31);
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const bf16x8 x = ds[i][q4 >> 1];
      const bf16x4 y = (q4 & 1) ? __builtin_shufflevector(x, x, 4, 5, 6, 7) : __builtin_shufflevector(x, x, 0, 1, 2, 3);
      *HSTU_LDS(bf16x4, dst + lds_off<GT>(row, 4 * i + q4) + 8 * hh) = y;
    }
#pragma unroll
  for (int s = 0; s < D / 16; ++s) *HSTU_LDS(bf16x8, kt + lds_off<D>(row, 2 * s + hh)) = kreg[s];
}

// dQ^T += K^T dS^T over the key blocks that some query of the wave's block sees; pos0: position of
// the first key.
template <int D>
__device__ __forceinline__ void query_grads(const ShortWave<D>& w, const char* dst, const char* kt, f32x16 (&acc)[D / 32],
                                            const Window& win, int pos0, int lane, int wave) {
  // the lane's operand of dS^T: rows 0..7 and 8..15 of 16 keys (see ColAddr)
  lane = opaque(lane);
  const int i16 = lane & 15, g = lane >> 4, row = ((g >> 1) << 2) + (i16 >> 2);
  const int col = wave * 32 + ((g & 1) << 4) + ((i16 & 3) << 2);
  const int a0 = lds_off<GT>(row, col >> 3) + ((col & 7) << 1), a1 = lds_off<GT>(row + 8, col >> 3) + ((col & 7) << 1);
#pragma unroll
  for (int i = 0; i < NBLK; ++i) {
    const int b = pos0 + 32 * i;
    if (b > win.hi_max || b + 31 < win.lo_min) continue;
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const char* base = dst + (2 * i + y) * 16 * GT * 2;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(HSTU_LDS(s16x4, base + a0));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(HSTU_LDS(s16x4, base + a1));
      typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      const bf16x8 bq = __builtin_bit_cast(bf16x8, both);
#pragma unroll
      for (int c = 0; c < D / 32; ++c) acc[c] = mfma(w.ca.read(kt, 2 * i + y, c), bq, acc[c]);
    }
  }
}

template <int D>
constexpr int short_lds() { return 2 * GT * D * 2 > GT * GT * 2 + GT * D * 2 ? 2 * GT * D * 2 : GT * GT * 2 + GT * D * 2; }

// What a workgroup's loads and stores of one head need.
template <int D>
struct ShortIo {
  const AttnArgs& a;
  char *qt, *gt, *dst, *kt;  // LDS: Q and dO, whose place dS and K take
  int64_t sr;                // row stride in elements
  int h, lane, wave, orow, hh;
  __device__ __forceinline__ void load_keys(bf16x8 (&kreg)[D / 16], bf16x8 (&vreg)[D / 16], int row, int rows) const {
    load_owner<D>(kreg, (const __bf16*)a.k + (int64_t)row * sr + h * D, sr, orow, rows, hh);
    load_owner<D>(vreg, (const __bf16*)a.v + (int64_t)row * sr + h * D, sr, orow, rows, hh);
  }
  __device__ __forceinline__ void load_queries(int row, int rows) const {  // (`rows` may be more than the 128 that are copied)
#pragma unroll
    for (int x = 0; x < GT / ST; ++x) {
      const int64_t at = (int64_t)(row + x * ST) * sr + h * D;
      tile_copy_async<D, 4>(qt + x * ST * D * 2, (const __bf16*)a.q + at, sr, rows - x * ST, wave, lane);
      tile_copy_async<D, 4>(gt + x * ST * D * 2, (const __bf16*)a.d_o + at, sr, rows - x * ST, wave, lane);
    }
  }
  __device__ __forceinline__ void landed() const {
    tile_copy_wait<0>();
    tile_barrier();
  }
  __device__ __forceinline__ void exchange(const bf16x8 (&kreg)[D / 16], const bf16x8 (&ds)[NBLK][2]) const {
    tile_barrier();
    hand_over<D>(dst, kt, kreg, ds, lane, wave);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    tile_barrier();
  }
  __device__ __forceinline__ void store(void* out, int row, int rows, const f32x16 (&acc)[D / 32]) const {
    if (orow < rows) store_owner_major<D>(out, ((int64_t)row + orow) * sr + h * D, acc, a.alpha * a.inv_n, hh, 0, a.out_f32);
  }
};
template <int D>
__device__ __forceinline__ void clear(f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
}

// The sequences of more than 128 rows, by `helpers` workgroups per head: every tile of 128 rows is three items, dV, dK and
// dQ, each a walk over the tiles its rows see, dealt out in turn, each sequence's longest first.  The first thing
// such a workgroup does is look whether there is any such sequence; if not, that look is all it costs, and it
// happens in the tail of the others.  (With the long sequences' tiles computed by the workgroups in whose shares
// of the rows they lie, three walks in a row, those were the last by far: 400 sequences of 16..100 rows and one of
// 4096, max_len = 128, H = 4, d = 128, 629 us against 320 of the two passes; now 256.)
template <int D>
__device__ __forceinline__ void long_sequences(const AttnArgs& a, char* smem, int h, int me, int helpers) {
  const int T = a.self.total_rows, B = a.self.batch, tid = threadIdx.x;
  const int32_t* off = a.self.off;
  int any = 0;
#pragma unroll 8
  for (int j = tid; j < B; j += 256) {
    int s, e;
    seq_range(off, j, T, s, e);
    any |= e - s > GT;
  }
  if (!__syncthreads_or(any)) return;

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float c1 = -a.alpha * 1.4426950408889634f;
  bf16x8 kreg[D / 16], vreg[D / 16], pk[NBLK][2], ds[NBLK][2];
  f32x16 acc[D / 32];
  int turn = me;  // items until this workgroup's next one
  for (int first = 0; first < B; first += 64) {
    int s = 0, e = 0;
    if (first + (tid & 63) < B) seq_range(off, first + (tid & 63), T, s, e);
    for (unsigned long long longs = __ballot(e - s > GT); longs; longs &= longs - 1) {
      const int l = __builtin_ctzll(longs);
      const int b0 = __builtin_amdgcn_readlane(s, l), len = __builtin_amdgcn_readlane(e, l) - b0;
      const int nt = (len >> 7) + ((len & (GT - 1)) != 0);
      for (; turn < 3 * nt; turn += helpers) {
        const int part = turn % 3, m = turn / 3, t = part < 2 ? m : nt - 1 - m;
        const int row = b0 + t * GT, rows = len - t * GT < GT ? len - t * GT : GT;
        const int2 whole = make_int2(0, len);
        // (worked out again for every item, as for every group below)
        const int lane = opaque(tid & 63), n = lane & 31, hh = lane >> 5, orow = wave * 32 + n;
        const ShortIo<D> io = {a, smem, smem + GT * D * 2, smem, smem + GT * GT * 2, (int64_t)a.num_heads * D, h, lane, wave,
                               orow, hh};
        ShortWave<D> w;
        w.ra.init(n, hh);
        w.ca.init(lane);
        clear<D>(acc);
        auto key_side = [&](auto tag) {
          constexpr bool DV = decltype(tag)::value;
          const Window wk = make_window(whole, t * GT + orow, orow < rows, 1, a.causal);
          io.load_keys(kreg, vreg, row, rows);
          for (int x = a.causal ? t : 0; x < nt; ++x) {
            io.load_queries(b0 + x * GT, len - x * GT);
            io.landed();
            const int seen = scores<D, DV, !DV>(w, io.qt, io.gt, kreg, vreg, pk, ds, wk, x * GT, hh, c1, a.alpha);
            contract<D>(w, DV ? io.gt : io.qt, DV ? pk : ds, acc, seen);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            tile_barrier();
          }
          io.store(DV ? a.dv : a.dk, row, rows, acc);
        };
        if (part == 0) { key_side(std::true_type{}); continue; }
        if (part == 1) { key_side(std::false_type{}); continue; }
        const Window wq = make_window(whole, t * GT + orow, orow < rows, 0, a.causal);
        for (int x = 0; x < (a.causal ? t + 1 : nt); ++x) {
          const int krow = x * GT, krows = len - krow < GT ? len - krow : GT;
          io.load_keys(kreg, vreg, b0 + krow, krows);
          io.load_queries(row, rows);
          const Window wx = make_window(whole, krow + orow, orow < krows, 1, a.causal);
          io.landed();
          scores<D, false, true>(w, io.qt, io.gt, kreg, vreg, pk, ds, wx, t * GT, hh, c1, a.alpha);
          io.exchange(kreg, ds);
          query_grads<D>(w, io.dst, io.kt, acc, wq, krow, lane, wave);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          tile_barrier();
        }
        io.store(a.dq, row, rows, acc);
      }
      turn -= 3 * nt;
    }
  }
}

// a.max_items: shares of the rows per head.  Workgroups beyond are long_sequences' helpers.
template <int D>
__global__ void __launch_bounds__(256, D == 64 ? 3 : 2) hstu_bwd_short_bf16(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[short_lds<D>()];

  const int H = a.num_heads, h = blockIdx.x % H, T = a.self.total_rows, B = a.self.batch;
  const int shares = a.max_items, share = blockIdx.x / H;
  if (share >= shares) {
    long_sequences<D>(a, smem, h, share - shares, (int)(gridDim.x / H) - shares);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float c1 = -a.alpha * 1.4426950408889634f;
  const int32_t* off = a.self.off;

  // The workgroup's share of the rows, and the first sequence that begins in it.
  const int r0 = (int)((int64_t)T * share / shares), r1 = (int)((int64_t)T * (share + 1) / shares);
  int i = 0;
  {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (off[mid] <= r0) lo = mid; else hi = mid;
    }
    int s, e;
    seq_range(off, lo, T, s, e);
    i = s < r0 ? lo + 1 : lo;
  }
  i = __builtin_amdgcn_readfirstlane(i);

  // Sequences i .. i + 63 as they lie in memory, one per lane, requested a unit ahead.
  int ob = 0, oe = 0;
  auto request = [&](int first) {
    const int j = first + (threadIdx.x & 63), x = j < B ? j : B, y = x + 1 < B ? x + 1 : B;
    ob = off[x];
    oe = off[y];
  };
  request(i);

  while (i < B) {
    // (worked out again for every unit: kept across the loop, the addresses would cost more registers
    // than there are)
    const int lane = opaque(threadIdx.x & 63);
    const int n = lane & 31, hh = lane >> 5, orow = wave * 32 + n;
    const ShortIo<D> io = {a, smem, smem + GT * D * 2, smem, smem + GT * GT * 2, (int64_t)H * D, h, lane, wave, orow, hh};
    ShortWave<D> w;
    w.ra.init(n, hh);
    w.ca.init(lane);
    bf16x8 kreg[D / 16], vreg[D / 16], pk[NBLK][2], ds[NBLK][2];
    f32x16 acc[D / 32];

    const int b = clampi(ob, 0, T), e = clampi(oe, b, T);
    const int b0 = __builtin_amdgcn_readfirstlane(b);
    if (b0 >= r1) break;  // all that follow begin in other shares or have no rows
    const int before = __shfl_up(e, 1, 64);
    // the sequences that follow one another from the first on and end within 128 rows
    const bool in = i + lane < B && e - b0 <= GT && b < r1 && (lane == 0 || b == before);
    const unsigned long long out = ~__ballot(in);
    const int count = out ? __builtin_ctzll(out) : 64;
    if (count == 0) {  // one of more than 128 rows
      request(++i);
      continue;
    }
    const int rows = __builtin_amdgcn_readlane(e, count - 1) - b0;
    i += count;
    request(i);
    if (rows <= 0) continue;
    io.load_keys(kreg, vreg, b0, rows);
    io.load_queries(b0, rows);
    // the sequence of the lane's row
    int l = 0;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) {
      const int m = l + step, bm = __shfl(b, m & 63, 64);
      if (m < count && bm - b0 <= orow) l = m;
    }
    const int2 sq = make_int2(__shfl(b, l, 64) - b0, __shfl(e, l, 64) - b0);
    const Window wk = make_window(sq, orow, orow < rows, 1, a.causal);
    const Window wq = make_window(sq, orow, orow < rows, 0, a.causal);
    io.landed();
    const int seen = scores<D, true, true>(w, io.qt, io.gt, kreg, vreg, pk, ds, wk, 0, hh, c1, a.alpha);
    clear<D>(acc);
    contract<D>(w, io.gt, pk, acc, seen);
    io.store(a.dv, b0, rows, acc);
    clear<D>(acc);
    contract<D>(w, io.qt, ds, acc, seen);
    io.store(a.dk, b0, rows, acc);
    io.exchange(kreg, ds);
    clear<D>(acc);
    query_grads<D>(w, io.dst, io.kt, acc, wq, 0, lane, wave);
    io.store(a.dq, b0, rows, acc);
    tile_barrier();
  }
}

}  // namespace

bool bwd_short_supported(int d_qk, int d_v) { return d_qk == d_v && (d_qk == 64 || d_qk == 128); }

hipError_t launch_bwd_short_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  if (!bwd_short_supported(d_qk, d_v) || !a.self.off || a.self.batch < 1 || a.ts_rec || a.accumulate) return hipErrorInvalidValue;
  // As many workgroups as are resident at once, but no more shares than groups; then the helpers of sequences
  // of more than 128 rows, on the slots that are left over or, if those are few, on all of them in turn.
  const int64_t resident = d_qk == 128 ? 512 : 768, groups = ((int64_t)a.self.total_rows + GT - 1) / GT;
  const int64_t slots = resident / a.num_heads < 1 ? 1 : resident / a.num_heads;
  const int64_t shares = slots > groups ? groups : slots;
  int64_t helpers = slots - shares > slots / 4 ? slots - shares : slots;
  if (helpers > groups) helpers = groups;
  AttnArgs args = a;
  args.max_items = (int32_t)shares;
  const dim3 grid((unsigned)((shares + helpers) * a.num_heads)), block(256);
  if (d_qk == 128) hipLaunchKernelGGL((hstu_bwd_short_bf16<128>), grid, block, 0, stream, args);
  else hipLaunchKernelGGL((hstu_bwd_short_bf16<64>), grid, block, 0, stream, args);
  return hipGetLastError();
}

}  // namespace hstu
