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
// 256 registers, so that two workgroups share a CU, one computing while the other's loads and stores are
// under way.
//
// Bound by memory: the seven tensors once.  8192 sequences of 16..64 rows, H = 4, d = 128 (2.35 GB): 848 us
// for schedule, dk/dv and dq pass (4.3 GB) -> 537 us, 4.4 TB/s; 1024 of 120..128 rows 386 -> 220; at d = 64, 4096
// of 64..128 rows 530 -> 360; small ones, where launches count: 256 of 64..128 rows, H = 2, d = 64 36 -> 23.
// (With silu' of all blocks kept in fp32 instead, so that dV needs no P kept, the registers do not suffice.)
//
// There is no schedule: a workgroup takes the units whose first row lies in its share of the rows, one
// head, and works the groups out from the offsets (64 sequences per look, one per lane).
// A sequence of more than 128 rows (the host sends batches whose max_len says there are none, but
// lengths above max_len are still computed) is cut into units of 128 rows which go over the other
// tiles of the sequence three times, once per accumulator.
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

template <int D>
__global__ void __launch_bounds__(256, 2) hstu_bwd_short_bf16(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[short_lds<D>()];
  char* const qt = smem;               // Q, then dS
  char* const gt = smem + GT * D * 2;  // dO
  char* const dst = smem;
  char* const kt = smem + GT * GT * 2;  // K

  const int H = a.num_heads, h = blockIdx.x % H, T = a.self.total_rows, B = a.self.batch;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t sr = (int64_t)H * D;
  const float c1 = -a.alpha * 1.4426950408889634f, scale = a.alpha * a.inv_n;
  const int32_t* off = a.self.off;

  // The workgroup's share of the rows, and the first unit that begins in it.
  const int shares = (int)(gridDim.x / H), share = blockIdx.x / H;
  const int r0 = (int)((int64_t)T * share / shares), r1 = (int)((int64_t)T * (share + 1) / shares);
  int i = 0, t = 0;  // first sequence of the unit, tile of a long one
  {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (off[mid] <= r0) lo = mid; else hi = mid;
    }
    int s, e;
    seq_range(off, lo, T, s, e);
    i = lo;
    if (s < r0) {
      t = e - s > GT ? (r0 - s + GT - 1) / GT : 0;
      if (t == 0 || t >= (e - s + GT - 1) / GT) { ++i; t = 0; }
    }
  }
  i = __builtin_amdgcn_readfirstlane(i);
  t = __builtin_amdgcn_readfirstlane(t);

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
    ShortWave<D> w;
    w.ra.init(n, hh);
    w.ca.init(lane);

    bf16x8 kreg[D / 16], vreg[D / 16], pk[NBLK][2], ds[NBLK][2];
    f32x16 acc[D / 32];
    auto clear_acc = [&] {
#pragma unroll
      for (int c = 0; c < D / 32; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
    };
    auto load_keys = [&](int row, int rows) {
      load_owner<D>(kreg, (const __bf16*)a.k + (int64_t)row * sr + h * D, sr, orow, rows, hh);
      load_owner<D>(vreg, (const __bf16*)a.v + (int64_t)row * sr + h * D, sr, orow, rows, hh);
    };
    auto load_queries = [&](int row, int rows) {  // (`rows` may be more than the 128 that are copied)
#pragma unroll
      for (int x = 0; x < GT / ST; ++x) {
        const int64_t at = (int64_t)(row + x * ST) * sr + h * D;
        tile_copy_async<D, 4>(qt + x * ST * D * 2, (const __bf16*)a.q + at, sr, rows - x * ST, wave, lane);
        tile_copy_async<D, 4>(gt + x * ST * D * 2, (const __bf16*)a.d_o + at, sr, rows - x * ST, wave, lane);
      }
    };
    auto landed = [&] {
      tile_copy_wait<0>();
      tile_barrier();
    };
    auto store = [&](void* out, int row, int rows) {
      if (orow < rows) store_owner_major<D>(out, ((int64_t)row + orow) * sr + h * D, acc, scale, hh, 0, a.out_f32);
    };
    auto exchange = [&] {  // dS and K take the place of Q and dO
      tile_barrier();
      hand_over<D>(dst, kt, kreg, ds, lane, wave);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      tile_barrier();
    };

    const int b = clampi(ob, 0, T), e = clampi(oe, b, T);
    const int b0 = __builtin_amdgcn_readfirstlane(b), e0 = __builtin_amdgcn_readfirstlane(e);
    if (b0 >= r1) break;  // all that follow begin in other shares or have no rows
    const int before = __shfl_up(e, 1, 64);
    // the sequences that follow one another from the first on and end within 128 rows
    const bool in = i + lane < B && e - b0 <= GT && b < r1 && (lane == 0 || b == before);
    const unsigned long long out = ~__ballot(in);
    const int count = out ? __builtin_ctzll(out) : 64;
    if (count > 0) {
      const int rows = __builtin_amdgcn_readlane(e, count - 1) - b0;
      i += count;
      request(i);
      if (rows <= 0) continue;
      load_keys(b0, rows);
      load_queries(b0, rows);
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
      landed();
      const int seen = scores<D, true, true>(w, qt, gt, kreg, vreg, pk, ds, wk, 0, hh, c1, a.alpha);
      clear_acc();
      contract<D>(w, gt, pk, acc, seen);
      store(a.dv, b0, rows);
      clear_acc();
      contract<D>(w, qt, ds, acc, seen);
      store(a.dk, b0, rows);
      exchange();
      clear_acc();
      query_grads<D>(w, dst, kt, acc, wq, 0, lane, wave);
      store(a.dq, b0, rows);
      tile_barrier();
      continue;
    }
    // a tile of a long sequence, or the end of the share
    const int len = e0 - b0, nt = (len + GT - 1) / GT;
    if (t >= nt) {
      t = 0;
      request(++i);
      continue;
    }
    const int row = b0 + t * GT;
    if (row >= r1) break;
    const int rows = len - t * GT < GT ? len - t * GT : GT;
    const int2 whole = make_int2(0, len);
    const int qfirst = a.causal ? t : 0, klast = a.causal ? t : nt - 1;
    const Window wk = make_window(whole, t * GT + orow, orow < rows, 1, a.causal);
    const Window wq = make_window(whole, t * GT + orow, orow < rows, 0, a.causal);
    auto key_side = [&](auto tag) {
      constexpr bool DV = decltype(tag)::value;
      clear_acc();
      for (int x = qfirst; x < nt; ++x) {
        load_keys(row, rows);
        load_queries(b0 + x * GT, len - x * GT);
        landed();
        const int seen = scores<D, DV, !DV>(w, qt, gt, kreg, vreg, pk, ds, wk, x * GT, hh, c1, a.alpha);
        contract<D>(w, DV ? gt : qt, DV ? pk : ds, acc, seen);
        tile_barrier();
      }
      store(DV ? a.dv : a.dk, row, rows);
    };
    key_side(std::true_type{});
    key_side(std::false_type{});
    clear_acc();
    for (int x = 0; x <= klast; ++x) {
      const int krow = x * GT, krows = len - krow < GT ? len - krow : GT;
      load_keys(b0 + krow, krows);
      load_queries(row, rows);
      const Window wx = make_window(whole, krow + orow, orow < krows, 1, a.causal);
      landed();
      scores<D, false, true>(w, qt, gt, kreg, vreg, pk, ds, wx, t * GT, hh, c1, a.alpha);
      exchange();
      query_grads<D>(w, dst, kt, acc, wq, krow, lane, wave);
      tile_barrier();
    }
    store(a.dq, row, rows);
    ++t;
  }
}

}  // namespace

bool bwd_short_supported(int d_qk, int d_v) { return d_qk == d_v && (d_qk == 64 || d_qk == 128); }

hipError_t launch_bwd_short_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  if (!bwd_short_supported(d_qk, d_v) || !a.self.off || a.self.batch < 1 || a.ts_rec || a.accumulate) return hipErrorInvalidValue;
  // as many workgroups as are resident at once, but no more shares than groups
  const int64_t resident = d_qk == 128 ? 512 : 768, groups = ((int64_t)a.self.total_rows + GT - 1) / GT;
  int64_t shares = resident / a.num_heads;
  shares = shares < 1 ? 1 : (shares > groups ? groups : shares);
  const dim3 grid((unsigned)(shares * a.num_heads)), block(256);
  if (d_qk == 128) hipLaunchKernelGGL((hstu_bwd_short_bf16<128>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((hstu_bwd_short_bf16<64>), grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace hstu
