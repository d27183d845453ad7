// bf16 dk/dv kernel for the large head dimensions, two waves per SIMD (see hstu_mfma.h for the
// common parts and hstu_dkdv.hip for the one-wave-per-SIMD kernel it replaces on long sequences).
#include "hstu_mfma.h"

namespace hstu {

namespace {

// =============================================================================================
// The dk/dv pass of section 2.1's attention (gradient derived: with x = alpha*s, sg = sigmoid(x),
// p = x*sg/N, dp = <dO_i, V_j>/N, ds = dp*silu'(x): dV_j += p*dO_i, dK_j += alpha*ds*Q_i).
//
// At d_qk + d_v > 128 one wave cannot hold K, V and both accumulators in the 256 registers it
// has when two waves share a SIMD, and with one wave per SIMD nothing overlaps that wave's own
// matrix and vector instructions.  Here two waves share every 32 keys of the tile and split the
// work without repeating any of it:
//   role A (waves 0..3):  S = Q K^T,  the SiLU arithmetic (p' = s*sg and silu'),  dV^T += dO^T P
//   role B (waves 4..7):  dP = dO V^T,  dS = dP * silu' (silu' handed over by A),   dK^T += Q^T dS
// Each role issues 16 of the step's 32 matrix instructions; A holds K and the dV accumulators, B
// holds V and the dK accumulators (about half of the one-wave kernel's registers each).  silu'
// travels from A to B through LDS as fp32 in the accumulator layout (the two waves of a pair
// have identical lane layouts, so the exchange is a plain 16-byte write and read per four
// values); the mask is applied by A alone (a hidden pair has p' = silu' = 0, which zeroes dS too).
// (Handing over sg and p' instead, with silu' worked out by B, balances the two roles' vector
// work but doubles the exchange, and the LDS pipe is what this kernel is shortest of: measured
// 7.1 ms against 5.9 ms on the long skewed batch.)
//
// The stream of query rows is processed in blocks of 32 rows that live in a ring of six LDS
// buffers.  Step t:
//   A: scores of block t | SiLU of block t-1 (writes silu' of t-1) | dV contraction of block t-2
//   B: dP of block t-1   | dS of block t-2 (reads silu' of t-2)    | dK contraction of block t-3
//   B: the copy of block t+2 is issued at the start; block t+1 has landed at the end.
// One workgroup barrier per step orders the hand-over (the exchange buffers alternate by parity)
// and the reuse of ring buffers.  Steps run from 0 to blocks + 2; the blocks before block 0 are
// zeros (their ring buffers are cleared at the start) and blocks at or beyond the end are treated
// as wholly masked, so one step body serves the whole item.
// Role A is the longer role (the SiLU arithmetic is its alone) and the two meet at the barrier,
// so the step's time is A's: inside the loop A issues no copies, keeps no cursor and waits for no
// memory (B's waves do), and its last exchange write leaves a slot before the step ends.
// With the timestamp bias (BIAS) role A writes the block's bias into its score accumulator before
// the block's first product (see bias_block); the table's gradient belongs to the dq pass.
// =============================================================================================

constexpr int BR = 32;     // streamed rows per block
constexpr int NSLOT = 6;   // ring buffers
constexpr int PW = 8;      // waves per workgroup
constexpr int AHEAD_COPY = 2;  // the copy of block t + AHEAD_COPY is issued in step t

// Where the next block to copy lies: the rows of one head of Q and dO (the same rows of both
// tensors, which have equal row lengths here) and how many of the rows from there on are visible.
// Advancing costs a handful of scalar instructions per block; the segment is looked up again
// only where the stream passes from its first segment to the second.
template <int D>
struct BlockCursor {
  const __bf16* q;
  const __bf16* g;
  int valid;  // visible rows from the block's first row on (<= 0: none)
  int b;      // block index
  int row;    // the block's first row in the streamed tensors (the bias variant copies its records)
  __device__ __forceinline__ void seek(const AttnArgs& a, const Item& it, const Stream& st, int h, int blk) {
    const TileRef t = tile_ref(it, st, blk >> 1);
    const int o = (blk & 1) * BR;
    const int64_t off = (int64_t)(t.row + o) * a.num_heads * D + h * D;
    q = (const __bf16*)a.q + off;
    g = (const __bf16*)a.d_o + off;
    valid = t.valid - o;
    b = blk;
    row = t.row + o;
  }
  __device__ __forceinline__ void next(const AttnArgs& a, const Item& it, const Stream& st, int h) {
    if (b + 1 == 2 * st.n[0]) {
      seek(a, it, st, h, b + 1);
    } else {
      const int64_t step = (int64_t)BR * a.num_heads * D;
      q += step; g += step; valid -= BR; ++b; row += BR;
    }
  }
};

// Asynchronous copy of one block (BR rows of one head) into its swizzled LDS layout; see
// tile_copy_async.  Rows >= valid arrive as zeros.  One wave-wide load per wave at D = 128.
template <int D>
__device__ __forceinline__ void block_copy_async(char* buf, const __bf16* base, int rs, int valid,
                                                 int wave, int voff) {
  constexpr int CPR = D / 8, RPL = 64 / CPR, LOADS = BR / RPL;
  static_assert(LOADS == PW, "one load per wave");
  const int rows = valid < 0 ? 0 : (valid < BR ? valid : BR);
  // (readfirstlane: the size is uniform, and must be seen to be, or the load is wrapped in a loop
  // over the distinct resources of the lanes)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)base, 0, __builtin_amdgcn_readfirstlane(rows * rs), 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, HSTU_LDS(void, buf + wave * 1024), 16, voff, 0, 0, 0);
}

// The same copy issued by the four waves of role B alone (two wave-wide loads per wave): inside the
// loop role A, whose vector work makes it the longer of the two, issues no copies, keeps no
// cursor and waits for no memory.
template <int D>
__device__ __forceinline__ void block_copy_async_half(char* buf, const __bf16* base, int rs, int valid,
                                                      int w, const int (&voff2)[2]) {
  static_assert(BR / (64 / (D / 8)) == PW, "two loads per wave of one role");
  const int rows = valid < 0 ? 0 : (valid < BR ? valid : BR);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)base, 0, __builtin_amdgcn_readfirstlane(rows * rs), 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, HSTU_LDS(void, buf + (2 * w) * 1024), 16, voff2[0], 0, 0, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, HSTU_LDS(void, buf + (2 * w + 1) * 1024), 16, voff2[1], 0, 0, 0);
}

// Asynchronous copy of the timestamp records of one block into a 1 KB buffer (one wave-wide load:
// 32 records of 16 bytes; the lanes beyond them and rows >= valid arrive as zeros).
__device__ __forceinline__ void rec_block_copy_async(char* buf, const TsRecord* rec, int valid, int lane) {
  const int rows = valid < 0 ? 0 : (valid < BR ? valid : BR);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)rec, 0, __builtin_amdgcn_readfirstlane(rows * (int)sizeof(TsRecord)), 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, HSTU_LDS(void, buf), 16, lane * 16, 0, 0, 0);
}

__device__ __forceinline__ void lds_writes_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// The ring buffers: six for the blocks of Q, six for those of dO.  One array per buffer, so that the compiler can see
// that a copy into one cannot alias operand reads from another.  The compiler lays LDS out by falling alignment, which is
// why the alignments differ (at D = 128): Q's buffers at 0..48 KB, dO's at 48..96 KB, the exchange buffers and the
// rest above.  An address reaches 64 KB: from 0 for Q's, from UP_G = 32 KB, i.e. 32..96 KB, for dO's, so that one set of
// addresses per tensor serves all reads (see raised; another layout would only cost additions).
struct Rings {
  char *q0, *q1, *q2, *q3, *q4, *q5, *g0, *g1, *g2, *g3, *g4, *g5;
  __device__ __forceinline__ char* q(int b) const {
    return b == 0 ? q0 : (b == 1 ? q1 : (b == 2 ? q2 : (b == 3 ? q3 : (b == 4 ? q4 : q5))));
  }
  __device__ __forceinline__ char* g(int b) const {
    return b == 0 ? g0 : (b == 1 ? g1 : (b == 2 ? g2 : (b == 3 ? g3 : (b == 4 ? g4 : g5))));
  }
};
constexpr int UP_Q = 0, UP_G = 32768;
#define HSTU_RINGS(QB)                                       \
  __shared__ __attribute__((aligned(4096))) char rq0[QB];    \
  __shared__ __attribute__((aligned(4096))) char rq1[QB];    \
  __shared__ __attribute__((aligned(4096))) char rq2[QB];    \
  __shared__ __attribute__((aligned(4096))) char rq3[QB];    \
  __shared__ __attribute__((aligned(4096))) char rq4[QB];    \
  __shared__ __attribute__((aligned(4096))) char rq5[QB];    \
  __shared__ __attribute__((aligned(2048))) char rg0[QB];    \
  __shared__ __attribute__((aligned(2048))) char rg1[QB];    \
  __shared__ __attribute__((aligned(2048))) char rg2[QB];    \
  __shared__ __attribute__((aligned(2048))) char rg3[QB];    \
  __shared__ __attribute__((aligned(2048))) char rg4[QB];    \
  __shared__ __attribute__((aligned(2048))) char rg5[QB];    \
  const Rings ring = {rq0, rq1, rq2, rq3, rq4, rq5, rg0, rg1, rg2, rg3, rg4, rg5}

// Exchange buffer of one (parity, 32 keys): [four accumulator elements][lane] as 16-byte groups;
// xw points at the lane's first group.
constexpr int XG = 256;        // floats between the groups of four elements
constexpr int XK = 4 * XG;     // floats per 32 keys

// The operand is complete here.  (Its use is in the next step; with a branch in between the compiler would move the
// instructions that make it there, in front of that step's first operand reads.)
__device__ __forceinline__ void complete(const bf16x8& x) { asm volatile("" ::"v"(__builtin_bit_cast(u32x4, x))); }

// Role A, one step: scores of the block at qn into s_out, SiLU of s_in (p' packed into p_cur,
// silu' written to xw), dV^T += dO^T P with the block at gp and p_prev.
template <int D, class Init, class Vis>
__device__ __forceinline__ void role_a_step(const Init& init, const char* qn, const char* gp, const RowAddr<D, UP_Q>& raq,
                                            const ColAddr<D, UP_G>& cag, const bf16x8 (&kreg)[D / 16],
                                            const f32x16& s_in, f32x16& s_out,
                                            const bf16x8 (&p_prev)[2], bf16x8 (&p_cur)[2],
                                            f32x16 (&dvacc)[D / 32], float* xw, float c1, float alpha,
                                            bool mask, const Vis& vis_of) {
  constexpr int NS = D / 16;
  constexpr int AHEAD = 3;  // operand reads in flight ahead of their use
  static_assert(NS == 8, "eight slots per step: two groups of four stages");
  bf16x8 op[NS], tp[NS];
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  init(s_out);  // zeros, or the block's bias
#pragma unroll
  for (int m = 0; m < AHEAD; ++m) {
    op[m] = raq.read(qn, 0, m);
    tp[m] = cag.read(gp, m & 1, m >> 1);
  }
  fence();
  // The arithmetic of eight elements per group, one stage per slot, so that no instruction consumes
  // its predecessor's result; a group's results leave the registers (silu' to the exchange buffer,
  // p' packed) as soon as they are complete.  The first group takes slots 0..3, the second slots
  // 3..6: the last slot has no stage, so the wave's exchange writes are under way while its last
  // matrix instructions issue, and the wait for them that ends the step finds them done.
  float p[2][8], st_t[2][8], st_g[2][8];
  auto stage = [&](auto gtag, int ph) {
    constexpr int G = decltype(gtag)::value, e0 = G * 8;
    if (ph == 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) st_t[G][j] = s_in[e0 + j] * c1;
#pragma unroll
      for (int j = 0; j < 8; ++j) st_t[G][j] = __builtin_amdgcn_exp2f(st_t[G][j]);
    } else if (ph == 1) {
#pragma unroll
      for (int j = 0; j < 8; ++j) st_t[G][j] = 1.0f + st_t[G][j];
#pragma unroll
      for (int j = 0; j < 8; ++j) st_g[G][j] = __builtin_amdgcn_rcpf(st_t[G][j]);
    } else if (ph == 2) {  // p' = s * sg, p' * (1 - sg) as p' - p' * sg
#pragma unroll
      for (int j = 0; j < 8; ++j) p[G][j] = s_in[e0 + j] * st_g[G][j];
#pragma unroll
      for (int j = 0; j < 8; ++j) st_t[G][j] = __builtin_fmaf(-p[G][j], st_g[G][j], p[G][j]);
    } else {               // silu' = sg + alpha * p' * (1 - sg): two fused multiply-adds after p'
#pragma unroll
      for (int j = 0; j < 8; ++j) st_g[G][j] = __builtin_fmaf(alpha, st_t[G][j], st_g[G][j]);
      if (mask) {
        asm volatile("" ::: "memory");  // not speculable: keeps the selects off the unmasked path
        const auto vis = vis_of();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool on = vis(e0 + j);
          p[G][j] = on ? p[G][j] : 0.f;
          st_g[G][j] = on ? st_g[G][j] : 0.f;
        }
      }
#pragma unroll
      for (int q4 = 0; q4 < 2; ++q4) {
        const f32x4 vf = {st_g[G][4 * q4], st_g[G][4 * q4 + 1], st_g[G][4 * q4 + 2], st_g[G][4 * q4 + 3]};
        *HSTU_LDS(f32x4, xw + (e0 / 4 + q4) * XG) = vf;
      }
      p_cur[G] = pack8(p[G]);
      complete(p_cur[G]);
    }
  };
#pragma unroll
  for (int m = 0; m < NS; ++m) {
    s_out = mfma(op[m], kreg[m], s_out);
    dvacc[m >> 1] = mfma(tp[m], p_prev[m & 1], dvacc[m >> 1]);
    if (m + AHEAD < NS) {
      op[m + AHEAD] = raq.read(qn, 0, m + AHEAD);
      tp[m + AHEAD] = cag.read(gp, (m + AHEAD) & 1, (m + AHEAD) >> 1);
    }
    if (m < 4) stage(std::integral_constant<int, 0>{}, m);
    if (m >= 3 && m < 7) stage(std::integral_constant<int, 1>{}, m - 3);
    fence();
  }
}

// Role B, one step: dP of the block at gn into d_out, dS = d_in * silu' (read from xr) packed into
// ds_cur, dK^T += Q^T dS with the block at qp and ds_prev.
template <int D>
__device__ __forceinline__ void role_b_step(const char* gn, const char* qp, const RowAddr<D, UP_G>& rag,
                                            const ColAddr<D, UP_Q>& caq, const bf16x8 (&vreg)[D / 16],
                                            const f32x16& d_in, f32x16& d_out,
                                            const bf16x8 (&ds_prev)[2], bf16x8 (&ds_cur)[2],
                                            f32x16 (&dkacc)[D / 32], const float* xr) {
  constexpr int NS = D / 16;
  constexpr int AHEAD = 3;
  bf16x8 op[NS], tp[NS];
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
#pragma unroll
  for (int r = 0; r < 16; ++r) d_out[r] = 0.f;
  f32x4 x4[4];
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) x4[q4] = *HSTU_LDS(const f32x4, xr + q4 * XG);
#pragma unroll
  for (int m = 0; m < AHEAD; ++m) {
    op[m] = rag.read(gn, 0, m);
    tp[m] = caq.read(qp, m & 1, m >> 1);
  }
  fence();
  float ds[16];
#pragma unroll
  for (int m = 0; m < NS; ++m) {
    d_out = mfma(op[m], vreg[m], d_out);
    dkacc[m >> 1] = mfma(tp[m], ds_prev[m & 1], dkacc[m >> 1]);
    if (m + AHEAD < NS) {
      op[m + AHEAD] = rag.read(gn, 0, m + AHEAD);
      tp[m + AHEAD] = caq.read(qp, (m + AHEAD) & 1, (m + AHEAD) >> 1);
    }
#pragma unroll
    for (int e = m * 16 / NS; e < (m + 1) * 16 / NS; ++e) ds[e] = d_in[e] * x4[e >> 2][e & 3];
    fence();
  }
  ds_cur[0] = pack8(ds);
  ds_cur[1] = pack8(ds + 8);
  complete(ds_cur[0]);
  complete(ds_cur[1]);
  fence();
}

// The whole item for one role (ROLE 0: A, 1: B).  SIDE 1: owners are keys, the dk/dv pass.  SIDE 0: owners are queries,
// forward and dq pass in one (see hstu_fwd_dq_pair_bf16), with the names of the other side:
// a.k, a.v: the rows owned (Q and dO); a.q, a.d_o: the rows streamed (K and V); a.dv, a.dk: the results (O and dQ).
template <int D, int ROLE, bool BIAS, int SIDE>
__device__ __forceinline__ void pair_body(const AttnArgs& a, const Item& it, int h, const Rings& ring, float* xbuf0, float* xbuf1, char* rec0, char* rec1,
                                          char* rec2, char* rec3, char* rec4, char* rec5, float* wtab) {
  constexpr int QB = BR * D * 2;
  auto recb = [&](int b) {  // the records of the block in ring buffer b (bias variant)
    return b == 0 ? rec0 : (b == 1 ? rec1 : (b == 2 ? rec2 : (b == 3 ? rec3 : (b == 4 ? rec4 : rec5))));
  };
  const int H = a.num_heads;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave & 3;  // which 32 keys of the tile
  const int64_t sr = (int64_t)H * D;
  const int rs = H * D * 2;  // bytes per row
  const int orow = g * 32 + n;

  const Stream st = make_stream<SIDE>(it, a.causal);
  const int NBLK = 2 * st.total;  // 32-row blocks of the stream
  // the lane's part of a block copy: row wave * RPL + lane / CPR, swizzled chunk
  const int crow = wave * (64 / (D / 8)) + lane / (D / 8);
  const int voff = crow * rs + (((lane % (D / 8)) ^ swz<D>(crow)) << 4);
  BlockCursor<D> cur;
  auto copy_next = [&](char* qbuf, char* gbuf, char* rbuf) {  // copies block cur.b, then moves on
    block_copy_async<D>(qbuf, cur.q, rs, cur.valid, wave, voff);
    block_copy_async<D>(gbuf, cur.g, rs, cur.valid, wave, voff);
    if (BIAS && wave == 0) rec_block_copy_async(rbuf, a.ts_rec + cur.row, cur.valid, lane);
    cur.next(a, it, st, h);
  };
  // The copy issued in every step, by role B: block cur.b while the stream lasts, afterwards a copy
  // of no rows (zeros arrive; the buffer is one that no later step reads for anything that counts).
  // Every step thus issues the same four loads and waits with the same count, with no branch around
  // either: the compiler's own bookkeeping of copies in flight follows that, whereas with a
  // condition evaluated at both places it assumed older copies pending and put a wait for
  // everything in front of some steps' first operand reads, i.e. right behind the copy just issued.
  int voff2[2] = {0, 0};
  if constexpr (ROLE == 1) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r2 = (2 * g + i) * (64 / (D / 8)) + lane / (D / 8);
      voff2[i] = r2 * rs + (((lane % (D / 8)) ^ swz<D>(r2)) << 4);
    }
  }
  // (With the bias every wave of role B also issues the load of the block's records: the same
  // kilobyte four times, so that all four keep the same count of loads in flight.)
  auto copy_step = [&](char* qbuf, char* gbuf, char* rbuf, bool live) {
    const int valid = live ? cur.valid : 0;
    block_copy_async_half<D>(qbuf, cur.q, rs, valid, g, voff2);
    block_copy_async_half<D>(gbuf, cur.g, rs, valid, g, voff2);
    if constexpr (BIAS) rec_block_copy_async(rbuf, a.ts_rec + (live ? cur.row : 0), valid, lane);
    if (live) cur.next(a, it, st, h);
  };
  auto block_pos = [&](int b) { return tile_ref(it, st, b >> 1).pos + (b & 1) * BR; };

  // Ring buffers 4 and 5 stand for the two blocks before the first one (the contractions of the
  // first two steps read them against operands that are zero): cleared, so that those products
  // are zeros whatever the memory held.
  {
    const u32x4 z = {0u, 0u, 0u, 0u};
    static_assert(QB / 16 == PW * 64, "one chunk per thread");
    *HSTU_LDS(u32x4, ring.q4 + tid * 16) = z;
    *HSTU_LDS(u32x4, ring.q5 + tid * 16) = z;
    *HSTU_LDS(u32x4, ring.g4 + tid * 16) = z;
    *HSTU_LDS(u32x4, ring.g5 + tid * 16) = z;
  }
  bf16x8 oreg[D / 16];  // A: the K rows, B: the V rows
  {
    const __bf16* og = (const __bf16*)(ROLE == 0 ? a.k : a.v) + (int64_t)it.row0 * sr + h * D;
    load_owner<D>(oreg, og, sr, orow, it.nrows, hh);
  }
  if (NBLK > 0) {
    cur.seek(a, it, st, h, 0);
    copy_next(ring.q0, ring.g0, rec0);
    copy_next(ring.q1, ring.g1, rec1);  // (NBLK is even)
  }
  // The bias enters the scores only, i.e. role A's product (the table's gradient is the dq pass's).
  BiasCtx bias = {};
  if constexpr (BIAS) bias = bias_setup<PW * 64>(a, wtab, it, orow, tid, hh);  // (all waves: has a barrier)

  const float c1 = -a.alpha * 1.4426950408889634f;
  const int o_lo = it.pos0 + g * 32, o_hi = o_lo + 31;  // positions of the wave's owner rows
  // The blocks the diagonal touches or hides: the first ones up to last_masked (keys own: position < o_hi), or the
  // last ones from first_masked on (queries own: position + 31 > o_lo); block positions grow with the index.
  int last_masked = -1, first_masked = NBLK;
  if (ROLE == 0 && a.causal) {
#pragma unroll
    for (int s = 1; s >= 0; --s) {
      const int i0 = s ? 2 * st.n[0] : 0, nb = 2 * st.n[s];
      const int p0 = it.seg_pos0[s] + st.beg[s];
      if (nb > 0) {
        const int m = (o_hi - 1 - p0) >> 5;
        if (m >= 0 && last_masked < 0) last_masked = i0 + (m < nb - 1 ? m : nb - 1);
        const int f0 = ((o_lo - 31 - p0) >> 5) + 1, f = f0 < 0 ? 0 : f0;
        if (f < nb) first_masked = i0 + f;
      }
    }
  }

  f32x16 acc[D / 32];  // A: dV^T, B: dK^T
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  RowAddr<D, ROLE == 0 ? UP_Q : UP_G> ra;  // A: rows of Q, B: rows of dO
  ColAddr<D, ROLE == 0 ? UP_G : UP_Q> ca;  // A: dO transposed, B: Q transposed
  ra.init(n, hh); ca.init(lane);

  lds_writes_done();
  tile_copy_wait<0>();
  tile_barrier();

  if (NBLK > 0) {
    f32x16 sd[2];     // A: S, B: dP of the blocks of even / odd index
    bf16x8 pk[2][2];  // A: P, B: dS of the blocks of even / odd index
#pragma unroll
    for (int x = 0; x < 2; ++x) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sd[x][r] = 0.f;
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int e = 0; e < 8; ++e) pk[x][y][e] = (__bf16)0.f;
    }
    float* xa0 = xbuf0 + g * XK + lane * 4;
    float* xa1 = xbuf1 + g * XK + lane * 4;
    const int nsteps = NBLK + 3;
    BlockTable tab = {};
    if constexpr (BIAS && ROLE == 0) {
      tab.fill(bias, 0, NBLK, it, st, lane);
      tab.fill(bias, 64, NBLK, it, st, lane);
    }

    auto step = [&](int t, auto tag) {
      constexpr int S = decltype(tag)::value;  // t mod 6; S & 1 is the parity of t
      if constexpr (ROLE == 1)
        copy_step(ring.q((S + AHEAD_COPY) % NSLOT), ring.g((S + AHEAD_COPY) % NSLOT), recb((S + AHEAD_COPY) % NSLOT),
                  t + AHEAD_COPY < NBLK);
      if constexpr (ROLE == 0) {
        if constexpr (BIAS)  // the stream enters one set of the block table: refill the other
          if (t > 0 && (t & 63) == 0) tab.fill(bias, t + 64, NBLK, it, st, lane);
        if (t <= NBLK + 1) {  // (nothing left to contract in the last step)
          // block t-1: masked when the diagonal touches it or when it lies beyond the stream
          const int b = t - 1;
          const bool mask = SIDE == 1 ? b <= last_masked || b >= NBLK : b >= first_masked;
          auto vis_of = [&] {
            const int rel = o_lo + n - block_pos(b < 0 ? 0 : b);
            if constexpr (SIDE == 1) return VisAfter{b >= NBLK ? (1 << 20) : rel, hh};
            else return VisBefore{b >= NBLK ? -(1 << 20) : rel, hh};
          };
          const ScoreInit<BIAS> init = {&bias, recb(S), 0, BIAS ? tab.get(t) : BlockBias{}};
          role_a_step<D>(init, ring.q(S), ring.g((S + 4) % NSLOT), ra, ca, oreg, sd[(S + 1) & 1], sd[S & 1],
                         pk[S & 1], pk[(S + 1) & 1], acc, (S + 1) & 1 ? xa1 : xa0, c1, a.alpha, mask, vis_of);
          lds_writes_done();
        }
      } else {
        if (t >= 1)  // (nothing to work on in the first step)
          role_b_step<D>(ring.g((S + 5) % NSLOT), ring.q((S + 3) % NSLOT), ra, ca, oreg, sd[S & 1],
                         sd[(S + 1) & 1], pk[(S + 1) & 1], pk[S & 1], acc, S & 1 ? xa1 : xa0);
      }
      // block t+1 must have landed; the copies of the later blocks may stay in flight
      if constexpr (ROLE == 1) tile_copy_wait<(BIAS ? 5 : 4) * (AHEAD_COPY - 1)>();
      tile_barrier();
    };
    for (int t = 0; t < nsteps; t += NSLOT) {
      step(t, std::integral_constant<int, 0>{});
      if (t + 1 < nsteps) step(t + 1, std::integral_constant<int, 1>{});
      if (t + 2 < nsteps) step(t + 2, std::integral_constant<int, 2>{});
      if (t + 3 < nsteps) step(t + 3, std::integral_constant<int, 3>{});
      if (t + 4 < nsteps) step(t + 4, std::integral_constant<int, 4>{});
      if (t + 5 < nsteps) step(t + 5, std::integral_constant<int, 5>{});
    }
    tile_copy_wait<0>();  // (the last steps' empty copies: nothing may be in flight when the workgroup's LDS is released)
  }

  // Accumulators: lane holds key row n, elements c*32 + 8*(r/4) + 4*hh + r%4 (P and dS are held
  // without their factor alpha / N).
  if (orow < it.nrows) {
    if (SIDE == 0 && it.part > 0)  // one part of a split tile: an fp32 partial result, summed by the reduce kernel
      store_owner_major<D>(ROLE == 0 ? a.partial : a.partial2, (((int64_t)(it.part - 1) * H + h) * 128 + orow) * D, acc,
                           a.alpha * a.inv_n, hh, 0, 1);
    else
      store_owner_major<D>(ROLE == 0 ? a.dv : a.dk, ((int64_t)it.row0 + orow) * sr + h * D, acc, a.alpha * a.inv_n, hh,
                           a.accumulate, a.out_f32);
  }
}

// SELF: the workgroup works its item out from the offsets (a variant of its own: with both ways in one
// kernel the long skewed batch took 1.6 % longer, the register allocation of the steps being different).
template <int D, bool BIAS, bool SELF, int SIDE>
__device__ __forceinline__ void pair_item(const AttnArgs& a, int unit, const Rings& ring, float* xbuf0, float* xbuf1, char* rec0,
                                          char* rec1, char* rec2, char* rec3, char* rec4, char* rec5, float* wtab) {
  const Unit un = unit_of(a, unit);
  Item it;
  if (!un.on || !(SELF ? get_item(a, un.slot, it) : fetch_item<false>(a.plan, un.slot, it))) return;
  const int role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  if (role == 0)
    pair_body<D, 0, BIAS, SIDE>(a, it, un.h, ring, xbuf0, xbuf1, rec0, rec1, rec2, rec3, rec4, rec5, wtab);
  else
    pair_body<D, 1, BIAS, SIDE>(a, it, un.h, ring, xbuf0, xbuf1, rec0, rec1, rec2, rec3, rec4, rec5, wtab);
}

template <int D, bool BIAS, bool SELF>
__global__ void __launch_bounds__(PW * 64) hstu_dkdv_pair_bf16(AttnArgs a) {
  HSTU_RINGS(BR * D * 2);
  __shared__ __attribute__((aligned(1024))) float xbuf0[4 * XK];  // silu' of blocks of even index
  __shared__ __attribute__((aligned(1024))) float xbuf1[4 * XK];  // ... of odd index
  // bias variant: the timestamp records of the blocks in the ring buffers, and the table
  __shared__ __attribute__((aligned(1024))) char rec0[BIAS ? 1024 : 16];
  __shared__ __attribute__((aligned(1024))) char rec1[BIAS ? 1024 : 16];
  __shared__ __attribute__((aligned(1024))) char rec2[BIAS ? 1024 : 16];
  __shared__ __attribute__((aligned(1024))) char rec3[BIAS ? 1024 : 16];
  __shared__ __attribute__((aligned(1024))) char rec4[BIAS ? 1024 : 16];
  __shared__ __attribute__((aligned(1024))) char rec5[BIAS ? 1024 : 16];
  __shared__ float wtab[BIAS ? MAX_TS_BUCKETS : 1];
  pair_item<D, BIAS, SELF, 1>(a, blockIdx.x, ring, xbuf0, xbuf1, rec0, rec1, rec2, rec3, rec4, rec5, wtab);
}

// Forward and dq pass in one, for calls that want both (a context-parallel rank's partial): the dk/dv pass with the
// sides' parts exchanged.  Queries own, K and V are streamed,
//   role A:  S^T = K Q^T,  the SiLU arithmetic,  O^T += V^T P^T
//   role B:  dP^T = V dO^T,  dS^T = dP^T * silu',  dQ^T += K^T dS^T
// so the steps, the hand-over and the buffers are the same to the instruction.  The scores, their exponentials and
// the copies of K and V are done once where the two passes did them twice: 8 units of matrix work (2 d flops per pair)
// instead of 10, one schedule instead of two.
template <int D, bool SELF>
__global__ void __launch_bounds__(PW * 64) hstu_fwd_dq_pair_bf16(AttnArgs a) {
  HSTU_RINGS(BR * D * 2);
  __shared__ __attribute__((aligned(1024))) float xbuf0[4 * XK];
  __shared__ __attribute__((aligned(1024))) float xbuf1[4 * XK];
  pair_item<D, false, SELF, 0>(a, blockIdx.x, ring, xbuf0, xbuf1, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
}

// =============================================================================================
// The same pair of roles for large batches of short sequences (natural order; per-sequence or packed
// tiles): 256 workgroups, one per CU, each walking over a run of (item, head) units whose blocks of
// query rows form one stream.  Step t is what it is above, but the block of the scores, the block of
// the SiLU and the block of the contraction may belong to different items: at an item's step 0 role A
// scores its first block with the new K rows while it does the SiLU of the previous item's last block
// and contracts the one before, and so on; the previous item's dV is complete after step 1, its dK
// after step 2.  So an item costs its blocks and nothing else: no fill and drain of the pipeline (three
// steps of the nine an item has on 300..600-row sequences), no wait for its first rows.
// Items have at least three blocks (blocks of no rows are added to shorter ones: zeros, which
// contribute nothing), so that at most two items are in the pipeline.  After the last unit comes an
// item of no rows whose three steps drain it.
// The next item's rows are on their way while an item is worked on: role A loads the K rows into registers of their own
// (32 a lane, which the ring's addresses within reach of one set of LDS offsets left free) and has the V rows copied into
// 32 KB of LDS, the last of the CU's 160, from which role B takes them after step 0.
// Measured against the one-wave kernel that walks items one after the other, H = 4: 1536 sequences of 300..600 rows
// 1560 -> 1415 us, 1024 of 350 +- 33 % 751 -> 659, 512 of 700 +- 33 % 1010 -> 977; with the next rows ahead and runs of
// equal work (balanced_run) the first 1466 -> 1320 in another session.
// =============================================================================================

// What a step of an item's middle does not take: kept out of line, so that such a step runs straight through (a branch
// taken costs some 30 cycles, and role A's issue is the step's time).
__device__ __forceinline__ bool rare(bool x) { return __builtin_expect(x, false); }

// What the roles know about an item of one streamed segment.
struct WalkItem {
  int row0, nrows, pos0, h;
  int srow, spos;  // streamed row and position of block 0
  int rows;        // streamed rows from block 0 on
  int nblk;        // blocks, at least three
};
__device__ __forceinline__ WalkItem walk_item(const Item& it, int h, int causal) {
  int beg, end;
  visible_range<1>(it, 0, causal, beg, end);
  if (it.nseg < 1 || it.nrows <= 0) beg = end = 0;
  WalkItem w;
  w.row0 = it.row0; w.nrows = it.nrows; w.pos0 = it.pos0; w.h = h;
  w.srow = it.seg_row0[0] + beg;
  w.spos = it.seg_pos0[0] + beg;
  w.rows = end - beg;
  const int n = (w.rows + BR - 1) / BR;
  w.nblk = n > 3 ? n : 3;
  return w;
}

// Workgroup u's run of a list in natural order, of equal work for each of the workgroups of a head
// (Item::before): slots [slot, slot + left).  The XCD of workgroup u works on head (u mod 8) mod H and, of 8 / H
// neighbouring parts of the list, on one.  Both ends are searched at once, 64 items at a time; whatever the
// items hold, the runs cover the list (every end is found by one rule, the first is 0 and the last the list's).
// Runs of equal numbers of items had 941 blocks at most where 862 are the mean for 1536 sequences of 300..600 rows, H = 4, and
// 848 of 691 for 512 of 200..1200; of equal work 874 and 721, and lists sorted by length no longer differ from shuffled ones
// (1536 sequences of median 256, H = 8, backward 5298 -> 4590 us sorted, 4993 -> 4230 shuffled).
__device__ __forceinline__ void balanced_run(const AttnArgs& a, int u, int count, int& slot, int& left) {
  const int lane = threadIdx.x & 63, x = u & 7, wgs = (int)(gridDim.x >> 3);
  const int runs = a.xcd_parts * wgs, run = (x / a.num_heads) * wgs + (u >> 3);
  const unsigned total = (unsigned)a.plan.header[3];
  int lo[2], hi[2];
  unsigned want[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = run + i;
    want[i] = (unsigned)((uint64_t)total * (unsigned)r / (unsigned)runs);
    lo[i] = r < runs ? 0 : count;
    hi[i] = r > 0 ? count : 0;
  }
  while (lo[0] < hi[0] || lo[1] < hi[1]) {  // (the first item of `want` blocks before it lies in lo..hi)
    int step[2];
    unsigned v[2];
    bool on[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      step[i] = (hi[i] - lo[i] + 63) >> 6;
      const int64_t at = lo[i] + (int64_t)lane * step[i];
      on[i] = at < hi[i];
      v[i] = on[i] ? (unsigned)a.plan.items[at].before : 0u;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int below = __builtin_popcountll(__ballot(on[i] && v[i] < want[i]));
      const int64_t upper = lo[i] + (int64_t)below * step[i];
      hi[i] = upper < hi[i] ? (int)upper : hi[i];
      if (below > 0) lo[i] += (below - 1) * step[i] + 1;
    }
  }
  slot = __builtin_amdgcn_readfirstlane(lo[0]);
  left = __builtin_amdgcn_readfirstlane(lo[1]) - slot;
}

template <int D, int ROLE, bool PACKED>
__device__ __forceinline__ void pair_walk(const AttnArgs& a, int u, int stride, int end, const Rings& ring, char* vrows,
                                          float* xbuf0, float* xbuf1) {
  constexpr int QB = BR * D * 2;
  const int H = a.num_heads;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave & 3;  // which 32 keys of the tile
  const int64_t sr = (int64_t)H * D;
  const int rs = H * D * 2;  // bytes per row
  const int orow = g * 32 + n;
  const float c1 = -a.alpha * 1.4426950408889634f;
  const int count = a.plan.header[0];

  // The workgroup's share, `left` units of `stride`: slot and head of the next one to be looked up (see unit_of).
  int slot, h, left, dslot, dh;
  if (!PACKED && a.walk_costs) {
    balanced_run(a, u, count, slot, left);
    h = (u & 7) % H; dslot = 1; dh = 0;
  } else if (a.xcd_parts <= 1) {
    slot = u / H; h = u % H; dslot = stride / H; dh = stride % H;
    left = (end - u + stride - 1) / stride;  // (end <= count * H)
  } else {  // stride is a multiple of 8: the same head and the same part of the list throughout
    const int per = (count + a.xcd_parts - 1) / a.xcd_parts, x = u & 7, part = (x / H) * per;
    slot = part + (u >> 3); h = x % H; dslot = stride >> 3; dh = 0;
    int last = part + ((end - x + 7) >> 3);
    last = last < part + per ? last : part + per;
    last = last < count ? last : count;
    left = last > slot ? (last - slot + dslot - 1) / dslot : 0;
  }
  if (left <= 0) return;  // (every wave alike; the loop below counts on one unit at least)
  // Descriptions: `raw` is that of the unit after the next one, one of its sixteen words per lane (zeros beyond the last
  // unit), brought into scalar registers by decode.
  const __amdgpu_buffer_rsrc_t items =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.plan.items, 0, a.max_items * (int)sizeof(Item), 0x00020000);
  int raw_h = 0;
  auto load_raw = [&] {
    raw_h = h;
    const int r = (int)__builtin_amdgcn_raw_buffer_load_b32(
        items, left > 0 ? (lane & 15) * 4 : -4, left > 0 ? slot * (int)sizeof(Item) : 0, 0);
    --left;
    slot += dslot;
    h += dh;
    if (h >= H) { h -= H; ++slot; }
    return r;
  };
  auto decode = [&](int raw) {
    Item it = {};
    auto word = [&](int i) { return __builtin_amdgcn_readlane(raw, i); };
    it.row0 = word(0); it.nrows = word(1); it.pos0 = word(2); it.nseg = word(3);
    it.seg_row0[0] = word(4); it.seg_len[0] = word(6); it.seg_pos0[0] = word(8);
    return walk_item(it, raw_h, a.causal);
  };
  int todo = left;  // units whose first step is still to come
  int raw = load_raw();
  WalkItem cur = decode(raw), nxt = {}, prev = {};
  raw = load_raw();

  // The rows of the item this role owns: K (role A), V (role B).  While an item is worked on role A loads the next one's K
  // rows into registers of their own and has its V rows copied into LDS, where role B picks them up.
  bf16x8 oreg[D / 16], knext[ROLE == 0 ? D / 16 : 1];
  auto request_rows = [&](const WalkItem& w, bf16x8 (&k)[D / 16]) {  // (role A)
    const int64_t off = (int64_t)w.row0 * sr + w.h * D;
    load_owner<D>(k, (const __bf16*)a.k + off, sr, orow, w.nrows, hh);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const __bf16*)a.v + off), 0, __builtin_amdgcn_readfirstlane(w.nrows * rs), 0x00020000);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = g * 32 + i * (64 / (D / 8)) + lane / (D / 8);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, HSTU_LDS(void, vrows + (g * 8 + i) * 1024), 16,
                                               r * rs + (((lane % (D / 8)) ^ swz<D>(r)) << 4), 0, 0, 0);
    }
  };
  // The stream of blocks as role B copies it, two blocks ahead.
  const __bf16 *cq = nullptr, *cg = nullptr;
  int cvalid = 0, cleft = 0;  // visible rows from the block on, blocks of the item from it on
  auto seek = [&](const WalkItem& w) {
    const int64_t off = (int64_t)w.srow * sr + w.h * D;
    cq = (const __bf16*)a.q + off;
    cg = (const __bf16*)a.d_o + off;
    cvalid = w.rows;
    cleft = w.nblk;
  };
  int voff2[2] = {0, 0};
  if constexpr (ROLE == 1) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r2 = (2 * g + i) * (64 / (D / 8)) + lane / (D / 8);
      voff2[i] = r2 * rs + (((lane % (D / 8)) ^ swz<D>(r2)) << 4);
    }
  }
  auto copy_step = [&](char* qbuf, char* gbuf) {
    block_copy_async_half<D>(qbuf, cq, rs, cvalid, g, voff2);
    block_copy_async_half<D>(gbuf, cg, rs, cvalid, g, voff2);
    const int64_t step = (int64_t)BR * sr;
    cq += step; cg += step; cvalid -= BR; --cleft;
  };

  {
    const u32x4 z = {0u, 0u, 0u, 0u};
    // (the two blocks before the first one)
    static_assert(QB / 16 == PW * 64, "one chunk per thread");
    *HSTU_LDS(u32x4, ring.q4 + tid * 16) = z;
    *HSTU_LDS(u32x4, ring.q5 + tid * 16) = z;
    *HSTU_LDS(u32x4, ring.g4 + tid * 16) = z;
    *HSTU_LDS(u32x4, ring.g5 + tid * 16) = z;
  }
  if constexpr (ROLE == 1) {
    seek(cur);
    copy_step(ring.q0, ring.g0);
    copy_step(ring.q1, ring.g1);
  }
  if constexpr (ROLE == 0) {
    request_rows(cur, oreg);
  } else {
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) oreg[i][e] = (__bf16)0.f;
  }

  f32x16 acc[D / 32];  // A: dV^T, B: dK^T
  auto clear_acc = [&] {
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  };
  clear_acc();
  RowAddr<D, ROLE == 0 ? UP_Q : UP_G> ra;  // A: rows of Q, B: rows of dO
  ColAddr<D, ROLE == 0 ? UP_G : UP_Q> ca;  // A: dO transposed, B: Q transposed
  ra.init(n, hh); ca.init(lane);

  // Role A's masks of the item whose block the SiLU stage works on.
  int2 wsq = {};
  Window win = {};
  int m_last = -1, m_pos = 0, m_klo = 0;  // last block the diagonal touches, position of block 0, the wave's first key
  auto bounds_of = [&](const WalkItem& w) {
    return PACKED ? window_bounds(a.row_seq, w.row0 + orow, orow < w.nrows) : make_int2(0, 0);
  };
  if constexpr (ROLE == 0) wsq = bounds_of(cur);

  f32x16 sd[2];     // A: S, B: dP of the blocks of even / odd index
  bf16x8 pk[2][2];  // A: P, B: dS of the blocks of even / odd index
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int r = 0; r < 16; ++r) sd[x][r] = 0.f;
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int e = 0; e < 8; ++e) pk[x][y][e] = (__bf16)0.f;
  }
  float* xa0 = xbuf0 + g * XK + lane * 4;
  float* xa1 = xbuf1 + g * XK + lane * 4;
  lds_writes_done();
  tile_copy_wait<0>();
  tile_barrier();

  int s = 0;            // step of the item
  bool first = true, drain = false, stored = false;  // stored: role B wrote the previous item's rows in the last step
  // The previous item's rows (see store_owner_major), through a buffer of its rows: the stores of lanes
  // beyond them are dropped, so a wave always issues eight.
  auto store_prev = [&] {
    __bf16* base = (__bf16*)(ROLE == 0 ? a.dv : a.dk) + (int64_t)prev.row0 * sr + prev.h * D;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, __builtin_amdgcn_readfirstlane(prev.nrows * rs), 0x00020000);
    const int voff = orow * rs + 16 * hh;
    const float scale = a.alpha * a.inv_n;
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
#pragma unroll
      for (int pr = 0; pr < 2; ++pr)
        __builtin_amdgcn_raw_buffer_store_b128(owner_chunk(acc[c], pr, scale), rsrc, voff + c * 64 + pr * 32, 0, 0);
    // (zeros the compiler cannot see: known ones it kept in 64 registers of their own and moved in every step)
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float z;
        asm volatile("v_mov_b32 %0, 0" : "=v"(z));
        acc[i][r] = z;
      }
  };

  auto step = [&](auto tag) {  // returns true when the stream has been drained
    constexpr int S = decltype(tag)::value;  // step number mod 6
    if (rare(s == 1)) {  // the next item's description, and the request for the one after
      nxt = decode(raw);
      raw = load_raw();
    }
    if constexpr (ROLE == 0) {
      bool mask;
      if (rare(s == 1)) {  // from here on the SiLU stage works on this item
        if constexpr (PACKED) {
          win = make_window(wsq, cur.row0 + orow, orow < cur.nrows, 1, a.causal);
          wsq = bounds_of(nxt);
        }
        request_rows(nxt, knext);
        m_klo = cur.pos0 + g * 32;
        m_last = !PACKED && a.causal ? (m_klo + 30 - cur.spos) >> 5 : -1;
        m_pos = cur.spos;
      } else {
        m_pos += BR;
        --m_last;
      }
      // m_pos: position of the block of the SiLU stage, m_last: blocks from it to the last masked one
      mask = PACKED ? win.masks(m_pos) : m_last >= 0;
      auto vis_of = [&] {
        if constexpr (PACKED) return win.vis(m_pos, hh);
        else return VisAfter{m_klo + n - m_pos, hh};
      };
      const ScoreInit<false> init = {nullptr, nullptr, 0, BlockBias{}};
      role_a_step<D>(init, ring.q(S), ring.g((S + 4) % NSLOT), ra, ca, oreg, sd[(S + 1) & 1], sd[S & 1], pk[S & 1],
                     pk[(S + 1) & 1], acc, (S + 1) & 1 ? xa1 : xa0, c1, a.alpha, mask, vis_of);
      lds_writes_done();
      if (rare(s == 1)) {
        store_prev();
        prev = cur;
      }
      if (rare(s + 1 == cur.nblk)) {
        // (Waited for here: with loads that may be pending when a step begins the compiler makes every step wait for all
        // of the wave's memory operations, the stores above among them.)
        tile_copy_wait<0>();
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) oreg[ks] = knext[ks];
      }
    } else {
      if (rare(cleft == 0)) seek(nxt);  // (in step 1 at the earliest)
      copy_step(ring.q((S + AHEAD_COPY) % NSLOT), ring.g((S + AHEAD_COPY) % NSLOT));
      __builtin_amdgcn_sched_barrier(0);  // (the waits below count on this order)
      if (!rare(first))
        role_b_step<D>(ring.g((S + 5) % NSLOT), ring.q((S + 3) % NSLOT), ra, ca, oreg, sd[S & 1], sd[(S + 1) & 1],
                       pk[(S + 1) & 1], pk[S & 1], acc, S & 1 ? xa1 : xa0);
      first = false;
      __builtin_amdgcn_sched_barrier(0);
      if (rare(s == 0)) {  // the item's V rows (they landed before the last barrier)
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) oreg[ks] = ra.read(vrows, g, ks);
        lds_writes_done();  // (role A has the next ones copied there in the next step)
      }
      // At the end of a step the previous step's copies must have landed.  Behind them are this step's copies, 4, and
      // the 8 stores of step 2.
      if (rare(s == 2)) {
        store_prev();
        prev = cur;
        __builtin_amdgcn_sched_barrier(0);
        tile_copy_wait<12>();
      } else if (rare(stored)) {
        tile_copy_wait<12>();
      } else {
        tile_copy_wait<4>();
      }
      stored = s == 2;
    }
    tile_barrier();
    if (rare(++s == cur.nblk)) {
      if (drain) return true;
      s = 0;
      cur = nxt;
      drain = --todo <= 0;
    }
    return false;
  };
  while (true) {
    if (step(std::integral_constant<int, 0>{})) break;
    if (step(std::integral_constant<int, 1>{})) break;
    if (step(std::integral_constant<int, 2>{})) break;
    if (step(std::integral_constant<int, 3>{})) break;
    if (step(std::integral_constant<int, 4>{})) break;
    if (step(std::integral_constant<int, 5>{})) break;
  }
  tile_copy_wait<0>();
}

template <int D, bool PACKED>
__global__ void __launch_bounds__(PW * 64) hstu_dkdv_walk_bf16(AttnArgs a) {
  constexpr int QB = BR * D * 2;
  HSTU_RINGS(QB);
  __shared__ __attribute__((aligned(1024))) char vrows[128 * D * 2];  // V rows of the next item
  __shared__ __attribute__((aligned(1024))) float xbuf0[4 * XK];
  __shared__ __attribute__((aligned(1024))) float xbuf1[4 * XK];
  int u = blockIdx.x, stride = (int)gridDim.x, end = unit_count(a, a.plan.header[0]);
  if (!a.walk_costs) {
    walk_share(a, u, stride, end);
    if (u >= end) return;
  }
  const int role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  if (role == 0)
    pair_walk<D, 0, PACKED>(a, u, stride, end, ring, vrows, xbuf0, xbuf1);
  else
    pair_walk<D, 1, PACKED>(a, u, stride, end, ring, vrows, xbuf0, xbuf1);
}

}  // namespace

// The pair kernel serves per-sequence schedules, with or without the timestamp bias (no packed
// tiles, no walking workgroups), of the head dimensions that do not fit two workgroups per CU.
bool dkdv_pair_supported(const AttnArgs& a, int d_qk, int d_v) {
  if (a.ts_rec && (a.nb < 1 || a.nb > MAX_TS_BUCKETS || !a.ts_w || !a.ts_rec_own)) return false;
  return d_qk == 128 && d_v == 128 && !a.row_seq && !a.large_batch && !a.walk_chunks && a.waves == 4;
}

// Large batches of short sequences: schedules in natural order, one streamed segment per item, bf16
// outputs that are not added to (the steps hold six copies of the epilogue, and the general one is
// large; fp32 outputs keep the one-wave kernel).
bool dkdv_walk_supported(const AttnArgs& a, int d_qk, int d_v) {
  return d_qk == 128 && d_v == 128 && !a.ts_rec && a.single_segment && (a.row_seq || a.walk_chunks) && a.waves == 4 &&
         !a.out_f32 && !a.accumulate && (int64_t)a.max_items * (int64_t)sizeof(Item) < (1ll << 31);
}

hipError_t launch_dkdv_walk_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  if (!dkdv_walk_supported(a, d_qk, d_v)) return hipErrorInvalidValue;
  const int64_t units = a.xcd_parts <= 1 ? (int64_t)a.max_items * a.num_heads
                                         : 8 * (((int64_t)a.max_items + a.xcd_parts - 1) / a.xcd_parts);
  const dim3 grid((unsigned)(units < 256 ? units : 256)), block(PW * 64);
  if (a.row_seq) hipLaunchKernelGGL((hstu_dkdv_walk_bf16<128, true>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((hstu_dkdv_walk_bf16<128, false>), grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_dkdv_pair_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  if (!dkdv_pair_supported(a, d_qk, d_v)) return hipErrorInvalidValue;
  const int64_t units = a.xcd_parts <= 1 ? (int64_t)a.max_items * a.num_heads
                                         : 8 * (((int64_t)a.max_items + a.xcd_parts - 1) / a.xcd_parts);
#define HSTU_PAIR(BIAS, SELF) \
  hipLaunchKernelGGL((hstu_dkdv_pair_bf16<128, BIAS, SELF>), dim3((unsigned)units), dim3(PW * 64), 0, stream, a)
  if (a.self.off) { if (a.ts_rec) HSTU_PAIR(true, true); else HSTU_PAIR(false, true); }
  else { if (a.ts_rec) HSTU_PAIR(true, false); else HSTU_PAIR(false, false); }
#undef HSTU_PAIR
  return hipGetLastError();
}

hipError_t launch_fwd_dq_pair_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  if (d_qk != 128 || d_v != 128 || a.ts_rec || a.row_seq || a.waves != 4) return hipErrorInvalidValue;
  const dim3 grid((unsigned)grid_units(a)), block(PW * 64);
  if (a.self.off) hipLaunchKernelGGL((hstu_fwd_dq_pair_bf16<128, true>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((hstu_fwd_dq_pair_bf16<128, false>), grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace hstu
