// fp32 jagged HSTU attention (forward, dk/dv pass, dq pass): the all-fp32 data type of the
// library, on the fp32 matrix instruction (products and sums in fp32), with a sigmoid to about an ulp
// (see sigmoid_precise), so that results stay within 1e-5 of a double-precision evaluation of the
// section 2.1 equation.
//
//   v_mfma_f32_32x32x2_f32  D[32x32] += A[32x2] * B[2x32]   (lane l: n = l%32, hh = l/32)
//     A: lane holds row n, k = hh      B: lane holds column n, k = hh
//     D: lane holds column n, rows 8*(r/4) + 4*hh + r%4   for r = 0..15
//
// What bounds it: the fp32 matrix rate (64 flops per cycle and SIMD, a sixteenth of the bf16 rate;
// 153 TFLOP/s in a large matrix product on this card), and on small problems the longest chain of
// blocks one wave works through: a 32x32 block of pairs at d = 64 is 4096 cycles of matrix
// instructions forward, so a 512-row sequence taken by one wave per 32 rows would last 30 us.
// Hence the split: a workgroup owns 32 rows and its four waves take every fourth 32-row block of
// the streamed side, each on its own (wave-private LDS buffers, no barrier inside the loop), and
// add their accumulators up through LDS at the end.  LDS and L2 traffic is no concern at this
// matrix rate: an operand read of 16 bytes per lane feeds four matrix instructions (256 cycles).
// Each streamed tensor has one buffer per wave, refilled by an asynchronous copy as soon as the
// block's last product that reads it has been issued; the products of the other tensor cover it.
// Measured against the vector-ALU kernels before it (four lanes per row, key by key, one LDS read
// per fused multiply-add): 16 sequences of 64..512 rows, H = 4, d = 64: forward 225 -> 21 us, dk/dv
// 281 -> 35, dq 269 -> 29; 4 sequences of 1..64 rows, H = 2, d = 32: 22 -> 5.3, 27 -> 6.6, 25 -> 6.1 us.
#include "hstu_mfma.h"

namespace hstu {

namespace {

constexpr int TILE = 32;     // owner rows per workgroup
constexpr int FW = 4;        // waves per workgroup
constexpr int THREADS = FW * 64;
constexpr int FB = 32;       // streamed rows per block

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Swizzle of a row's 16-byte chunks (see swz_rb): 16 consecutive rows at one logical chunk land on
// 16 different positions of the 64 banks, and so do rows r and r + 4 at the eight chunks of 32
// consecutive columns (what a transposed operand read touches), except at D = 32.
template <int D>
__device__ __forceinline__ int fswz(int row) {
  if (D == 32) return (row >> 1) & 7;  // two rows per 256 bytes
  return (row & 3) | (((row >> 3) & 1) << 2) | (((row >> 2) & 1) << 3);
}

// Waits until at most N of the wave's vector memory operations are in flight.
template <int N>
__device__ __forceinline__ void vm_wait() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Rows of so many elements (a tensor's heads together) are further apart than 32-bit offsets inside a block of
// rows reach: the kernels have a variant for those (WIDE) that keeps its offsets inside one load's rows.
// (One form for both costs the others 1 to 8 %, in scalar instructions and registers.)
constexpr int64_t WIDE_ROW = 1 << 25;

// A wave's copy of one block: FB rows of one head, D / 8 wave-wide loads; rows >= valid are zeros.
template <int D>
constexpr int block_loads() { return D / 8; }
template <int D, bool WIDE>
__device__ __forceinline__ void block_copy(float* buf, const float* base, int64_t row_stride, int valid, int lane) {
  constexpr int CPR = D / 4, RPL = 64 / CPR, SPAN = WIDE ? RPL : FB;  // rows per buffer
  const int rows = valid < 0 ? 0 : (valid < FB ? valid : FB), rs = (int)row_stride * 4;
  __amdgpu_buffer_rsrc_t rsrc;
#pragma unroll
  for (int i = 0; i < block_loads<D>(); ++i) {
    if (WIDE || i == 0) {
      const int left = rows - i * RPL;
      rsrc = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(base + i * RPL * row_stride), 0,
          __builtin_amdgcn_readfirstlane((left < 0 ? 0 : (left < SPAN ? left : SPAN)) * rs), 0x00020000);
    }
    const int row = i * RPL + lane / CPR;
    const int chunk = (lane % CPR) ^ fswz<D>(row);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, HSTU_LDS(void, buf + i * 256), 16,
                                             (WIDE ? lane / CPR : row) * rs + chunk * 16, 0, 0, 0);
  }
}

// Owner rows as B operands: lane (n, hh) holds elements 8*t + 4*hh + {0..3} of row n.
template <int D, bool WIDE>
__device__ __forceinline__ void load_rows(f4 (&reg)[D / 8], const float* base, int64_t row_stride, int row, int nrows, int hh) {
  if constexpr (WIDE) {
    const f4* src = (const f4*)(base + (int64_t)(row < nrows ? row : 0) * row_stride + hh * 4);
#pragma unroll
    for (int t = 0; t < D / 8; ++t) {
      const f4 x = src[2 * t];
#pragma unroll
      for (int e = 0; e < 4; ++e) reg[t][e] = row < nrows ? x[e] : 0.f;
    }
  } else {
    const int rs = (int)row_stride * 4;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)base, 0, __builtin_amdgcn_readfirstlane(nrows * rs), 0x00020000);
#pragma unroll
    for (int t = 0; t < D / 8; ++t)
      reg[t] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, row * rs + t * 32 + hh * 16, 0, 0));
  }
}

__device__ __forceinline__ void clear(f32x16& x) {
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = 0.f;
}

// acc[streamed row][owner row] += block (rows of the block) x owners^T.  At D = 128 in two chains of half the
// elements each: a sum's rounding error grows with its chain (outputs off 64 bits by 2.70e-7 of their norm in one
// chain, 2.14e-7 in two, where one key after the other on the vector pipe had been off by 2.42e-7; 1.5 % slower.
// At 64 and 32 one chain is within 2.4e-7, and at 32 a second one takes dk/dv from three waves per SIMD to two).
template <int D>
__device__ __forceinline__ void scores(f32x16& acc, const float* buf, const f4 (&own)[D / 8], int n, int hh) {
  const int s = fswz<D>(n);
  f32x16 odd;
  clear(odd);
#pragma unroll
  for (int t = 0; t < D / 8; ++t) {
    const f4 x = *HSTU_LDS(const f4, buf + n * D + (((2 * t + hh) ^ s) << 2));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (D == 128 && (t & 1)) odd = mfma_f32(x[e], own[t][e], odd);
      else acc = mfma_f32(x[e], own[t][e], acc);
    }
  }
  if constexpr (D == 128)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] += odd[r];
}

// acc[column][owner row] += block^T x w, w[r] belonging to streamed row 8*(r/4) + 4*hh + r%4: the
// accumulator layout of scores() is the B operand of this product as it stands.
template <int D>
__device__ __forceinline__ void contract(f32x16 (&acc)[D / 32], const float* buf, const float (&w)[16], int n, int hh) {
  __builtin_amdgcn_sched_barrier(0);  // (operand reads hoisted further up would only take registers)
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r >> 2) + 4 * hh + (r & 3);
    const float* p = buf + row * D;
    const int s = fswz<D>(row);
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
      const float x = *HSTU_LDS(const float, p + (((c * 8 + (n >> 2)) ^ s) << 2) + (n & 3));
      acc[c] = mfma_f32(x, w[r], acc[c]);
    }
  }
}

// Adds up the four waves' accumulators through LDS (buf: the waves' FB x D blocks, no longer
// needed) and stores the 32 owner rows.  All threads of the workgroup call it.
template <int D>
__device__ __forceinline__ void sum_and_store(float* buf, const f32x16 (&acc)[D / 32], float* out, int64_t elem0,
                                              int64_t row_stride, int nrows, float scale, int accumulate, int wave,
                                              int lane) {
  float* mine = buf + wave * (FB * D);
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f4 x = {acc[c][4 * q], acc[c][4 * q + 1], acc[c][4 * q + 2], acc[c][4 * q + 3]};
      *HSTU_LDS(f4, mine + ((c * 4 + q) * 64 + lane) * 4) = x;
    }
  __syncthreads();
  const int n = lane & 31, hh = lane >> 5;
#pragma unroll
  for (int i = 0; i < D / 32; ++i) {
    const int g = i * FW + wave;  // group c * 4 + q of the accumulators
    f4 x = *HSTU_LDS(const f4, buf + (g * 64 + lane) * 4);
#pragma unroll
    for (int w = 1; w < FW; ++w) x += *HSTU_LDS(const f4, buf + w * (FB * D) + (g * 64 + lane) * 4);
    x *= scale;
    if (n < nrows) {
      f4* dst = (f4*)(out + elem0 + (int64_t)n * row_stride + g * 8 + hh * 4);
      if (accumulate) x += *dst;
      *dst = x;
    }
  }
}

// sigmoid(x) to about an ulp, from z = e^-|x| <= 1, which overflows nowhere: 1 / (1 + z) for x >= 0,
// z / (1 + z) below, and 1 - sigmoid(x) the other way round (subtracted, it would have no digits left where
// the sigmoid saturates, and the derivative multiplies it by x).  z as 2^t with t = -|x| * log2(e) rounded and the product's rounding error carried as a
// first-order factor (1 + ln2 * error), so that a large |x| costs no accuracy; the reciprocal with one
// Newton step.  |x| is cut at 104, where z is exactly zero: the sigmoid of anything beyond, infinities
// included, is exactly 0 or 1 (an |x| that were not cut would make the error term infinite times zero, a
// z that were kept above zero would let x * sigmoid(x) grow with -x).  NaN stays NaN in x * sigmoid(x).
// Fifteen vector instructions against 27 for expf and an IEEE division.
struct Sigmoid {
  float sg, rest;  // sigmoid(x), 1 - sigmoid(x)
};
__device__ __forceinline__ Sigmoid sigmoid_precise(float x) {
  constexpr float LOG2E = 1.44269504088896341f, LOG2E_LO = 1.92596299e-8f, LN2 = 0.693147180559945309f;
  const float y = -__builtin_fminf(__builtin_fabsf(x), 104.0f);
  const float t = y * LOG2E;
  const float err = __builtin_fmaf(y, LOG2E_LO, __builtin_fmaf(y, LOG2E, -t));
  const float e = __builtin_amdgcn_exp2f(t);
  const float z = __builtin_fmaf(e, err * LN2, e);
  const float d = 1.0f + z;
  const float r = __builtin_amdgcn_rcpf(d);
  const float s = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
  const bool below = x < 0.0f;
  return Sigmoid{below ? z * s : s, below ? s : z * s};
}
// silu'(x) = sg * (1 + x * (1 - sg))
__device__ __forceinline__ float silu_slope(float x, const Sigmoid& g) { return g.sg * __builtin_fmaf(x, g.rest, 1.0f); }

// The streamed blocks of an item: [first, end) of Stream's 32-row blocks, without the leading block
// wholly before the owners and the trailing one without rows; wave w takes first + w, + FW, ...
struct Blocks {
  Stream st;
  int first, end;
};
template <int SIDE>
__device__ __forceinline__ Blocks make_blocks(const Item& it, int causal) {
  Blocks b;
  b.st = make_stream<SIDE>(it, causal);
  b.first = 0;
  b.end = 2 * b.st.total;
  if (b.end > 0) {
    if (tile_ref(it, b.st, b.st.total - 1).valid <= FB) --b.end;
    if (SIDE == 1 && causal && tile_ref(it, b.st, 0).pos + FB <= it.pos0) b.first = 1;
  }
  return b;
}
struct BlockRef { int row, valid, pos; };
__device__ __forceinline__ BlockRef block_ref(const Item& it, const Blocks& b, int i) {
  if (i >= b.end) return BlockRef{0, 0, 0};
  const TileRef t = tile_ref(it, b.st, i >> 1);
  const int o = (i & 1) * FB;
  return BlockRef{t.row + o, t.valid - o, t.pos + o};
}

// Timestamp bias of the lane's 16 pairs (see bias_bucket): adds the table entries to the scores and
// keeps the buckets.  Streamed rows beyond the block's valid ones take the last valid row's
// timestamp: their products are zero whatever the score.  (The records are padded by 64 rows.)
__device__ __forceinline__ void add_bias(f32x16& s, int (&bk)[16], const AttnArgs& a, int t_own, const BlockRef& b, int hh) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    int row = 8 * (r >> 2) + 4 * hh + (r & 3);
    row = row < b.valid ? row : (b.valid > 0 ? b.valid - 1 : 0);
    bk[r] = bias_bucket(abs_diff(t_own, a.ts_rec[(int64_t)b.row + row].ts), a.nb, a.fbits);
    s[r] += a.ts_w[bk[r]];
  }
}

// The head and the 32 rows of an item (AttnArgs::item_parts; grid.y counts them) that are (item, head) pair `unit`.
// False: no owner rows.
__device__ __forceinline__ bool half_item(const AttnArgs& a, int unit, Item& it, int& h) {
  const int skip = blockIdx.y * TILE;
  h = unit % a.num_heads;
  if (!get_item(a, unit / a.num_heads, it)) return false;
  it.row0 += skip;
  it.pos0 += skip;
  it.nrows -= skip;
  if (it.nrows > TILE) it.nrows = TILE;
  return it.nrows > 0;
}

// Waves per SIMD the kernels are built for: what the LDS of a workgroup leaves room for.
constexpr int f32_waves(int dqk, int dv, bool one = false) { return dqk + dv <= 128 && !one ? 2 : 1; }
// The dq pass at d_qk = d_v = 32 without bias: four, in 128 registers (with the 130 it takes if it may, 4000
// sequences of 1..60 rows, H = 2: 80 -> 94 us).
constexpr int f32_dq_waves(int dqk, int dv, bool bias) { return dqk + dv <= 64 && !bias ? 4 : f32_waves(dqk, dv); }

// The dk/dv pass with the bias: one, except at d_qk + d_v = 96, where it fits two if it must and a few registers more keep one
// workgroup on a CU if it need not (24 sequences of 64..512 rows, H = 2, fwd + bwd, d_qk = 64 123 -> 118 us, 32 110 -> 102;
// at d_qk = d_v = 32 the bound makes the pass slower, 91 -> 96).
constexpr int f32_dkdv_waves(int dqk, int dv, bool bias) { return dqk + dv == 96 ? 2 : f32_waves(dqk, dv, bias); }

// The masks' form: sums held in registers at d_qk + d_v <= 96 without the bias.  There the compiler needs fewer registers so
// in the d = 32 forward kernel (93 against 121, five workgroups a CU against four: 128 sequences of 64..512 rows, H = 4, 60.4
// -> 58.0 us; fwd + bwd of 64 128 -> 123, of 4 of 1000..3000, H = 2, 185 -> 171).  Beyond, and with the bias, they only
// take registers (d = 64 within 0.7 % either way; the bias's dk/dv kernel at d = 128 spills 13 with them and 3 without).
template <int DQK, int DV, bool BIAS>
constexpr bool f32_held = DQK + DV <= 96 && !BIAS;

struct Lane {
  int tid, lane, n, hh, wave;
  __device__ __forceinline__ Lane() {
    tid = threadIdx.x; lane = tid & 63; n = lane & 31; hh = lane >> 5;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  }
};

// ---------------------------------------------------------------------------------------------
template <int DQK, int DV, bool BIAS, bool WIDE>
__global__ void __launch_bounds__(THREADS, f32_waves(DQK, DV)) hstu_fwd_f32(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) float kbuf[FW * FB * DQK];
  __shared__ __attribute__((aligned(1024))) float vbuf[FW * FB * DV];
  const int H = a.num_heads;
  int h;
  Item it;
  if (!half_item(a, blockIdx.x, it, h)) return;
  const Lane l;
  const int64_t sq = (int64_t)H * DQK, sv = (int64_t)H * DV;
  const float* kg = (const float*)a.k + h * DQK;
  const float* vg = (const float*)a.v + h * DV;
  float* kb = kbuf + l.wave * (FB * DQK);
  float* vb = vbuf + l.wave * (FB * DV);
  f4 q[DQK / 8];
  load_rows<DQK, WIDE>(q, (const float*)a.q + (int64_t)it.row0 * sq + h * DQK, sq, l.n, it.nrows, l.hh);
  const Blocks bl = make_blocks<0>(it, a.causal);
  const int t_own = BIAS && l.n < it.nrows ? a.ts_rec_own[(int64_t)it.row0 + l.n].ts : 0;
  auto copy_k = [&](const BlockRef& b) { block_copy<DQK, WIDE>(kb, kg + (int64_t)b.row * sq, sq, b.valid, l.lane); };
  auto copy_v = [&](const BlockRef& b) { block_copy<DV, WIDE>(vb, vg + (int64_t)b.row * sv, sv, b.valid, l.lane); };
  f32x16 o[DV / 32];
#pragma unroll
  for (int c = 0; c < DV / 32; ++c) clear(o[c]);
  int i = bl.first + l.wave;
  BlockRef b = block_ref(it, bl, i);
  copy_k(b);
  copy_v(b);
  for (; i < bl.end; i += FW) {
    const BlockRef nx = block_ref(it, bl, i + FW);
    f32x16 s;
    clear(s);
    vm_wait<block_loads<DV>()>();
    scores<DQK>(s, kb, q, l.n, l.hh);
    lds_reads_done();
    copy_k(nx);
    if constexpr (BIAS) {
      int bk[16];
      add_bias(s, bk, a, t_own, b, l.hh);
    }
    float p[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = a.alpha * s[r];
      p[r] = x * sigmoid_precise(x).sg;
    }
    if (a.causal && b.pos + FB - 1 > it.pos0) {
      const std::conditional_t<f32_held<DQK, DV, BIAS>, VisBeforeHeld, VisBefore> vis{it.pos0 + l.n - b.pos, l.hh};
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = vis(r) ? p[r] : 0.f;
    }
    vm_wait<block_loads<DQK>()>();
    contract<DV>(o, vb, p, l.n, l.hh);
    lds_reads_done();
    copy_v(nx);
    b = nx;
  }
  vm_wait<0>();
  sum_and_store<DV>(vbuf, o, (float*)a.o, (int64_t)it.row0 * sv + h * DV, sv, it.nrows, a.inv_n, a.accumulate, l.wave,
                    l.lane);
}

// ---------------------------------------------------------------------------------------------
// qbuf, gbuf: FW blocks of DQK and of DV columns (LDS).
template <int DQK, int DV, bool BIAS, bool WIDE>
__device__ __forceinline__ void dkdv_unit(const AttnArgs& a, int unit, float* qbuf, float* gbuf) {
  const int H = a.num_heads;
  int h;
  Item it;
  if (!half_item(a, unit, it, h)) return;
  const Lane l;
  const int64_t sq = (int64_t)H * DQK, sv = (int64_t)H * DV;
  const float* qg = (const float*)a.q + h * DQK;
  const float* gg = (const float*)a.d_o + h * DV;
  float* qb = qbuf + l.wave * (FB * DQK);
  float* gb = gbuf + l.wave * (FB * DV);
  f4 k[DQK / 8], v[DV / 8];
  load_rows<DQK, WIDE>(k, (const float*)a.k + (int64_t)it.row0 * sq + h * DQK, sq, l.n, it.nrows, l.hh);
  load_rows<DV, WIDE>(v, (const float*)a.v + (int64_t)it.row0 * sv + h * DV, sv, l.n, it.nrows, l.hh);
  const Blocks bl = make_blocks<1>(it, a.causal);
  const int t_own = BIAS && l.n < it.nrows ? a.ts_rec_own[(int64_t)it.row0 + l.n].ts : 0;
  auto copy_q = [&](const BlockRef& b) { block_copy<DQK, WIDE>(qb, qg + (int64_t)b.row * sq, sq, b.valid, l.lane); };
  auto copy_g = [&](const BlockRef& b) { block_copy<DV, WIDE>(gb, gg + (int64_t)b.row * sv, sv, b.valid, l.lane); };
  f32x16 dk[DQK / 32], dv[DV / 32];
#pragma unroll
  for (int c = 0; c < DQK / 32; ++c) clear(dk[c]);
#pragma unroll
  for (int c = 0; c < DV / 32; ++c) clear(dv[c]);
  int i = bl.first + l.wave;
  BlockRef b = block_ref(it, bl, i);
  copy_g(b);
  copy_q(b);
  for (; i < bl.end; i += FW) {
    const BlockRef nx = block_ref(it, bl, i + FW);
    f32x16 s, dp;
    clear(s); clear(dp);
    vm_wait<block_loads<DQK>()>();
    scores<DV>(dp, gb, v, l.n, l.hh);
    vm_wait<0>();
    scores<DQK>(s, qb, k, l.n, l.hh);
    if constexpr (BIAS) {
      int bk[16];
      add_bias(s, bk, a, t_own, b, l.hh);
    }
    float p[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = a.alpha * s[r];
      const Sigmoid g = sigmoid_precise(x);
      p[r] = x * g.sg;
      ds[r] = dp[r] * silu_slope(x, g);
    }
    if (a.causal && b.pos < it.pos0 + TILE - 1) {
      const std::conditional_t<f32_held<DQK, DV, BIAS>, VisAfterHeld, VisAfter> vis{it.pos0 + l.n - b.pos, l.hh};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool on = vis(r);
        p[r] = on ? p[r] : 0.f;
        ds[r] = on ? ds[r] : 0.f;
      }
    }
    contract<DV>(dv, gb, p, l.n, l.hh);
    lds_reads_done();
    copy_g(nx);
    contract<DQK>(dk, qb, ds, l.n, l.hh);
    lds_reads_done();
    copy_q(nx);
    b = nx;
  }
  vm_wait<0>();
  sum_and_store<DV>(gbuf, dv, (float*)a.dv, (int64_t)it.row0 * sv + h * DV, sv, it.nrows, a.inv_n, a.accumulate, l.wave,
                    l.lane);
  sum_and_store<DQK>(qbuf, dk, (float*)a.dk, (int64_t)it.row0 * sq + h * DQK, sq, it.nrows, a.alpha * a.inv_n,
                     a.accumulate, l.wave, l.lane);
}

template <int DQK, int DV, bool BIAS, bool WIDE>
__global__ void __launch_bounds__(THREADS, f32_dkdv_waves(DQK, DV, BIAS)) hstu_dkdv_f32(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) float qbuf[FW * FB * DQK];
  __shared__ __attribute__((aligned(1024))) float gbuf[FW * FB * DV];
  dkdv_unit<DQK, DV, BIAS, WIDE>(a, blockIdx.x, qbuf, gbuf);
}

// ---------------------------------------------------------------------------------------------
// kbuf, vbuf: FW blocks of DQK and of DV columns; dwl: the workgroup's sums of dS per bucket (fixed point, BIAS only).
template <int DQK, int DV, bool BIAS, bool WIDE>
__device__ __forceinline__ void dq_unit(const AttnArgs& a, int unit, float* kbuf, float* vbuf, unsigned long long* dwl) {
  const int H = a.num_heads;
  int h;
  Item it;
  if (!half_item(a, unit, it, h)) return;
  const Lane l;
  if constexpr (BIAS) {
    for (int i = l.tid; i < a.nb; i += THREADS) dwl[i] = 0ull;
    __syncthreads();
  }
  const int64_t sq = (int64_t)H * DQK, sv = (int64_t)H * DV;
  const float* kg = (const float*)a.k + h * DQK;
  const float* vg = (const float*)a.v + h * DV;
  float* kb = kbuf + l.wave * (FB * DQK);
  float* vb = vbuf + l.wave * (FB * DV);
  f4 q[DQK / 8], g[DV / 8];
  load_rows<DQK, WIDE>(q, (const float*)a.q + (int64_t)it.row0 * sq + h * DQK, sq, l.n, it.nrows, l.hh);
  load_rows<DV, WIDE>(g, (const float*)a.d_o + (int64_t)it.row0 * sv + h * DV, sv, l.n, it.nrows, l.hh);
  const Blocks bl = make_blocks<0>(it, a.causal);
  const int t_own = BIAS && l.n < it.nrows ? a.ts_rec_own[(int64_t)it.row0 + l.n].ts : 0;
  auto copy_k = [&](const BlockRef& b) { block_copy<DQK, WIDE>(kb, kg + (int64_t)b.row * sq, sq, b.valid, l.lane); };
  auto copy_v = [&](const BlockRef& b) { block_copy<DV, WIDE>(vb, vg + (int64_t)b.row * sv, sv, b.valid, l.lane); };
  f32x16 dq[DQK / 32];
#pragma unroll
  for (int c = 0; c < DQK / 32; ++c) clear(dq[c]);
  int i = bl.first + l.wave;
  BlockRef b = block_ref(it, bl, i);
  copy_v(b);
  copy_k(b);
  for (; i < bl.end; i += FW) {
    const BlockRef nx = block_ref(it, bl, i + FW);
    f32x16 s, dp;
    clear(s); clear(dp);
    vm_wait<block_loads<DQK>()>();
    scores<DV>(dp, vb, g, l.n, l.hh);
    lds_reads_done();
    copy_v(nx);
    vm_wait<block_loads<DV>()>();
    scores<DQK>(s, kb, q, l.n, l.hh);
    int bk[16];
    if constexpr (BIAS) add_bias(s, bk, a, t_own, b, l.hh);
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = a.alpha * s[r];
      ds[r] = dp[r] * silu_slope(x, sigmoid_precise(x));
    }
    if (a.causal && b.pos + FB - 1 > it.pos0) {
      const std::conditional_t<f32_held<DQK, DV, BIAS>, VisBeforeHeld, VisBefore> vis{it.pos0 + l.n - b.pos, l.hh};
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = vis(r) ? ds[r] : 0.f;
    }
    if constexpr (BIAS)  // (pairs beyond the owner or streamed rows have dS = 0)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (ds[r] != 0.f) atomicAdd(dwl + bk[r], dw_to_fixed(ds[r]));
    contract<DQK>(dq, kb, ds, l.n, l.hh);
    lds_reads_done();
    copy_k(nx);
    b = nx;
  }
  vm_wait<0>();
  sum_and_store<DQK>(kbuf, dq, (float*)a.dq, (int64_t)it.row0 * sq + h * DQK, sq, it.nrows, a.alpha * a.inv_n,
                     a.accumulate, l.wave, l.lane);
  if constexpr (BIAS)  // (ordered by the barrier in sum_and_store)
    for (int j = l.tid; j < a.nb; j += THREADS)
      if (dwl[j] != 0ull) atomicAdd(a.d_ts_acc + j, dw_from_fixed(dwl[j]));
}

template <int DQK, int DV, bool BIAS, bool WIDE>
__global__ void __launch_bounds__(THREADS, f32_dq_waves(DQK, DV, BIAS)) hstu_dq_f32(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) float kbuf[FW * FB * DQK];
  __shared__ __attribute__((aligned(1024))) float vbuf[FW * FB * DV];
  __shared__ unsigned long long dwl[BIAS ? MAX_TS_BUCKETS : 1];
  dq_unit<DQK, DV, BIAS, WIDE>(a, blockIdx.x, kbuf, vbuf, dwl);
}

// Both backward passes in one launch, for calls whose workgroups are a few rounds at most: the passes do not depend
// on each other, and each by itself lasts as long as its longest items while other CUs idle, and as a launch.  Groups of
// eight workgroups (one per XCD) alternate between the passes, so that both lists run heaviest first.
template <int D>
__global__ void __launch_bounds__(THREADS, f32_waves(D, D)) hstu_bwd_f32(AttnArgs k, AttnArgs q) {
  __shared__ __attribute__((aligned(1024))) float buf0[FW * FB * D];
  __shared__ __attribute__((aligned(1024))) float buf1[FW * FB * D];
  const int unit = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7);
  if (blockIdx.x & 8) {
    if (unit < q.max_items * q.num_heads) dq_unit<D, D, false, false>(q, unit, buf0, buf1, nullptr);
  } else {
    if (unit < k.max_items * k.num_heads) dkdv_unit<D, D, false, false>(k, unit, buf0, buf1);
  }
}

}  // namespace

int tile_rows_f32(int /*pass*/) { return TILE; }

#define HSTU_LAUNCH_F32(KERNEL, A, B)                                                      \
  do {                                                                                     \
    const bool wide = (int64_t)a.num_heads * (A > B ? A : B) >= WIDE_ROW;                  \
    if (a.ts_rec && wide) hipLaunchKernelGGL((KERNEL<A, B, true, true>), grid, block, 0, stream, a);   \
    else if (a.ts_rec) hipLaunchKernelGGL((KERNEL<A, B, true, false>), grid, block, 0, stream, a);     \
    else if (wide) hipLaunchKernelGGL((KERNEL<A, B, false, true>), grid, block, 0, stream, a);         \
    else hipLaunchKernelGGL((KERNEL<A, B, false, false>), grid, block, 0, stream, a);      \
  } while (0)
#define HSTU_DISPATCH_F32(KERNEL)                                                          \
  do {                                                                                     \
    const dim3 grid((unsigned)((int64_t)a.max_items * a.num_heads), (unsigned)a.item_parts), block(THREADS); \
    if (d_qk == 128 && d_v == 128) HSTU_LAUNCH_F32(KERNEL, 128, 128);                      \
    else if (d_qk == 64 && d_v == 64) HSTU_LAUNCH_F32(KERNEL, 64, 64);                     \
    else if (d_qk == 32 && d_v == 32) HSTU_LAUNCH_F32(KERNEL, 32, 32);                     \
    else if (d_qk == 128 && d_v == 64) HSTU_LAUNCH_F32(KERNEL, 128, 64);                   \
    else if (d_qk == 64 && d_v == 128) HSTU_LAUNCH_F32(KERNEL, 64, 128);                   \
    else if (d_qk == 128 && d_v == 32) HSTU_LAUNCH_F32(KERNEL, 128, 32);                   \
    else if (d_qk == 32 && d_v == 128) HSTU_LAUNCH_F32(KERNEL, 32, 128);                   \
    else if (d_qk == 64 && d_v == 32) HSTU_LAUNCH_F32(KERNEL, 64, 32);                     \
    else if (d_qk == 32 && d_v == 64) HSTU_LAUNCH_F32(KERNEL, 32, 64);                     \
    else return hipErrorInvalidValue;                                                      \
    return hipGetLastError();                                                              \
  } while (0)

hipError_t launch_fwd_f32(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  HSTU_DISPATCH_F32(hstu_fwd_f32);
}
hipError_t launch_dkdv_f32(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  HSTU_DISPATCH_F32(hstu_dkdv_f32);
}
// Where the two passes in one launch are the faster form: up to three rounds of the two workgroups a CU holds, and at d =
// 128, where it holds one, while the workgroups of both passes are resident at once.  (Beyond, the register allocation of
// the larger pass costs the other one more than the shared tail gives.)  Measured, two launches -> one (workgroups
// per pass), H = 2 and 4: d = 32 4 sequences of 1..64 rows (20) 20.1 -> 15.6 us, 16 of 64..512 (656) 48.8 -> 39.6, 64 of
// 32..256 (1384) 48.8 -> 46.0, 64 of 64..512 (2508) 102 -> 101, 128 (5232) 182 -> 188; d = 64 22.6 -> 16.0, 68.8 ->
// 63.7, 80.1 -> 77.5, 172 -> 180, 339 -> 352, 8 of 500..1024 (420) 102 -> 76; d = 128 (20) 35.6 -> 20.9, (420) 155 ->
// 162, (656) 130 -> 134.
// At d = 64 sequences of more than 1024 rows (max_len) only up to 600 workgroups a pass: their items are long beside the
// tail that the passes share.  4 sequences of 1000..3000 rows (520) 261 -> 214 us and (1050) 374 -> 394, 4 of 2000..5000 (440)
// 404 -> 295 and (880) 530 -> 568, 3 of 3000..8000 (520) 577 -> 459 and (1040) 814 -> 870; 8 of 500..1024 (780) 130 -> 126.  (At d =
// 32 such calls gain up to the limit: 226 -> 217, 342 -> 310, 503 -> 481.)
bool bwd_f32_supported(const AttnArgs& k, const AttnArgs& q, int d_qk, int d_v, int max_len) {
  const int64_t most = k.max_items > q.max_items ? k.max_items : q.max_items;
  return d_qk == d_v && !k.ts_rec && !q.ts_rec && (int64_t)k.num_heads * d_qk < WIDE_ROW &&
         most * k.num_heads * k.item_parts <= (d_qk == 128 ? 128 : d_qk == 64 && max_len > 1024 ? 600 : 1536);
}
hipError_t launch_bwd_f32(const AttnArgs& k, const AttnArgs& q, int d_qk, int d_v, int max_len, hipStream_t stream) {
  if (!bwd_f32_supported(k, q, d_qk, d_v, max_len)) return hipErrorInvalidValue;
  const int64_t most = (k.max_items > q.max_items ? k.max_items : q.max_items) * (int64_t)k.num_heads;
  const dim3 grid((unsigned)((most + 7) / 8 * 16), (unsigned)k.item_parts), block(THREADS);
  if (d_qk == 128) hipLaunchKernelGGL((hstu_bwd_f32<128>), grid, block, 0, stream, k, q);
  else if (d_qk == 64) hipLaunchKernelGGL((hstu_bwd_f32<64>), grid, block, 0, stream, k, q);
  else hipLaunchKernelGGL((hstu_bwd_f32<32>), grid, block, 0, stream, k, q);
  return hipGetLastError();
}
hipError_t launch_dq_f32(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream) {
  if (a.ts_rec && !a.d_ts_acc) return hipErrorInvalidValue;
  HSTU_DISPATCH_F32(hstu_dq_f32);
}

}  // namespace hstu
