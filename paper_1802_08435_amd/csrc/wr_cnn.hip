// The masked dilated 1-D CNN that conditions the Subscale WaveRNN (Sec. 4.1,
// Sec. 5): for every utterance u, sub-tensor s and row (block of B samples)
// k, a Dx-wide conditioning vector computed from the previous sub-tensors'
// samples of rows k .. k + 124 (the mask keeps the future taps only).
//
// All rows of all sub-tensors are computed at once: every layer is one GEMM of
// M = utterances x B x rows activation rows against a weight matrix on the
// matrix cores (v_mfma_f32_16x16x32_bf16).  Weights are bf16; activations are
// split into a bf16 high part and a bf16 remainder by the kernel that makes
// them (two products per weight, about 16 significant bits; the residual is
// also kept in fp32), so the layers keep fp32-level accuracy.  A dilated convolution layer reads its
// three taps (rows k, k + d, k + 2d of the same sub-tensor, zero past the
// utterance's last row, as the mask of an utterance-long network has it)
// straight from the previous layer's rows, without an unfolded copy.  The
// network can also run over windows of rows (sampling runs it ahead in
// chunks): taps past a window are zero too, which changes only rows whose
// reach leaves the window.  Layer by layer:
//   input   r = Win x + bin         K = 2B (padded to 32)  N = Rc
//   conv l  a = relu(Wc [r_k | r_k+d | r_k+2d] + bc)  K = 3 Rc  N = Cc
//   proj l  r = r + (Wo a + bo)     K = Cc                 N = Rc
//   output  o = Wp r + bp           K = Rc                 N = Dx
#include "wr_kern.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Streamed runs: the sub-tensor and the utterance row of run row m (see CnnGemmArgs).
__device__ __forceinline__ int cnn_rng_row(const CnnGemmArgs& a, int m, int* s, int* blk) {
  const int b = m / a.rows;
  *s = a.out_s0 + b % a.B;
  *blk = (b / a.B) * a.out_B + *s;                  // (utterance, sub-tensor) of the whole-utterance arrays
  return a.lo[*s] + m % a.rows;
}

// Source row of run row m for a tap (-1: read as zero).
__device__ __forceinline__ int64_t cnn_src_row(const CnnGemmArgs& a, int m, int tap) {
  if (m >= a.M) return -1;
  if (a.rng) {
    int s = 0, blk = 0;
    const int q = cnn_rng_row(a, m, &s, &blk) + tap * a.dil;   // the tap's utterance row
    if (q >= a.rows_utt) return -1;
    return a.src_abs ? (int64_t)blk * a.rows_utt + q : m;
  }
  const int kb = m % a.rows + tap * a.dil;           // row within the block of the tap
  const int64_t q = a.row0 + (int64_t)((m / a.rows) % a.B) * a.row_step + kb;   // its utterance row
  return kb < a.rows && q < a.rows_utt ? (int64_t)m + tap * a.dil : -1;
}

// Destination row of run row m (-1: not stored).
__device__ __forceinline__ int64_t cnn_dst_row(const CnnGemmArgs& a, int m) {
  if (m >= a.M) return -1;
  if (a.rng) {
    int s, b2;
    const int q = cnn_rng_row(a, m, &s, &b2);
    if (q >= a.hi[s]) return -1;                     // not a row of this run
    return a.dst_abs ? (int64_t)b2 * a.rows_utt + q : m;
  }
  const int blk = m / a.rows;
  return (int64_t)((blk / a.B) * a.out_B + a.out_s0 + blk % a.B) * a.rows + m % a.rows;
}

__device__ __forceinline__ uint16_t cnn_hi(float v) { return (uint16_t)(__float_as_uint(v) >> 16); }
__device__ __forceinline__ uint16_t cnn_lo(float v) {
  return __builtin_bit_cast(uint16_t, (__bf16)(v - __uint_as_float(__float_as_uint(v) & 0xffff0000u)));
}
// Column c of split row m.
__device__ __forceinline__ void cnn_split_put(uint16_t* x, int64_t m, int K, int c, float v) {
  uint16_t* p = x + m * 2 * K + (c >> 5) * 64 + (c & 31);
  p[0] = cnn_hi(v);
  p[32] = cnn_lo(v);
}

}  // namespace

// Tiles of 32 MI rows x 128 columns on 4 waves (2 x 2 of 16 MI x 64), two
// workgroups a CU.  Both operands are staged in LDS by 16-byte copies, a K-step
// double-buffered there and two more on their way in registers: what bounds a
// tile is the latency of its first touch of memory (each kernel starts with
// cold L2s, about 0.9 us a load) and then, at MI = 4, LDS (1,152 clocks a
// K-step and CU against 1,024 of products).  Rows of activations come whole
// (8 lanes a 128-byte line of a split row).  The first version converted fp32
// rows again for every tap and column tile, had one K-step on its way and read
// the residual's old values one by one between the epilogue's stores.  24,000
// rows at the paper's widths (22 GEMMs): 2.73 -> 1.65-1.95 ms over the devices
// measured (350 to 296 TFLOP/s; twice that issued, high and low part); a sampling chunk's
// GEMM of 700 rows: 12.8 -> 11.5 us, its 10 projections without a reduction.
//
// Workgroup b takes work item L = (b % 8) per_xcd + b / 8 (tile L mod tiles,
// group L / tiles when split): consecutive tiles (the column tiles of one row
// tile, which read the same activations) share an XCD and its L2.  The K loop
// sums in groups of `group` K-steps, each group from zero, added in order: the
// same arithmetic whether one workgroup runs every group or, where a GEMM has
// fewer tiles than the card has room for, each group runs on its own workgroup
// and wr_cnn_reduce adds them, so results never depend on how many rows a run
// has, nor on MI.
template <int MI>
__global__ __launch_bounds__(CNN_THREADS, 2) void wr_cnn_gemm(CnnGemmArgs a) {
  constexpr int TM = 32 * MI, ABUF = 4 * MI * WR_FRAGP, BUF = ABUF + 8 * WR_FRAG;
  __shared__ __align__(16) unsigned char lds[2 * BUF];   // [2]: A [row tile 2 MI][high, low], W [column tile 8]
  __shared__ int64_t drow[TM], srows[3 * TM];       // destination rows, source rows of each tap (-1: none)
  const int b = blockIdx.x;
  const int L = (b % 8) * a.per_xcd + b / 8;
  if (b / 8 >= a.per_xcd || L >= a.tiles * a.split) return;
  const int tile = L % a.tiles, q = L / a.tiles, nt = a.N / CNN_TN;
  const int m0 = tile / nt * TM, n0 = tile % nt * CNN_TN;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, wm = wave >> 1, wn = wave & 1;
  if (tid < TM) drow[tid] = a.split > 1 ? (m0 + tid < a.M ? m0 + tid : -1) : cnn_dst_row(a, m0 + tid);
  for (int i = tid; i < a.taps * TM; i += CNN_THREADS) srows[i] = cnn_src_row(a, m0 + i % TM, i / TM);
  __syncthreads();
  f32x4 acc[MI][4], grp[MI][4];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = grp[i][j] = f32x4{0, 0, 0, 0};
  const int KT = a.K / 32, kc = a.kin / 32;
  const int k_lo = a.split > 1 ? q * a.group : 0, k_hi = a.split > 1 ? min(KT, k_lo + a.group) : KT;
  // staging: 8 lanes copy one row's line (4 octets high, 4 low), a wave rows 8 (wave + 4 i) .. + 7
  const int srow = 8 * wave + (lane >> 3), piece = lane & 7;
  unsigned char* sdst = lds + ((srow >> 4) * 2 + (piece >> 2)) * WR_FRAGP + (piece & 3) * WR_KGP + (srow & 15) * 16;
  const uint16_t* p[MI];
  int step[MI];
  int tap = k_lo / kc, col = k_lo % kc;              // of the next K-step to load
  auto rows = [&]() {                                // row pointers of tap `tap` at column group `col`
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int64_t r = srows[tap * TM + srow + 32 * i];
      p[i] = (r >= 0 ? a.src + (r * kc + col) * 64 : a.zero) + 8 * piece;
      step[i] = r >= 0 ? 64 : 0;
    }
  };
  rows();
  // W: this wave copies column tiles wave and wave + 4
  const u32x4* wp = (const u32x4*)a.w + ((size_t)(n0 / 16 + wave) * KT + k_lo) * 64 + lane;
  unsigned char* wdst = lds + ABUF + wave * WR_FRAG + lane * 16;
  struct Stage {                                     // a K-step on its way
    u32x4 x[MI], w[2];
  };
  auto load = [&](Stage& g) {
#pragma unroll
    for (int i = 0; i < MI; ++i) g.x[i] = *(const u32x4*)p[i];
    g.w[0] = wp[0];
    g.w[1] = wp[(size_t)4 * KT * 64];
    wp += 64;
    if (++col == kc) {
      col = 0;
      if (++tap < a.taps) rows();
    } else {
#pragma unroll
      for (int i = 0; i < MI; ++i) p[i] += step[i];
    }
  };
  int left = a.group;                                // K-steps left of the group
  bool first = true;
  auto k_step = [&](int kt, Stage& g, int s) {       // s: the LDS buffer
#pragma unroll
    for (int i = 0; i < MI; ++i) *(u32x4*)(sdst + s * BUF + 4 * i * WR_FRAGP) = g.x[i];
    *(u32x4*)(wdst + s * BUF) = g.w[0];
    *(u32x4*)(wdst + s * BUF + 4 * WR_FRAG) = g.w[1];
    __syncthreads();
    if (kt + 2 < k_hi) load(g);                      // in flight for two K-steps
    const unsigned char* buf = lds + s * BUF;
    bf16x8 bw[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bw[j] = *(const bf16x8*)(buf + ABUF + (4 * wn + j) * WR_FRAG + lane * 16);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const bf16x8 ah = afrag_p(buf, 2 * (MI * wm + i)), al = afrag_p(buf, 2 * (MI * wm + i) + 1);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        grp[i][j] = mfma(ah, bw[j], grp[i][j]);
        grp[i][j] = mfma(al, bw[j], grp[i][j]);
      }
    }
    if (--left == 0 || kt + 1 == k_hi) {             // a group ends: acc = acc + g (the first: acc = g)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[i][j] = first ? grp[i][j] : acc[i][j] + grp[i][j];
          grp[i][j] = f32x4{0, 0, 0, 0};
        }
      left = a.group;
      first = false;
    }
  };
  Stage g0, g1;
  load(g0);
  if (k_lo + 1 < k_hi) load(g1);
  for (int kt = k_lo; kt < k_hi; kt += 2) {
    k_step(kt, g0, 0);
    if (kt + 1 < k_hi) k_step(kt + 1, g1, 1);
  }
  // lane l of tile (i, j) holds rows 4 (l / 16) .. +3, column l % 16.  The
  // residual's old values are all read before the first is replaced: read one by
  // one between the stores, each waited for memory on its own.
  float* part = a.split > 1 ? a.part + (size_t)q * a.M * a.N : nullptr;
  const int nc = n0 + 64 * wn + (lane & 15);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    int64_t dm[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) dm[r] = drow[16 * (MI * wm + i) + 4 * (lane >> 4) + r];
    if (part) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (dm[r] >= 0)
#pragma unroll
          for (int j = 0; j < 4; ++j) part[(size_t)dm[r] * a.N + nc + 16 * j] = acc[i][j][r];
      continue;
    }
    f32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = acc[i][j] + a.bias[nc + 16 * j];
    if (a.epi == 2) {
      f32x4 o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j][r] = a.dst[(size_t)(dm[r] >= 0 ? dm[r] : 0) * a.N + nc + 16 * j];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = o[j] + v[j];
    } else if (a.epi == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[j][r] = wr_relu(v[j][r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (dm[r] < 0) continue;
      if (a.dst)
#pragma unroll
        for (int j = 0; j < 4; ++j) a.dst[(size_t)dm[r] * a.N + nc + 16 * j] = v[j][r];
      if (a.dsts)
#pragma unroll
        for (int j = 0; j < 4; ++j) cnn_split_put(a.dsts, dm[r], a.N, nc + 16 * j, v[j][r]);
    }
  }
}

// Split GEMMs: out = ((part[0] + part[1]) + part[2]) + ... + bias, then the
// epilogue, as wr_cnn_gemm's own when one workgroup runs every group.  Thread
// (x, y): columns 4 (32 blockIdx.y + x) .. +3 of row 8 blockIdx.x + y, so a
// block has 256 threads whatever N.
__global__ void wr_cnn_reduce(CnnGemmArgs a) {
  const int m = blockIdx.x * blockDim.y + threadIdx.y, n = 4 * (blockIdx.y * blockDim.x + threadIdx.x);
  const int64_t dm = cnn_dst_row(a, m);
  if (dm < 0) return;
  const float* p = a.part + (size_t)m * a.N + n;
  float4 v = *(const float4*)p;
#pragma unroll 4
  for (int q = 1; q < a.split; ++q) {
    const float4 w = *(const float4*)(p + (size_t)q * a.M * a.N);
    v.x = v.x + w.x;
    v.y = v.y + w.y;
    v.z = v.z + w.z;
    v.w = v.w + w.w;
  }
  const float4 bn = *(const float4*)(a.bias + n);
  float y[4] = {v.x + bn.x, v.y + bn.y, v.z + bn.z, v.w + bn.w};
  float* d = a.dst + dm * a.N + n;
  if (a.epi == 2) {
    const float4 o = *(const float4*)d;
    y[0] = o.x + y[0];
    y[1] = o.y + y[1];
    y[2] = o.z + y[2];
    y[3] = o.w + y[3];
  } else if (a.epi == 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = wr_relu(y[e]);
  }
  if (a.dst) *(float4*)d = float4{y[0], y[1], y[2], y[3]};
  if (a.dsts) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    uint16_t* s = a.dsts + dm * 2 * a.N + (n >> 5) * 64 + (n & 31);
    *(u16x4*)s = u16x4{cnn_hi(y[0]), cnn_hi(y[1]), cnn_hi(y[2]), cnn_hi(y[3])};
    *(u16x4*)(s + 32) = u16x4{cnn_lo(y[0]), cnn_lo(y[1]), cnn_lo(y[2]), cnn_lo(y[3])};
  }
}

// Input rows of a window of `win` rows per (utterance u, sub-tensor s) for the
// sub-tensors s0 .. s0 + nsb - 1: row m = (u nsb + s - s0) win + k is
// utterance row q = row0 + s row_step + k.  x[m][2z],
// x[m][2z + 1] = the scaled (c, f) of sample B q + z for z < s (the previous
// sub-tensors of row q) when q is a row of the utterance and sub-tensor z has
// made it (q <= front0 + z front_step); zero otherwise and in the padding up
// to kin.
__global__ void wr_cnn_input(CnnInputArgs a) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)a.M * a.kin) return;
  const int m = (int)(idx / a.kin), ch = (int)(idx % a.kin);
  const int k = m % a.win, s = a.s0 + (m / a.win) % a.nsb, u = m / a.win / a.nsb, z = ch >> 1;
  const int64_t q = a.rng ? (int64_t)a.lo[s] + k : a.row0 + (int64_t)s * a.row_step + k;
  float v = 0.0f;
  if (z < s && q >= 0 && q < a.rows && q <= a.front0 + (int64_t)z * a.front_step) {
    const int smp = a.seq[(size_t)u * a.n_samples + (size_t)a.B * q + z];
    v = wr_scale((ch & 1) ? (smp & 255) : (smp >> 8));
  }
  cnn_split_put(a.x, m, a.kin, ch, v);
}

const void* wr_cnn_gemm_ptr(int MI) {
  switch (MI) {
    case 2: return (const void*)wr_cnn_gemm<2>;
    case 3: return (const void*)wr_cnn_gemm<3>;
    default: return (const void*)wr_cnn_gemm<4>;
  }
}
const void* wr_cnn_input_ptr() { return (const void*)wr_cnn_input; }
const void* wr_cnn_reduce_ptr() { return (const void*)wr_cnn_reduce; }
