// Teacher-forced scoring of the dense batch-1 model (the NLL of Sec. 5 on
// given audio).  With every byte of every step given, a step only updates h
// (the gates of Eq. 2): no draw and no output layer sits in the serial loop,
// so one kind of workgroup does it all, with one exchange per step.
//
// The utterances of a call are dealt to up to 8 groups of LV of them (LV = 1,
// 2, 4 or 8: as few a group as 8 groups allow), group g on XCD g (or `rot`
// XCDs on, beside another model's launch), all in one launch.  Workgroup k of a group owns hidden units 32 k .. 32 k + 31 (all in
// one half) of its vectors.  Waves 0-3 hold the six tiles of their gate rows of
// R (u, r, e) in VGPRs and form R h on the matrix cores; of waves 4-7, 32 LV
// threads finish the gates with the given bytes and publish the new slice of
// h, and all gather the next h from the group's workgroups into the operand image (an
// all-gather: one hop per step).
//
// What bounds it is that hop and the products between two of them, so a group
// fits one XCD (28 of its 32 CUs at H = 896) and publishes into its L2 when it
// finds itself there.  H = 896, us a step, with 56 workgroups of 16 units over
// all XCDs (grids of several utterances on streams of their own) and now: one
// utterance 2.27 -> 1.42, 21 utterances 5.3 -> 2.2 with their output layers (4.1
// before where the four grids' streams had a hardware queue each).
//
// The products and the gate arithmetic are the sampling kernel's operation for
// operation, so a scored trajectory reproduces the sampler's state bit for
// bit: a fine row's R h is one pass over all columns (even and odd column
// tiles in two accumulation chains), a coarse row's is the sampling units'
// coarse-column part (two chains, + bias and conditioning) plus the sampling
// mirrors' fine-column part (one chain per half of the fine columns, the
// halves added), each rounded as the exchange delivers it (lowest bit
// cleared).  Every chain is one wave's, over several row tiles, so that an
// operand read from LDS serves 3 (fine) or 6 (coarse) products: fine wave w
// runs chain w % 2 of unit tile w / 2, coarse wave w chain w of both.  Vector b
// sits in rows 2b and 2b + 1 of the operand image, so the products cost what
// one vector's do and do not depend on the others.  The output layers run
// afterwards over all steps at once (wr_cnn_gemm), and the NLL per step in
// wr_score_nll.
//
// Exchange: h_s goes to buffer s mod 2 of [2][LV][H] words, tagged with the
// parity of its generation s / 2 + 1.  A workgroup writes h_{s+2} into a
// buffer only after it has read every workgroup's h_{s+1}, which each
// publishes only after reading all of h_s: no reader is overtaken, and the
// generation bit tells h_s from h_{s-2} in the same buffer.
#include "wr_kern.h"

// Delay (x 64 clocks) before a gather's first probe (one utterance of 24,000
// steps, ms: 0 34.5, 2 34.1, 4 35.2, 8 37.4; eight a group: 0 and 2 alike).
#define WR_SCORE_DELAY 2

template <int KT2, int LV>
__global__ __launch_bounds__(WR_THREADS, 1) void wr_score_kernel(ScoreArgs a) {
  constexpr int H = 32 * KT2, Hh = H / 2, KT = KT2 / 2, NW = H / 32;
  constexpr int FH = KT2 / 2, CH = KT / 2, NF = 3 * FH;   // column tiles of a fine and a coarse chain, fragments
  const int b = wr_block(a.by_xcd), g = (b - a.rot) & 7, k = b / 8;
  if (g >= a.G || k >= NW) return;
  __shared__ __align__(16) unsigned char img[KT2 * WR_FRAGP];   // operand image of h
  __shared__ float part[24 * LV * 16];               // [chain][unit tile][gate][LV][16] products
  __shared__ int tgt[2][64 * LV];                    // [j][LV] targets of a batch of 64 steps
  __shared__ int misc[2];                            // [0] abort
  const int v0 = g * LV, nv = min(LV, a.S - v0);     // this group's vectors
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const bool fine = 32 * k >= Hh;
  xw* X = a.xc + (size_t)g * score_words(H, LV);
  for (int i = tid; i < KT2 * WR_FRAGP / 16; i += WR_THREADS) ((uint4*)img)[i] = uint4{0, 0, 0, 0};
  if (tid == 0) misc[0] = 0;
  __syncthreads();
  for (int i = tid; i < nv * H; i += WR_THREADS)
    aput_p(img, i % H, a.h_in ? xround(a.h_in[(size_t)v0 * H + i]) : 0.0f, i / H);
  if (wave < 4) {   // products; each role has its own step loop, so its registers are its own
    bf16x8 W[NF];
    const uint4* src = a.w + ((size_t)(k * 4 + wave) * NF) * 64 + lane;
#pragma unroll
    for (int i = 0; i < NF; ++i) W[i] = __builtin_bit_cast(bf16x8, src[(size_t)i * 64]);
    group_shares_xcd(X + 2 * LV * H, NW, k, misc + 1, a);
    __syncthreads();
    const int row = lane & 15, b0 = 2 * (lane >> 4);
    auto put = [&](int i, f32x4 d) {                 // tile i = chain * 6 + unit tile * 3 + gate
      if (b0 < LV) part[(i * LV + b0) * 16 + row] = mfma_row(d);
      if (b0 + 1 < LV) part[(i * LV + b0 + 1) * 16 + row] = mfma_row_hi(d);
    };
    for (int64_t s = 0; s < a.T; ++s) {
      if (s > 0) {
        __syncthreads();                             // h_{s-1} is in the image
        if (misc[0]) return;
      }
      if (fine) {
        f32x4 acc[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) acc[q] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < FH; ++i) {
          const bf16x8 x = afrag_p(img, 2 * i + (wave & 1));
#pragma unroll
          for (int q = 0; q < 3; ++q) acc[q] = mfma(x, W[q * FH + i], acc[q]);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) put((wave & 1) * 6 + (wave >> 1) * 3 + q, acc[q]);
      } else {
        f32x4 acc[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) acc[q] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          const bf16x8 x = afrag_p(img, wave < 2 ? 2 * i + wave : KT + (wave - 2) * CH + i);
#pragma unroll
          for (int q = 0; q < 6; ++q) acc[q] = mfma(x, W[q * CH + i], acc[q]);
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) put(wave * 6 + q, acc[q]);
      }
      __syncthreads();                               // the products are in
    }
    return;
  }
  // waves 4-7.  Gate thread r < 32 nv: unit u of vector ub, its I* row, its
  // full-precision state and last bytes
  const int r = tid - 256, ub = r >> 5, vb = v0 + (ub < nv ? ub : 0);
  const bool gt = ub < nv;
  const int u = 32 * k + (r & 31);
  float cf[3][3];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) cf[q][c] = gt ? a.Iw[3 * (q * H + u) + c] : 0.0f;
  float h = gt && a.h_in ? a.h_in[(size_t)vb * H + u] : 0.0f;
  int cp = a.c_in ? a.c_in[vb] : 128, fp = a.f_in ? a.f_in[vb] : 0;
  // this vector's bias + conditioning of unit u, read once a frame; the frame
  // changes at step `edge` (the last one stays)
  const float* cbv = a.cb + (size_t)vb * a.n_cb * 3 * H + u;
  float cb[3] = {0.0f, 0.0f, 0.0f};
  int64_t fr = a.t0 / a.frame_len, edge = 0;
  if (fr >= a.n_cb) fr = a.n_cb - 1;
  auto frame = [&]() {
    if (gt)
#pragma unroll
      for (int q = 0; q < 3; ++q) cb[q] = cbv[fr * 3 * H + q * H];
    edge = fr + 1 < a.n_cb ? (fr + 1) * a.frame_len - a.t0 : INT64_MAX;
    ++fr;
  };
  frame();
  // targets of 64 steps, read here and put into LDS a step later
  constexpr int TN = (64 * LV + 255) / 256;
  int tv[TN] = {};
  auto targets = [&](int64_t s) {
#pragma unroll
    for (int m = 0; m < TN; ++m) {
      const int i = r + 256 * m, b = i % LV;
      const int64_t n = s + i / LV;
      if (i < 64 * LV && b < nv && n < a.T) tv[m] = a.target[(size_t)(v0 + b) * a.T + n];
    }
  };
  auto put_targets = [&](int buf) {
#pragma unroll
    for (int m = 0; m < TN; ++m)
      if (r + 256 * m < 64 * LV) tgt[buf][r + 256 * m] = tv[m];
  };
  targets(0);
  put_targets(0);
  const bool lx = group_shares_xcd(X + 2 * LV * H, NW, k, misc + 1, a) && WR_LOCAL_XCHG;
  __builtin_amdgcn_s_waitcnt(0);   // prologue loads in before the loop (see the persistent heads)
  __syncthreads();
  for (int64_t s = 0; s < a.T; ++s) {
    if (s > 0) {   // h_{s-1} of every workgroup and vector into the image
      __builtin_amdgcn_s_sleep(WR_SCORE_DELAY);
      if (!gather_y<LV, H, 256, true>(X + ((s - 1) & 1) * (LV * H),
                                      (uint32_t)((s - 1) >> 1) + 1u, img, r, -1, a))
        misc[0] = 1;
      __syncthreads();
      if (misc[0]) return;
    }
    if ((s & 63) == 0) targets(s + 64);
    if ((s & 63) == 1) put_targets((int)(((s >> 6) + 1) & 1));
    __syncthreads();                                 // the products are in
    xw* Y = X + (size_t)((s & 1) * LV + ub) * H + u;
    const uint32_t tag = (uint32_t)(s >> 1) + 1u;
    if (!gt && ub < LV) xpub_l(Y, tag, 0.0f, lx);      // a vector not in use: its words are waited for too
    if (gt) {
      const int ut = (r >> 4) & 1, row = r & 15;
      auto P = [&](int chain, int q) { return part[((chain * 6 + ut * 3 + q) * LV + ub) * 16 + row]; };
      float v[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        float x = P(0, q) + P(1, q);
        if (q < 2) x += cb[q];                       // bias + conditioning of u and r
        v[q] = fine ? xround(x) : xround(x) + xround(P(2, q) + P(3, q));
      }
      const float v0 = v[0], v1 = v[1], v2 = v[2], cbe = cb[2];
      const int tg = tgt[(s >> 6) & 1][(int)(s & 63) * LV + ub], c = tg >> 8;
      const float x0 = fscale(cp), x1 = fscale(fp);
      float uu, rr, e;
      if (!fine) {   // the sampling head's coarse terms, then its gates with f_{t-1}
        const float cu = v0 + cf[0][0] * x0, cr = v1 + cf[1][0] * x0, cie = cf[2][0] * x0;
        uu = fsig(__builtin_fmaf(cf[0][1], x1, cu)), rr = fsig(__builtin_fmaf(cf[1][1], x1, cr));
        e = ftanh(__builtin_fmaf(rr, v2, __builtin_fmaf(cf[2][1], x1, cie) + cbe));
      } else {       // its fine terms, then its gates with c_t
        const float fu = v0 + __builtin_fmaf(cf[0][1], x1, cf[0][0] * x0);
        const float fr = v1 + __builtin_fmaf(cf[1][1], x1, cf[1][0] * x0);
        const float fie = __builtin_fmaf(cf[2][1], x1, cf[2][0] * x0);
        const float x2 = fscale(c);
        uu = fsig(__builtin_fmaf(cf[0][2], x2, fu)), rr = fsig(__builtin_fmaf(cf[1][2], x2, fr));
        e = ftanh(__builtin_fmaf(rr, v2, __builtin_fmaf(cf[2][2], x2, fie) + cbe));
      }
      h = __builtin_fmaf(uu, h, (1.0f - uu) * e);
      xpub_l(Y, tag, h, lx);
      // a split row (CnnGemmArgs): units 32 k .. are one of its groups
      uint16_t* tr = (fine ? a.traj_f : a.traj_c) + ((size_t)vb * a.T + s) * H + 64 * (fine ? k - NW / 2 : k) + (r & 31);
      tr[0] = (uint16_t)(__float_as_uint(h) >> 16);
      tr[32] = __builtin_bit_cast(uint16_t, (__bf16)(h - __uint_as_float(__float_as_uint(h) & 0xffff0000u)));
      cp = c;
      fp = tg & 255;
      if (s + 1 == edge) frame();
    }
  }
  if (gt && a.h_out) a.h_out[(size_t)vb * H + u] = h;
  if (k == 0 && gt && (r & 31) == 0) {
    if (a.c_out) a.c_out[vb] = (uint8_t)cp;
    if (a.f_out) a.f_out[vb] = (uint8_t)fp;
  }
}

// NLL of each scored step from its logits: (lse z_c - z_c[c]) + (lse z_f - z_f[f]),
// one wave per row, with the draw's reduction (max, hardware exp2, sum, log).
extern "C" __global__ void wr_score_nll(const float* zc, const float* zf, const uint16_t* target, int64_t rows,
                                        float* nll) {
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int l = threadIdx.x & 63, tg = target[row];
  float r[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float* z = (q ? zf : zc) + row * 256;
    const float4 z4 = *(const float4*)(z + 4 * l);
    const float mx = wave_maxf(fmaxf(fmaxf(z4.x, z4.y), fmaxf(z4.z, z4.w)));
    float sm = fexp(z4.x - mx) + fexp(z4.y - mx) + fexp(z4.z - mx) + fexp(z4.w - mx);
    for (int o = 32; o >= 1; o >>= 1) sm += __shfl_xor(sm, o, 64);
    r[q] = (mx + __logf(sm)) - z[q ? (tg & 255) : (tg >> 8)];
  }
  if (l == 0) nll[row] = r[0] + r[1];
}

template <int LV>
static const void* score_ptr(int KT2) {
  switch (KT2) {
    case 4: return (const void*)wr_score_kernel<4, LV>;
    case 8: return (const void*)wr_score_kernel<8, LV>;
    case 12: return (const void*)wr_score_kernel<12, LV>;
    case 16:   // H = 512 has no batched kernel, so its models serve one utterance
      if constexpr (LV == 1) return (const void*)wr_score_kernel<16, 1>;
      else return nullptr;
    case 28: return (const void*)wr_score_kernel<28, LV>;
    default: return nullptr;
  }
}
const void* wr_score_kernel_ptr(int KT2, int LV) {
  return LV == 1 ? score_ptr<1>(KT2) : LV == 2 ? score_ptr<2>(KT2) : LV == 4 ? score_ptr<4>(KT2) : score_ptr<8>(KT2);
}
const void* wr_score_nll_ptr() { return (const void*)wr_score_nll; }
