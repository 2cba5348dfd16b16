// Single-workgroup WaveRNN sampler for small hidden sizes (fp32 weights in the
// registers of one CU).  One workgroup per utterance.  It evaluates Eq. 2 and
// the dual softmax in one fixed order -- every dot product is an fma chain in
// increasing index order from +0, running sums of the softmax weights are
// sequential -- so its samples are deterministic and reproducible bit for bit
// by any implementation of the same order.
//
// What bounds it: the step's serial chain on one CU, of which the two running
// sums of 256 weights, dependent adds that the order fixes, are the longest
// part.  So each wave keeps one role and its weights in registers:
//   wave 0  coarse gates, O1, O2, coarse draw    (2 HP rows of weights a lane)
//   wave 1  fine gates, O3, O4, fine draw
//   wave 2  G = R h of the coarse units (lane i: the u, r, e rows of unit i)
//   wave 3  the same of the fine units
//   wave 4  the uniforms and targets of the next 64 steps, and the next
//           frame's bias + conditioning terms
// R h of the next step over the coarse columns runs beside the coarse output
// layers and draw, and over the fine columns beside the fine ones, so it is
// off the chain.  Halves are padded to HP units (HP inputs a chain): a padded
// term is fma(0, 0, acc) = acc.
// Measured at H = 64, 2,400 steps: 4.26 us a step, against 17.4 with the weights
// in LDS, one sampling thread walking the running sum there and every thread
// computing every step's uniforms.  A dependent fp32 add takes 8 clocks here,
// so the two running sums alone are 1.7 us of it.
#include "wr_kern.h"

namespace {

// Inverse-CDF draw from softmax(z), classes 4 l .. 4 l + 3 on lane l, by one
// wave.  The running sums are sequential over the 256 classes: in round i lane
// i gets the sum up to its last class from lane i - 1's of the round before
// (every lane adds in every round, its result standing from round i on), 4
// adds a round and no memory.  Returns the class (`forced` when >= 0); with NLL
// lse = max z + log(sum exp(z - max z)).
__device__ __forceinline__ int small_draw(float4 z, float u, int forced, bool nll, float& lse) {
  if (forced >= 0 && !nll) return forced;
  const float m = wave_maxf(fmaxf(fmaxf(z.x, z.y), fmaxf(z.z, z.w)));
  const float w0 = wr_exp(z.x - m), w1 = wr_exp(z.y - m), w2 = wr_exp(z.z - m), w3 = wr_exp(z.w - m);
  float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, c3 = 0.0f;
#pragma unroll 16
  for (int i = 0; i < 64; ++i) {
    c0 = dpp<0x138, 0xf, true>(0.0f, c3) + w0;   // wave_shr:1, lane 0 gets 0
    c1 = c0 + w1;
    c2 = c1 + w2;
    c3 = c2 + w3;
  }
  const float Z = lane63(c3);
  if (nll) lse = m + logf(Z);
  if (forced >= 0) return forced;
  const float thr = u * Z;
  int count = __popcll(__ballot(c0 <= thr)) + __popcll(__ballot(c1 <= thr)) + __popcll(__ballot(c2 <= thr)) +
              __popcll(__ballot(c3 <= thr));
  if (count == WR_CLASSES) {   // clamp to the last class with nonzero weight
    int last = -1;
    u64 bb;
    if ((bb = __ballot(w3 > 0.0f))) last = max(last, 4 * (63 - __clzll(bb)) + 3);
    if ((bb = __ballot(w2 > 0.0f))) last = max(last, 4 * (63 - __clzll(bb)) + 2);
    if ((bb = __ballot(w1 > 0.0f))) last = max(last, 4 * (63 - __clzll(bb)) + 1);
    if ((bb = __ballot(w0 > 0.0f))) last = max(last, 4 * (63 - __clzll(bb)));
    count = last;
  }
  return count;
}

struct SmallShared {
  float *h, *G, *add, *hid, *zk, *fm;
  float2* uni;
  int *tgt, *cls;
};

// acc = fma(w[j], x[j], acc), j = 0 .. HP - 1, x in LDS (16-byte aligned).
template <int HP>
__device__ __forceinline__ float chain_r(const float* w, const float* x, float acc) {
#pragma unroll
  for (int j = 0; j < HP; j += 4) {
    const float4 v = *(const float4*)(x + j);
    acc = __builtin_fmaf(w[j], v.x, acc);
    acc = __builtin_fmaf(w[j + 1], v.y, acc);
    acc = __builtin_fmaf(w[j + 2], v.z, acc);
    acc = __builtin_fmaf(w[j + 3], v.w, acc);
  }
  return acc;
}

// Waves 0 (coarse half) and 1 (fine half): gates, output head and draw.
template <int HP, bool FINE>
__device__ __forceinline__ void small_half(const SmallArgs& a, const SmallShared& s, int st) {
  const int H = a.H, Hh = H / 2, l = threadIdx.x & 63;
  const SmallLayout L = small_layout(H);
  const float* img = a.image;
  const bool unit = l < Hh;
  const int i = (FINE ? Hh : 0) + l;               // this lane's unit
  const int Oa = FINE ? L.O3t : L.O1t, ba = FINE ? L.b3 : L.b1, Ob = FINE ? L.O4t : L.O2t, bb = FINE ? L.b4 : L.b2;
  float W1[HP], I[3][3];
  float4 W2[HP];
#pragma unroll
  for (int j = 0; j < HP; ++j) {
    W1[j] = unit && j < Hh ? img[Oa + j * Hh + l] : 0.0f;
    W2[j] = j < Hh ? *(const float4*)(img + Ob + j * WR_CLASSES + 4 * l) : float4{0.0f, 0.0f, 0.0f, 0.0f};
  }
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int q = 0; q < 3; ++q) I[g][q] = unit ? img[L.I + (g * H + i) * 3 + q] : 0.0f;
  const float b1 = unit ? img[ba + l] : 0.0f;
  const float4 b2 = *(const float4*)(img + bb + 4 * l);
  float h = unit && a.h_in ? a.h_in[(size_t)st * H + i] : 0.0f;
  int cp = a.c_in ? a.c_in[st] : 128, fp = a.f_in ? a.f_in[st] : 0;
  const int hp = l < HP ? l : 0;
  int64_t fr = a.Dc > 0 ? a.t0 / a.frame_len : 0, edge = a.Dc > 0 ? (fr + 1) * a.frame_len : INT64_MAX;
  int ab = 0;                                      // buffer of this frame's additive terms
  __syncthreads();                                 // h, G and the first frame's terms are in
  for (int64_t t = 0; t < a.T; ++t) {
    if (a.t0 + t == edge) {
      edge += a.frame_len;
      ab ^= 1;
    }
    const int bs = (int)(t >> 6 & 1) * 64 + (int)(t & 63);
    const float2 un = s.uni[bs];
    const int tg = s.tgt[bs];
    const float* G = s.G + (FINE ? 3 * HP : 0) + hp;
    const float* add = s.add + ab * 6 * HP + (FINE ? 3 * HP : 0) + hp;
    const float gu = G[0], gr = G[HP], ge = G[2 * HP], du = add[0], dr = add[HP], de = add[2 * HP];
    const float x0 = wr_scale(cp), x1 = wr_scale(fp);
    int c = 0;
    float x2 = 0.0f;
    if (FINE) {
      __syncthreads();                             // (a) coarse gates done
      __syncthreads();                             // (b) c_t drawn
      c = s.cls[0];
      x2 = wr_scale(c);
    }
    float ix[3];
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      ix[g] = __builtin_fmaf(I[g][1], x1, __builtin_fmaf(I[g][0], x0, 0.0f));
      if (FINE) ix[g] = __builtin_fmaf(I[g][2], x2, ix[g]);
    }
    const float u = wr_sigmoid(gu + (ix[0] + du));
    const float r = wr_sigmoid(gr + (ix[1] + dr));
    const float e = wr_tanh(__builtin_fmaf(r, ge, ix[2] + de));
    h = __builtin_fmaf(u, h, (1.0f - u) * e);
    float* y = s.h + (FINE ? HP : 0);
    if (unit) y[l] = h;
    __syncthreads();                               // (a) / (c) gates done
    const float hv = wr_relu(chain_r<HP>(W1, y, 0.0f) + b1);
    float* hid = s.hid + (FINE ? HP : 0);
    if (unit) hid[l] = hv;
    __builtin_amdgcn_wave_barrier();               // (one wave: its LDS accesses are in order)
    float4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < HP; j += 4) {
      const float4 v = *(const float4*)(hid + j);
      const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        z.x = __builtin_fmaf(W2[j + q].x, x[q], z.x);
        z.y = __builtin_fmaf(W2[j + q].y, x[q], z.y);
        z.z = __builtin_fmaf(W2[j + q].z, x[q], z.z);
        z.w = __builtin_fmaf(W2[j + q].w, x[q], z.w);
      }
    }
    z.x += b2.x;
    z.y += b2.y;
    z.z += b2.z;
    z.w += b2.w;
    const int64_t o = (int64_t)st * a.T + t;
    float* zo = FINE ? a.zf_out : a.zc_out;
    if (zo) *(float4*)(zo + o * WR_CLASSES + 4 * l) = z;
    float lse = 0.0f;
    const int d = small_draw(z, FINE ? un.y : un.x, a.target ? (FINE ? tg & 255 : tg >> 8) : -1,
                             a.nll_out != nullptr, lse);
    float zd = 0.0f;
    if (a.nll_out) {                               // the drawn class's logit
      float* zk = s.zk + (FINE ? WR_CLASSES : 0);
      *(float4*)(zk + 4 * l) = z;
      __builtin_amdgcn_wave_barrier();
      zd = zk[d];
    }
    if (!FINE) {
      if (l == 0) {
        s.cls[0] = d;
        s.fm[0] = lse;
        s.fm[1] = zd;
      }
      __syncthreads();                             // (b) c_t drawn
      cp = d;
      __syncthreads();                             // (c) fine gates done
      __syncthreads();                             // (d) f_t drawn, G of the next step ready
      fp = s.cls[1];
    } else {
      if (l == 0) {
        s.cls[1] = d;
        if (a.out) a.out[o] = (uint16_t)(256 * c + d);
        if (a.nll_out) a.nll_out[o] = (s.fm[0] - s.fm[1]) + (lse - zd);
      }
      cp = c;
      fp = d;
      __syncthreads();                             // (d)
    }
  }
  if (a.h_out && unit) a.h_out[(size_t)st * H + i] = h;
  if (FINE && l == 0) {
    if (a.c_out) a.c_out[st] = (uint8_t)cp;
    if (a.f_out) a.f_out[st] = (uint8_t)fp;
  }
}

// Waves 2 and 3: R h of the coarse and of the fine units.
template <int HP>
__device__ __forceinline__ void small_matvec(const SmallArgs& a, const SmallShared& s, bool fine) {
  const int H = a.H, Hh = H / 2, l = threadIdx.x & 63;
  const float* Rt = a.image + small_layout(H).Rt;
  const int i = (fine ? Hh : 0) + l;
  float W[3][2 * HP];
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int j = 0; j < 2 * HP; ++j) {
      const int k = j < HP ? j : Hh + j - HP;      // column of padded input j
      W[g][j] = l < Hh && (j < HP ? j : j - HP) < Hh ? Rt[(size_t)k * 3 * H + g * H + i] : 0.0f;
    }
  float acc[3];
  auto columns = [&](bool f) {
#pragma unroll
    for (int j = 0; j < HP; j += 4) {
      const float4 v = *(const float4*)(s.h + (f ? HP : 0) + j);
      const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int g = 0; g < 3; ++g)
          acc[g] = __builtin_fmaf(f ? W[g][HP + j + q] : W[g][j + q], x[q], acc[g]);
    }
  };
  auto put = [&]() {
    if (l < HP)
#pragma unroll
      for (int g = 0; g < 3; ++g) s.G[(fine ? 3 * HP : 0) + g * HP + l] = acc[g];
  };
  acc[0] = acc[1] = acc[2] = 0.0f;
  columns(false);
  columns(true);
  put();
  __syncthreads();
  for (int64_t t = 0; t < a.T; ++t) {
    __syncthreads();                               // (a)
    acc[0] = acc[1] = acc[2] = 0.0f;
    columns(false);
    __syncthreads();                               // (b)
    __syncthreads();                               // (c)
    columns(true);
    put();                                         // (the fine gates of this step have read theirs)
    __syncthreads();                               // (d)
  }
}

// Wave 4: uniforms, targets and the additive terms of the gates.
template <int HP>
__device__ __forceinline__ void small_side(const SmallArgs& a, const SmallShared& s, int st) {
  const int H = a.H, Hh = H / 2, l = threadIdx.x & 63;
  const SmallLayout L = small_layout(H);
  auto batch = [&](int64_t t, int buf) {
    const int64_t n = t + l;
    if (n >= a.T) return;
    float uc, uf;
    wr_uniforms(a.seed, (uint64_t)st, (uint64_t)(a.t0 + n), &uc, &uf);
    s.uni[buf * 64 + l] = float2{uc, uf};
    s.tgt[buf * 64 + l] = a.target ? a.target[(int64_t)st * a.T + n] : 0;
  };
  auto frame = [&](int64_t fr, int buf) {          // bias (+ conditioning of the frame)
    if (a.Dc > 0 && fr >= a.n_frames) fr = a.n_frames - 1;
    for (int row = l; row < 3 * H; row += 64) {
      const float b = a.image[L.bias + row];
      float v = b;
      if (a.Dc > 0) {
        const float* w = a.Wc + (size_t)row * a.Dc;
        const float* x = a.feat + ((size_t)st * a.n_frames + fr) * a.Dc;
        float acc = 0.0f;
        for (int j = 0; j < a.Dc; ++j) acc = __builtin_fmaf(w[j], x[j], acc);
        v = acc + b;
      }
      const int g = row / H, i = row % H;
      s.add[buf * 6 * HP + (i >= Hh ? 3 * HP + i - Hh : i) + g * HP] = v;
    }
  };
  int64_t fr = a.Dc > 0 ? a.t0 / a.frame_len : 0, edge = a.Dc > 0 ? (fr + 1) * a.frame_len : INT64_MAX;
  int ab = 0;
  frame(fr, 0);
  batch(0, 0);
  __syncthreads();
  for (int64_t t = 0; t < a.T; ++t) {
    if ((t & 63) == 0) batch(t + 64, (int)((t >> 6) + 1 & 1));
    if (a.t0 + t + 1 == edge) {                    // the next step starts a frame
      ab ^= 1;
      if (t + 1 < a.T) frame(++fr, ab);
      edge += a.frame_len;
    }
    __syncthreads();
    __syncthreads();
    __syncthreads();
    __syncthreads();
  }
}

}  // namespace

template <int HP>
__global__ __launch_bounds__(WR_SMALL_THREADS, 1) void wr_small_kernel(SmallArgs a) {
  __shared__ __align__(16) float hs[2 * HP], G[6 * HP], add[12 * HP], hid[2 * HP], zk[2 * WR_CLASSES], fm[4];
  __shared__ float2 uni[128];
  __shared__ int tgt[128], cls[2];
  const SmallShared s{hs, G, add, hid, zk, fm, uni, tgt, cls};
  const int Hh = a.H / 2, tid = threadIdx.x, wave = tid >> 6;
  const int st = blockIdx.x;  // utterance = Philox stream
  for (int i = tid; i < 2 * HP; i += WR_SMALL_THREADS) {
    const int f = i >= HP, k = i - f * HP;
    hs[i] = k < Hh && a.h_in ? a.h_in[(size_t)st * a.H + f * Hh + k] : 0.0f;
    hid[i] = 0.0f;
  }
  for (int i = tid; i < 12 * HP; i += WR_SMALL_THREADS) add[i] = 0.0f;
  __syncthreads();
  if (wave == 0) small_half<HP, false>(a, s, st);
  else if (wave == 1) small_half<HP, true>(a, s, st);
  else if (wave < 4) small_matvec<HP>(a, s, wave == 3);
  else small_side<HP>(a, s, st);
}

// HP: units of a half, padded; Hh <= 36 fits the registers (and the plan's limit).
const void* wr_small_kernel_ptr(int H) {
  const int Hh = H / 2;
  if (Hh <= 16) return (const void*)wr_small_kernel<16>;
  if (Hh <= 32) return (const void*)wr_small_kernel<32>;
  if (Hh <= 36) return (const void*)wr_small_kernel<36>;
  return nullptr;
}

// Uniforms exactly as the sampling kernels draw them (for tests).
extern "C" __global__ void wr_uniforms_kernel(uint64_t seed, uint64_t stream, int64_t t0, int64_t n, float* out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float uc, uf;
  wr_uniforms(seed, stream, (uint64_t)(t0 + i), &uc, &uf);
  out[2 * i] = uc;
  out[2 * i + 1] = uf;
}

const void* wr_uniforms_kernel_ptr() { return (const void*)wr_uniforms_kernel; }
