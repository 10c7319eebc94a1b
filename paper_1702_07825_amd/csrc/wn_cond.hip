// Conditioning network on gfx950 (Deep Voice, arXiv 1702.07825, Appendix A.2): two
// bidirectional fo-pooling QRNN layers with width-2 convolutions, the two directions' channels
// interleaved, and upsampling to the audio rate by repetition.  Declarations and contracts are
// in include/wn_cond.h.
//
// Each layer is two kernels.  The gate pre-activations of all frames at once are a dense
// contraction, [3h x 2 cin] . [2 cin x B*Tf] per direction (the width-2 convolution: tap 0 is the
// direction's previous frame, tap 1 the current one), run as split bf16 products that keep fp32's
// precision, in tiles staged through LDS; the weights are stored split, with each tap padded to a
// multiple of 32 inputs so that K chunks never straddle the taps.  The fo-pool is a linear recurrence
// along the frames, independent per (stream, direction, channel), run in segments of frames.  The second
// layer's pool writes its output interleaved, and a last kernel repeats every frame over its audio steps
// (bound by the HBM write of [B][T][2 h2]).
#include "wn_cond.h"
#include "wn.h"
#include "wn_internal.h"
#include "wn_mfma.h"
#include "wn_wave.h"

#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

struct wn_cond {
  int device = 0;
  int F = 0, h1 = 0, h2 = 0, fr = 1, ar = 1;
  int cinp1 = 0, cinp2 = 0;  // per-tap input widths of the two layers rounded up to 32
  void* dmem = nullptr;
  const unsigned short *w1 = nullptr, *w2 = nullptr;  // split (see split3)
  const float *wf1 = nullptr, *wf2 = nullptr;         // what they are split from
  const float *b1 = nullptr, *b2 = nullptr;
  void* scratch = nullptr;  // device address of this device's copy of `scratch` (wn_condition_static)
};

// Scratch of wn_condition_static: one copy per device, held until the process ends.  Host code
// never uses the array's name as an address (on the host it is only a stand-in for the symbol);
// wn_cond_create looks up each device's address of it once, with that device current.
static __device__ __align__(256) unsigned char scratch[WN_COND_SCRATCH_BYTES];

namespace {

using wnk::bf16x8;
using wnk::f32x4;
using wnk::u16;
using wnk::u32x4;

struct GateArgs {
  const float* x;  // [B][Tf][cin]
  const u16* w;    // [2][N][2 cinp / 32][3][32]: split weights; tap 0 (previous frame) inputs 0..cin-1, tap 1 at cinp.., zeros past cin
  const float* wf; // [2][N][2 cinp]: the fp32 weights
  const float* b;  // [2][N]
  float* p;        // [B][Tf][2][N]
  int B, Tf, cin, cinp, N;
};

// fp32 products on bf16 MFMA.  A value is split into three bf16 parts, each the nearest to what the ones
// before leave, v = h + m + l to 2^-25 of it, and a product takes the six of the nine part products that
// reach fp32's precision (the others are below 2^-26 of it), smallest first, summed in fp32.  An infinity
// stays in h alone, but its products with the other side's parts can be of both signs or with a zero part,
// a value within 2^-9 of fp32's largest has no finite h, and a product within 2^-8 of it can be an infinity
// as h h alone: such a sum ends as NaN or infinite and is taken again in fp32 (exact_gate).
__device__ __forceinline__ void split3(f32x4 v, uint2& h, uint2& m, uint2& l) {
  h = make_uint2(wnk::pack_bf16(v[0], v[1]), wnk::pack_bf16(v[2], v[3]));
  const float hv[4] = {wnk::low_bf16(h.x), wnk::high_bf16(h.x), wnk::low_bf16(h.y), wnk::high_bf16(h.y)};
  float r[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = hv[e] == v[e] ? 0.f : v[e] - hv[e];
  m = make_uint2(wnk::pack_bf16(r[0], r[1]), wnk::pack_bf16(r[2], r[3]));
  l = make_uint2(wnk::pack_bf16(r[0] - wnk::low_bf16(m.x), r[1] - wnk::high_bf16(m.x)),
                 wnk::pack_bf16(r[2] - wnk::low_bf16(m.y), r[3] - wnk::high_bf16(m.y)));
}

// Weights [rows][K] (K a multiple of 32) to [rows][K / 32][3][32].
__global__ __launch_bounds__(256) void split_weights(const float* src, u16* dst, size_t n) {
  const size_t i = 4 * ((size_t)blockIdx.x * 256 + threadIdx.x);
  if (i >= n) return;
  uint2 h, m, l;
  split3(*reinterpret_cast<const f32x4*>(src + i), h, m, l);
  u16* d = dst + i / 32 * 96 + i % 32;
  *reinterpret_cast<uint2*>(d) = h;
  *reinterpret_cast<uint2*>(d + 32) = m;
  *reinterpret_cast<uint2*>(d + 64) = l;
}

// One gate pre-activation (row n, direction dir, frame m) in plain fp32, without the bias.
__device__ __forceinline__ float exact_gate(const GateArgs& a, int dir, int n, int m) {
  const int bb = m / a.Tf, t = m - bb * a.Tf, tp = dir == 0 ? t - 1 : t + 1;
  const float* xc = a.x + (size_t)m * a.cin;
  const bool has = tp >= 0 && tp < a.Tf;
  const float* xp = has ? a.x + ((size_t)bb * a.Tf + tp) * a.cin : xc;
  const float* w = a.wf + ((size_t)dir * a.N + n) * 2 * a.cinp;
  float s = 0.f;
  for (int k = 0; k < a.cin && s == s; ++k) s = fmaf(w[a.cinp + k], xc[k], fmaf(w[k], has ? xp[k] : 0.f, s));
  return s;
}

// Gate pre-activations of every frame of a layer, both directions (grid.z):
//   p[b][t][dir][n] = b[dir][n] + sum_k w[dir][n][0][k] x[b][t'][k] + w[dir][n][1][k] x[b][t][k]
// with t' = t - 1 (forward) or t + 1 (backward) and x = 0 outside the frames: the width-2
// convolution as one dense contraction [N x 2 cinp] . [2 cinp x B Tf], in split bf16 products
// (v_mfma_f32_16x16x32_bf16).  VT x VT output tiles (gate rows x frames) per 256 threads, each wave a
// quarter; K in chunks of 32 that never straddle the two taps (cinp is a multiple of 32), staged in LDS as
// the three parts of a row's chunk, with the next chunk's global loads in flight during the current
// chunk's products and a second block on the CU beside them.  The MFMA A operand is the weight rows and B
// the frames, so each lane ends with four consecutive gate rows of one frame.  VX: the input rows are
// float4 aligned (cin % 4 == 0), else they are read one float at a time.
// Bound: the bf16 matrix rate, six products for one.  Measured, 32 streams x 512 frames: second layer (281
// GFLOP) 2244 us on fp32 MFMA, 1359 so (207 TFLOP/s, 1.24 PFLOP/s of bf16 products, about what a large
// bf16 matrix product reaches on the card); error against 64 bits 3.4e-7 and 3.2e-7 (of the whole network).
constexpr int NTG = 256;
constexpr int VK = 32, VLD = 3 * VK + 16;  // K chunk; LDS row (16-bit units): 32 bytes mod 64 (conflicts a quarter of the LDS cycles)

template <int VT, bool VX>
__global__ __launch_bounds__(NTG, 2) void qrnn_gate_gemm(const GateArgs a) {
  constexpr int NI = VT / 32, ND = VT / 32;  // rows per thread of a chunk of x; 16 x 16 tiles per wave side
  constexpr int NW = VT * 12 / NTG;          // 16-byte pieces of a chunk of weights per thread
  const int dir = blockIdx.z;
  const int m0 = blockIdx.x * VT, n0 = blockIdx.y * VT;
  const int M = a.B * a.Tf, K = 2 * a.cinp, N = a.N;
  __shared__ __align__(16) u16 Ws[VT][VLD];
  __shared__ __align__(16) u16 Xs[VT][VLD];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wn = (wave >> 1) * (VT / 2), wm = (wave & 1) * (VT / 2);
  const int r16 = lane & 15, q = lane >> 4;
  // x: rows tid / 8 + 32 i, float4 column tid % 8 of the chunk
  const int lr = tid >> 3, lc = (tid & 7) * 4;
  const float* xcur[NI];
  const float* xprev[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = m0 + lr + 32 * i;
    xcur[i] = xprev[i] = nullptr;
    if (m < M) {
      const int bb = m / a.Tf, t = m - bb * a.Tf;
      const int tp = dir == 0 ? t - 1 : t + 1;
      xcur[i] = a.x + ((size_t)bb * a.Tf + t) * a.cin;
      if (tp >= 0 && tp < a.Tf) xprev[i] = a.x + ((size_t)bb * a.Tf + tp) * a.cin;
    }
  }
  // weights: piece tid + 256 i is piece (.. % 12) of row (.. / 12); rows past N repeat the last one
  const u32x4* wsrc[NW];
  int wdst[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int pc = tid + NTG * i, row = pc / 12, c = pc % 12;
    wsrc[i] = reinterpret_cast<const u32x4*>(a.w + ((size_t)dir * N + min(n0 + row, N - 1)) * K * 3) + c;
    wdst[i] = row * VLD + c * 8;
  }
  f32x4 gx[NI];
  u32x4 gw[NW];
  auto load = [&](int c) {
    const int k0 = c * VK;
    const bool prev = k0 < a.cinp;
    const int kk = (prev ? k0 : k0 - a.cinp) + lc;  // input index of this thread's first float
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const float* xp = prev ? xprev[i] : xcur[i];
      if (VX) {
        gx[i] = xp && kk < a.cin ? *reinterpret_cast<const f32x4*>(xp + kk) : f32x4{0.f, 0.f, 0.f, 0.f};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) gx[i][e] = xp && kk + e < a.cin ? xp[kk + e] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) gw[i] = wsrc[i][12 * c];
  };
  auto stash = [&] {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      uint2 h, m, l;
      split3(gx[i], h, m, l);
      u16* d = &Xs[lr + 32 * i][lc];
      *reinterpret_cast<uint2*>(d) = h;
      *reinterpret_cast<uint2*>(d + 32) = m;
      *reinterpret_cast<uint2*>(d + 64) = l;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) *reinterpret_cast<u32x4*>(&Ws[0][0] + wdst[i]) = gw[i];
  };
  f32x4 acc[ND][ND];
#pragma unroll
  for (int i = 0; i < ND; ++i)
#pragma unroll
    for (int j = 0; j < ND; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  load(0);
  const int nk = K / VK;
  for (int c = 0; c < nk; ++c) {
    stash();
    wnk::lds_barrier();
    load(min(c + 1, nk - 1));
    bf16x8 wa[ND][3], xb[ND][3];
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        wa[i][s] = *reinterpret_cast<const bf16x8*>(&Ws[wn + 16 * i + r16][32 * s + 8 * q]);
        xb[i][s] = *reinterpret_cast<const bf16x8*>(&Xs[wm + 16 * i + r16][32 * s + 8 * q]);
      }
    constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int s = 0; s < 6; ++s)
#pragma unroll
      for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int j = 0; j < ND; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[i][PA[s]], xb[j][PB[s]], acc[i][j], 0, 0, 0);
    wnk::lds_barrier();
  }
  // acc[i][j]: lane holds gate rows wn + 16 i + 4 q .. +3 of frame wm + 16 j + r16
  const float* bd = a.b + (size_t)dir * N;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int n = n0 + wn + 16 * i + 4 * q;
    if (n >= N) continue;
    const bool whole = (N & 3) == 0;  // then n + 3 < N and the row offsets are float4 aligned
    f32x4 bias;
#pragma unroll
    for (int v = 0; v < 4; ++v) bias[v] = n + v < N ? bd[n + v] : 0.f;
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      const int m = m0 + wm + 16 * j + r16;
      if (m >= M) continue;
      float* dst = a.p + ((size_t)m * 2 + dir) * N + n;
      f32x4 v4 = acc[i][j] + bias;
      if (!__builtin_isfinite(v4[0]) || !__builtin_isfinite(v4[1]) || !__builtin_isfinite(v4[2]) || !__builtin_isfinite(v4[3])) {
#pragma unroll 1
        for (int v = 0; v < 4 && n + v < N; ++v) {
          const float e = exact_gate(a, dir, n + v, m) + bd[n + v];
          v4 = f32x4{v == 0 ? e : v4[0], v == 1 ? e : v4[1], v == 2 ? e : v4[2], v == 3 ? e : v4[3]};
        }
      }
      if (whole) {
        *reinterpret_cast<f32x4*>(dst) = v4;
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (n + v < N) dst[v] = v4[v];
      }
    }
  }
}

struct PoolArgs {
  const float* p;  // [B][Tf][2][3H]: blocks h~, o, f
  float* out;      // [B][Tf][2H]: stacked (forward then backward) or interleaved (2k + dir)
  int B, Tf, H, interleave;
};

// fo-pool h_t = f_t h_{t-1} + (1 - f_t) tanh(a_h), z_t = sigmoid(a_o) h_t, over the frames in the
// direction's own order.  The recurrence is linear in h, so the frames go in segments of PU, a thread
// each: it runs its segment from h = 0, keeping the gates in registers, the segments' (product of f, end
// value) chain through LDS, and it runs it again from where the segment before ends.  PC channels by
// PS segments of PU frames per block; longer sequences take further passes of PS segments.  Sequences of up to
// 16, 4 and 1 frames are one segment of 16, 4 and 1 (2048 streams of one frame, l = 20, r = 64, with 8 segments
// of 16: 829 us a call, 480 with a thread per channel, 334 so).  Bound: the reads of p; a
// thread per channel over all frames took 37 us for one stream of 256 frames, the loads' latency
// sixteen times, so 6.8;
// 32 streams of 512, 1280 channels: 262 -> 185 us.
constexpr int NTP = 256;
template <int PS, int PU>
__global__ __launch_bounds__(NTP) void qrnn_pool(const PoolArgs a) {
  constexpr int PC = NTP / PS;
  __shared__ float s_f[PS][PC], s_h[PS][PC];
  const int c = threadIdx.x % PC, seg = threadIdx.x / PC;
  const int k = blockIdx.x * PC + c;
  const int b = blockIdx.y >> 1, dir = blockIdx.y & 1;
  const bool on = k < a.H;
  const size_t fstride = (size_t)6 * a.H;  // floats per frame of p
  const float* base = a.p + (size_t)b * a.Tf * fstride + (size_t)dir * 3 * a.H + (on ? k : 0);
  float* ob = a.out + (size_t)b * a.Tf * 2 * a.H + (a.interleave ? 2 * k + dir : dir * a.H + k);
  float carry = 0.f;  // h before this pass
  for (int s0 = 0; s0 < a.Tf; s0 += PS * PU) {
    const int first = s0 + seg * PU;
    float ah[PU], ao[PU], af[PU];
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int s = min(first + u, a.Tf - 1), t = dir ? a.Tf - 1 - s : s;
      const float* q = base + (size_t)t * fstride;
      ah[u] = q[0];
      ao[u] = q[a.H];
      af[u] = q[2 * a.H];
    }
    float pf = 1.f, h = 0.f;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const float f = wnk::sigmoid_f(af[u]);
      ah[u] = (1.f - f) * wnk::tanh_f(ah[u]);
      af[u] = f;
      if (first + u < a.Tf) {
        h = f * h + ah[u];
        pf *= f;
      }
    }
    __syncthreads();  // the pass before has read its values
    s_f[seg][c] = pf;
    s_h[seg][c] = h;
    __syncthreads();
    h = carry;
#pragma unroll
    for (int g = 0; g < PS; ++g) {
      if (g == seg) carry = h;
      h = s_f[g][c] * h + s_h[g][c];
    }
    const float next = h;
    h = carry;
    carry = next;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int s = first + u;
      if (s < a.Tf && on) {
        const int t = dir ? a.Tf - 1 - s : s;
        h = af[u] * h + ah[u];
        ob[(size_t)t * 2 * a.H] = wnk::sigmoid_f(ao[u]) * h;
      }
    }
  }
}

// Upsampling by repetition: cond[b][tau][:] = src[b][floor(tau fr / ar)][:], in runs of 1024 pieces of the
// output per block, so that the blocks in flight write one moving window of memory, and past the caches.
// Bound: the write of the output.  Measured, 32 streams x 2 s at l = 20, r = 64 (10.5 GB): 1673 us, 6.3 TB/s
// (a fill reaches 6.8); a block per source frame, each writing its 62 rows (640 KB), 1970 us; the same
// window with plain stores 2010.
constexpr int RU = 4;
template <class V>
__global__ __launch_bounds__(256) void cond_repeat(const V* src, V* cond, long long block0, int B, int Tf, int T, int C,
                                               int fr, int ar) {
  const long long n = (long long)B * T * C, i0 = (block0 + blockIdx.x) * (256 * RU);
  const bool narrow = (long long)T * fr < 1LL << 32;
  // the block's first row (stream b0, step tau0) and piece of it
  const long long row0 = i0 / C;
  const unsigned c0 = (unsigned)(i0 - row0 * C);
  const long long b0 = row0 / T;
  const unsigned tau0 = (unsigned)(row0 - b0 * T);
  V v[RU];
#pragma unroll
  for (int u = 0; u < RU; ++u) {
    const unsigned at = 256 * u + threadIdx.x;
    if (i0 + at < n) {
      const unsigned l = c0 + at, r = l / (unsigned)C, c = l - r * (unsigned)C;
      const unsigned s = tau0 + r, q = s / (unsigned)T, tau = s - q * (unsigned)T;
      const unsigned t = narrow ? tau * (unsigned)fr / (unsigned)ar : (unsigned)((unsigned long long)tau * fr / ar);
      v[u] = src[((size_t)(b0 + q) * Tf + t) * C + c];
    }
  }
#pragma unroll
  for (int u = 0; u < RU; ++u) {
    const long long i = i0 + 256 * u + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(v[u], cond + i);
  }
}

size_t align_up(size_t v, size_t al) { return (v + al - 1) / al * al; }

struct CondLayout {
  size_t p_off, z1_off, c_off, total;
};
CondLayout cond_layout(const wn_cond* c, int B, int Tf) {
  CondLayout l;
  const size_t frames = (size_t)B * Tf;
  l.p_off = 0;
  l.z1_off = align_up(l.p_off + frames * 6 * (size_t)std::max(c->h1, c->h2) * 4, 256);
  l.c_off = align_up(l.z1_off + frames * 2 * (size_t)c->h1 * 4, 256);
  l.total = align_up(l.c_off + frames * 2 * (size_t)c->h2 * 4, 256);
  return l;
}

class DeviceScope {
 public:
  explicit DeviceScope(int dev) {
    ok_ = hipGetDevice(&prev_) == hipSuccess;
    if (ok_ && prev_ != dev) ok_ = hipSetDevice(dev) == hipSuccess;
  }
  ~DeviceScope() {
    int cur = -1;
    if (hipGetDevice(&cur) == hipSuccess && cur != prev_) (void)hipSetDevice(prev_);
  }
  bool ok() const { return ok_; }

 private:
  int prev_ = 0;
  bool ok_ = false;
};

hipError_t run_layer(const float* x, int B, int Tf, int cin, int cinp, int H, const u16* w, const float* wf,
                     const float* b, float* p, float* out, int interleave, hipStream_t st) {
  GateArgs g{x, w, wf, b, p, B, Tf, cin, cinp, 3 * H};
  const bool vx = cin % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
  // 128 x 128 tiles where they fill the chip twice (two blocks share a CU), else 64 x 64: one
  // stream of 256 frames, second layer, 120 blocks of 128 x 128 on fp32 MFMA 85 us, 480 of 64 x 64 41 us.
  auto blocks = [&](int t) { return dim3((unsigned)((B * Tf + t - 1) / t), (unsigned)((3 * H + t - 1) / t), 2); };
  const dim3 big = blocks(128), small = blocks(64);
  if ((size_t)big.x * big.y * 2 >= 512) {
    if (vx) hipLaunchKernelGGL((qrnn_gate_gemm<128, true>), big, dim3(NTG), 0, st, g);
    else hipLaunchKernelGGL((qrnn_gate_gemm<128, false>), big, dim3(NTG), 0, st, g);
  } else {
    if (vx) hipLaunchKernelGGL((qrnn_gate_gemm<64, true>), small, dim3(NTG), 0, st, g);
    else hipLaunchKernelGGL((qrnn_gate_gemm<64, false>), small, dim3(NTG), 0, st, g);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  PoolArgs pa{p, out, B, Tf, H, interleave};
  auto pool = [&](auto kernel, int segments) {
    const int pc = NTP / segments;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((H + pc - 1) / pc), (unsigned)(2 * B)), dim3(NTP), 0, st, pa);
  };
  if (Tf <= 1) pool(qrnn_pool<1, 1>, 1);
  else if (Tf <= 4) pool(qrnn_pool<1, 4>, 1);
  else if (Tf <= 16) pool(qrnn_pool<1, 16>, 1);
  else pool(qrnn_pool<8, 16>, 8);
  return hipGetLastError();
}

// [2][n][2][cin] -> [2][n][2][cinp], zeros in inputs cin..cinp-1 of each tap.
std::vector<float> pad_taps(const float* w, int n, int cin, int cinp) {
  std::vector<float> out((size_t)2 * n * 2 * cinp, 0.f);
  for (size_t row = 0; row < (size_t)2 * n * 2; ++row)
    std::memcpy(out.data() + row * cinp, w + row * cin, (size_t)cin * sizeof(float));
  return out;
}

// Device address of `scratch` on device dev (the current device), looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

int scratch_address(int dev, void** out) {
  if (dev < 0 || dev >= kMaxDevices) return wn_set_last_error(WN_EUNSUPPORTED, "device index beyond 63");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return wn_set_last_error(WN_EHIP, "hipGetSymbolAddress of the scratch array failed");
    g_scratch_addr[dev] = p;
  }
  *out = g_scratch_addr[dev];
  return WN_OK;
}

// The three kernels of one call, with the scratch at ws (cond_layout(c, B, n_frames) bytes).
int run_condition(wn_cond* c, int B, int n_frames, const float* features, int T, float* cond, char* ws,
                  hipStream_t st) {
  const CondLayout l = cond_layout(c, B, n_frames);
  float* p = reinterpret_cast<float*>(ws + l.p_off);
  float* z1 = reinterpret_cast<float*>(ws + l.z1_off);
  float* cf = reinterpret_cast<float*>(ws + l.c_off);
  hipError_t e = run_layer(features, B, n_frames, c->F, c->cinp1, c->h1, c->w1, c->wf1, c->b1, p, z1, 0, st);
  if (e == hipSuccess) e = run_layer(z1, B, n_frames, 2 * c->h1, c->cinp2, c->h2, c->w2, c->wf2, c->b2, p, cf, 1, st);
  if (e == hipSuccess) {
    const int C = 2 * c->h2;
    const bool wide = C % 4 == 0 && reinterpret_cast<uintptr_t>(cond) % 16 == 0;
    const int per = wide ? C / 4 : C;
    // (launches of up to 2^22 blocks: the blocks walking over the output in a loop took 2200 us against 1670)
    const long long blocks = ((long long)B * T * per + 256 * RU - 1) / (256 * RU);
    for (long long b0 = 0; b0 < blocks; b0 += 1 << 22) {
      const dim3 grid((unsigned)std::min<long long>(1 << 22, blocks - b0));
      if (wide)
        hipLaunchKernelGGL(cond_repeat<f32x4>, grid, dim3(256), 0, st, reinterpret_cast<const f32x4*>(cf),
                           reinterpret_cast<f32x4*>(cond), b0, B, n_frames, T, per, c->fr, c->ar);
      else
        hipLaunchKernelGGL(cond_repeat<float>, grid, dim3(256), 0, st, cf, cond, b0, B, n_frames, T, per, c->fr, c->ar);
    }
    e = hipGetLastError();
  }
  if (e != hipSuccess) return wn_set_last_error(WN_EHIP, hipGetErrorString(e));
  return WN_OK;
}

// Checks shared by wn_condition and wn_condition_static (all but the workspace).
int check_condition(const wn_cond* c, int B, int n_frames, const float* features, int T, const float* cond) {
  if (!c) return wn_set_last_error(WN_EINVAL, "null handle");
  if (B < 1 || n_frames < 1 || T < 0) return wn_set_last_error(WN_EINVAL, "B and n_frames must be >= 1, T >= 0");
  if (T == 0) return WN_OK;
  if (!features || !cond) return wn_set_last_error(WN_EINVAL, "null pointer");
  if ((long long)B * n_frames > (1LL << 31) - 1) return wn_set_last_error(WN_EINVAL, "B * n_frames too large");
  if ((long long)(T - 1) * c->fr / c->ar >= n_frames)
    return wn_set_last_error(WN_EINVAL, "audio steps beyond the last frame");
  return WN_OK;
}

}  // namespace

extern "C" {

int wn_cond_create(const wn_cond_config* cfg, const wn_cond_weights* w, wn_cond** out) {
  wn_clear_last_error();
  if (!cfg || !w || !out || !w->w1 || !w->b1 || !w->w2 || !w->b2) return wn_set_last_error(WN_EINVAL, "null argument");
  if (cfg->n_features < 1 || cfg->n_features > 4096) return wn_set_last_error(WN_EINVAL, "n_features must be 1..4096");
  if (cfg->h1 < 1 || cfg->h1 > 4096) return wn_set_last_error(WN_EINVAL, "h1 must be 1..4096");
  if (cfg->n_layers < 1 || cfg->r < 1 || (long long)cfg->n_layers * cfg->r > 8192)
    return wn_set_last_error(WN_EINVAL, "n_layers * r must be 1..8192");
  if (cfg->frame_rate < 1 || cfg->audio_rate < 1) return wn_set_last_error(WN_EINVAL, "rates must be >= 1");
  wn_cond* c = new (std::nothrow) wn_cond();
  if (!c) return wn_set_last_error(WN_ENOMEM, "host allocation");
  c->F = cfg->n_features;
  c->h1 = cfg->h1;
  c->h2 = cfg->n_layers * cfg->r;
  c->fr = cfg->frame_rate;
  c->ar = cfg->audio_rate;
  if (hipGetDevice(&c->device) != hipSuccess) {
    delete c;
    return wn_set_last_error(WN_EHIP, "hipGetDevice failed");
  }
  {
    const int rc = scratch_address(c->device, &c->scratch);
    if (rc != WN_OK) {
      delete c;
      return rc;
    }
  }
  c->cinp1 = (c->F + 31) / 32 * 32;
  c->cinp2 = (2 * c->h1 + 31) / 32 * 32;
  std::vector<float> w1p, w2p;
  try {
    w1p = pad_taps(w->w1, 3 * c->h1, c->F, c->cinp1);
    w2p = pad_taps(w->w2, 3 * c->h2, 2 * c->h1, c->cinp2);
  } catch (const std::bad_alloc&) {
    delete c;
    return wn_set_last_error(WN_ENOMEM, "host allocation");
  }
  const size_t n_b1 = (size_t)2 * 3 * c->h1, n_b2 = (size_t)2 * 3 * c->h2;
  // split weights, biases, and the fp32 weights they are split from
  const size_t o_w2 = align_up(w1p.size() * 6, 256), o_b1 = align_up(o_w2 + w2p.size() * 6, 256);
  const size_t o_b2 = align_up(o_b1 + n_b1 * 4, 256), o_f = align_up(o_b2 + n_b2 * 4, 256);
  const size_t total = align_up(o_f + (w1p.size() + w2p.size()) * 4, 256);
  hipError_t e = hipMalloc(&c->dmem, total);
  if (e != hipSuccess) {
    delete c;
    return e == hipErrorOutOfMemory ? wn_set_last_error(WN_ENOMEM, "hipMalloc of weights")
                                    : wn_set_last_error(WN_EHIP, hipGetErrorString(e));
  }
  char* d = static_cast<char*>(c->dmem);
  auto upload = [&](size_t off, const float* src, size_t n) {
    if (e == hipSuccess) e = hipMemcpy(d + off, src, n * 4, hipMemcpyHostToDevice);
  };
  auto split = [&](size_t off, size_t from, const std::vector<float>& w) {
    upload(from, w.data(), w.size());
    if (e != hipSuccess) return;
    hipLaunchKernelGGL(split_weights, dim3((unsigned)((w.size() / 4 + 255) / 256)), dim3(256), 0, nullptr,
                       reinterpret_cast<const float*>(d + from), reinterpret_cast<u16*>(d + off), w.size());
    e = hipGetLastError();
  };
  split(0, o_f, w1p);
  split(o_w2, o_f + w1p.size() * 4, w2p);
  upload(o_b1, w->b1, n_b1);
  upload(o_b2, w->b2, n_b2);
  if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  if (e != hipSuccess) {
    (void)hipFree(c->dmem);
    delete c;
    return wn_set_last_error(WN_EHIP, hipGetErrorString(e));
  }
  c->w1 = reinterpret_cast<const u16*>(d);
  c->w2 = reinterpret_cast<const u16*>(d + o_w2);
  c->wf1 = reinterpret_cast<const float*>(d + o_f);
  c->wf2 = c->wf1 + w1p.size();
  c->b1 = reinterpret_cast<const float*>(d + o_b1);
  c->b2 = reinterpret_cast<const float*>(d + o_b2);
  *out = c;
  return WN_OK;
}

size_t wn_cond_workspace_bytes(const wn_cond* c, int32_t B, int32_t n_frames) {
  if (!c || B < 1 || n_frames < 1) return 0;
  return cond_layout(c, B, n_frames).total;
}

int wn_condition(wn_cond* c, int32_t B, int32_t n_frames, const float* features, int32_t T, float* cond,
                 void* workspace, size_t ws_bytes, void* stream) {
  wn_clear_last_error();
  int rc = check_condition(c, B, n_frames, features, T, cond);
  if (rc != WN_OK || T == 0) return rc;
  if (!workspace) return wn_set_last_error(WN_EINVAL, "null pointer");
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
    return wn_set_last_error(WN_EINVAL, "workspace must be 256-byte aligned");
  if (ws_bytes < cond_layout(c, B, n_frames).total) return wn_set_last_error(WN_EINVAL, "workspace too small");
  DeviceScope scope(c->device);
  if (!scope.ok()) return wn_set_last_error(WN_EHIP, "cannot select the handle's device");
  return run_condition(c, B, n_frames, features, T, cond, static_cast<char*>(workspace),
                       static_cast<hipStream_t>(stream));
}

int wn_condition_static(wn_cond* c, int32_t B, int32_t n_frames, const float* features, int32_t T, float* cond,
                        void* stream) {
  wn_clear_last_error();
  int rc = check_condition(c, B, n_frames, features, T, cond);
  if (rc != WN_OK || T == 0) return rc;
  if (cond_layout(c, B, n_frames).total > WN_COND_SCRATCH_BYTES)
    return wn_set_last_error(WN_EINVAL, "B * n_frames needs more scratch than the static array holds "
                                        "(wn_cond_workspace_bytes > WN_COND_SCRATCH_BYTES)");
  DeviceScope scope(c->device);
  if (!scope.ok()) return wn_set_last_error(WN_EHIP, "cannot select the handle's device");
  return run_condition(c, B, n_frames, features, T, cond, static_cast<char*>(c->scratch),
                       static_cast<hipStream_t>(stream));
}

void wn_cond_destroy(wn_cond* c) {
  if (!c) return;
  {
    DeviceScope scope(c->device);
    if (c->dmem) (void)hipFree(c->dmem);
  }
  delete c;
}

}  // extern "C"
