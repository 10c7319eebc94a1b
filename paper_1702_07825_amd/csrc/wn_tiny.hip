// Generation with the smallest models (r = 16, s = 32, up to 8 layers), gfx950: one workgroup per stream
// with every weight resident in the CU, W_skip, W_relu and W_out (64 floats per thread) in VGPRs, the
// layers' small matrices and the embedding in LDS.  (The per-stream kernel reads them from L2 in every
// phase of a step: 7.3 us/step at l = 4.)
//
// Per step (Deep Voice, arXiv 1702.07825, Appendix A.1), 16 waves:
//   wave 0      x0 from the sample, then the layers one after the other without a barrier: a quad of lanes
//               holds gate pair c and row c of W_res, each lane four of the 16 inputs; h and x go through
//               LDS, which a wave's accesses use in order
//   waves 0-7   the skip sum of all layers' h, 16 lanes a row
//   waves 8-15  load the next step's history rows and conditioning (issued a step before) beside the chain,
//               store this step's rows, and beside the logits compute W_prev x[t + 1 - d] + B + L, the
//               off-chain half of Section 5.1
//   all         z_a, 4 lanes a row; the logits, 16 lanes by 4 rows
//   wave 0      the draw
// with four LDS barriers.  Histories and state have the per-stream kernel's layout.  Bound: the serial
// chain of LDS round trips, reductions and barriers.  Measured, l = 4, one stream: 2.8
// us/step.
#include "wn_tiny.h"
#include "wn_wave.h"

#include "wn.h"

namespace {

using namespace wnk;

constexpr int R = 16, S = 32, A = WN_A, NT = 1024, LM = WN_TINY_MAX_LAYERS;

// Weight i of a matrix whose rows have `cols` inputs, in fp32.
template <typename WT>
__device__ __forceinline__ float weight(const void* w, const float* scale, size_t i, int cols) {
  if constexpr (sizeof(WT) == 4) return static_cast<const float*>(w)[i];
  else if constexpr (sizeof(WT) == 2) return __uint_as_float((unsigned)static_cast<const uint16_t*>(w)[i] << 16);
  else return (float)static_cast<const int8_t*>(w)[i] * scale[i / cols];
}
__device__ __forceinline__ float dot4(float4 w, float4 x) {
  return fmaf(w.w, x.w, fmaf(w.z, x.z, fmaf(w.y, x.y, w.x * x.x)));
}
__device__ __forceinline__ void wave_order() { asm volatile("" ::: "memory"); }
// The thread's index, anew at each use: addresses made from it as a loop invariant would be spilled.
__device__ __forceinline__ int tid_now() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <typename WT>
__global__ __launch_bounds__(NT) void wn_tiny_kernel(const WnStreamArgs g) {
  __shared__ __align__(16) float s_wc[LM][2][R][R], s_wr[LM][R][R], s_wp[LM][2][R][R];  // [layer](tanh, sigmoid)[row][input]
  __shared__ __align__(16) float s_x[LM][R], s_h[LM][R], s_hx[LM][R];  // x_{j-1}, h_j, x_{j-1}[t + 1 - d]
  __shared__ float s_pre[LM][2 * R], s_cd[LM][2 * R], s_bg[LM][2 * R], s_br[LM][R];
  __shared__ __align__(16) float s_q[S], s_z[A], s_lg[A];
  __shared__ __align__(16) float s_e[A][R];
  __shared__ int s_stop;
  const int L = g.d.L, T = g.io.T, b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* const hist = g.ws.hist + (size_t)b * g.d.hist_len;
  int64_t* const state = g.ws.state + WN_STATE_WORDS * (size_t)b;
  const float* const cond = g.io.cond + (size_t)b * T * L * 2 * R;

  for (int i = tid; i < L * 2 * R * R; i += NT) {
    (&s_wc[0][0][0][0])[i] = weight<WT>(g.w.w_cur, g.w.s_cur, i, R);
    (&s_wp[0][0][0][0])[i] = weight<WT>(g.w.w_prev, g.w.s_prev, i, R);
  }
  for (int i = tid; i < L * R * R; i += NT) (&s_wr[0][0][0])[i] = weight<WT>(g.w.w_res, g.w.s_res, i, R);
  for (int i = tid; i < L * 2 * R; i += NT) (&s_bg[0][0])[i] = g.w.b_gate[i];
  for (int i = tid; i < L * R; i += NT) (&s_br[0][0])[i] = g.w.b_res[i];
  for (int i = tid; i < A * R; i += NT) s_e[i / R][i % R] = weight<WT>(g.w.embed, g.w.s_embed, i, R) + g.w.b_embed[i % R];
  // skip row tid / 16, input tid % 16 of every layer; z_a row tid / 4, inputs 8 (tid % 4) ..; logits rows
  // 4 (tid / 16) .., inputs 4 (tid % 16 + 16 c) ..
  float wk[LM], wz[8], wo[4][16];
#pragma unroll
  for (int j = 0; j < LM; ++j)
    wk[j] = tid < 512 && j < L ? weight<WT>(g.w.w_skip, g.w.s_skip, ((size_t)j * S + tid / 16) * R + tid % 16, R) : 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) wz[k] = weight<WT>(g.w.w_relu, g.w.s_relu, (size_t)(tid / 4) * S + 8 * (tid % 4) + k, S);
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int k = 0; k < 16; ++k)
      wo[r][k] = weight<WT>(g.w.w_out, g.w.s_out, (size_t)(4 * (tid / 16) + r) * A + 4 * (tid % 16 + 16 * (k / 4)) + k % 4, A);
  const float bq = g.w.b_skip[tid / 16 % S], bz = g.w.b_relu[tid / 4];
  // this lane's logit after the reduction: row 2 (bit 3) + (bit 2) of its group of four
  const int orow = 4 * (tid / 16) + ((tid >> 3) & 1) * 2 + ((tid >> 2) & 1);
  const float bo = g.w.b_out[orow];

  const int64_t tg0 = g.io.reset ? 0 : state[0];
  int y1 = g.io.reset ? g.io.init_sample : (int)state[1], y2 = g.io.reset ? -1 : (int)state[2];
  if (g.io.reset)
    for (int i = tid; i < g.d.hist_len / 4; i += NT) reinterpret_cast<float4*>(hist)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (tid == 0) s_stop = 0;
  __syncthreads();  // the cleared histories too

  // waves 8 on: piece p of the next step's inputs, conditioning element p and (p < 16 L) history element p
  const int p = tid - 512;
  const bool cd_on = p >= 0 && p < L * 2 * R, hx_on = p >= 0 && p < L * R;
  const int hj = hx_on ? p / R : 0, hd = g.d.dil[hj];
  float* const hrow = hist + g.d.hoff[hj] + (hx_on ? p % R : 0);  // this thread alone uses its element of the history
  auto load_cond = [&](int t) { return cd_on && t < T ? __builtin_nontemporal_load(cond + (size_t)t * L * 2 * R + p) : 0.f; };
  auto pre_of = [&] {  // s_pre = W_prev s_hx + B + s_cd, 4 lanes a row
    const int p = tid_now() - 512;
    for (int r = p >> 2; r < L * 2 * R; r += 128) {
      const int j = r / (2 * R), row = r % (2 * R), i = p & 3;
      const float v = gsum4(dot4(*reinterpret_cast<const float4*>(&s_wp[j][0][0][0] + row * R + 4 * i),
                                 *reinterpret_cast<const float4*>(&s_hx[j][4 * i])));
      if (i == 0) s_pre[j][row] = v + (s_bg[j][row] + s_cd[j][row]);
    }
  };
  // the first step's: every history row is final
  if (hx_on) (&s_hx[0][0])[p] = hrow[(int)(tg0 % hd) * R];
  if (cd_on) (&s_cd[0][0])[p] = load_cond(0);
  float cnext = load_cond(1);
  int hslot = (int)(tg0 % hd);  // of step t
  __syncthreads();
  if (wave >= 8) pre_of();

  // wave 0: quad c = lane / 4, inputs 4 i ..
  const int c = (lane >> 2) & 15, i4 = 4 * (lane & 3);
  float u64 = 0.f;  // lane k: the uniform of step t - t % 64 + k
  auto prev_row = [&](int y) {  // E_prev[y], loaded when y is drawn and used a step later
    return g.w.embed_prev && y >= 0 ? weight<WT>(g.w.embed_prev, g.w.s_embed_prev, (size_t)(y > A - 1 ? A - 1 : y) * R + c, R) : 0.f;
  };
  float ep = prev_row(y2), ep1 = prev_row(y1);  // of y_{t-2} and y_{t-1}
  int stop = 0;  // an abort request, read one step ahead
  __syncthreads();

  for (int t = 0; t < T; ++t) {
    if (wave == 0) {
      if ((t & 63) == 0) u64 = t + lane < T ? g.io.u[(size_t)b * T + t + lane] : 0.f;
      float x = s_e[y1 < 0 ? 0 : (y1 > A - 1 ? A - 1 : y1)][c] + ep;
      ep = ep1;
#pragma unroll
      for (int j = 0; j < LM; ++j) {
        if (j < L) {
          if ((lane & 3) == 0) s_x[j][c] = x;
          wave_order();
          const float4 x4 = *reinterpret_cast<const float4*>(&s_x[j][i4]);
          const float ah = gsum4(dot4(*reinterpret_cast<const float4*>(&s_wc[j][0][c][i4]), x4)) + s_pre[j][c];
          const float ag = gsum4(dot4(*reinterpret_cast<const float4*>(&s_wc[j][1][c][i4]), x4)) + s_pre[j][R + c];
          const float h = g.w.approx_nl ? tanh_paper(ah) * sigmoid_paper(ag) : gate_pair(ah, ag, lane);
          if ((lane & 3) == 0) s_h[j][c] = h;
          wave_order();
          if (j + 1 < L) {
            const float4 h4 = *reinterpret_cast<const float4*>(&s_h[j][i4]);
            x = x + (gsum4(dot4(*reinterpret_cast<const float4*>(&s_wr[j][c][i4]), h4)) + s_br[j][c]);
          }
        }
      }
    } else if (wave >= 8) {
      // x_{j-1}[t + 1 - d] of the layers with d >= 2 (slot (t + 1) mod d), and the conditioning of t + 1
      const int p = tid_now() - 512;
      if (hx_on && hd >= 2) (&s_hx[0][0])[p] = hrow[(hslot + 1 == hd ? 0 : hslot + 1) * R];
      if (cd_on) (&s_cd[0][0])[p] = cnext;
      cnext = load_cond(t + 2);
    } else if (tid == 64) {
      if (t == 0) stop = abort_requested(g.io.abort_flag);
      if ((t & (WN_ABORT_CHECK - 1)) == 0 && stop) {
        atomicCAS(g.ws.status, 0, (int)WN_EABORTED);
        s_stop = 1;
      }
      if ((t & (WN_ABORT_CHECK - 1)) == WN_ABORT_CHECK - 1) stop = abort_requested(g.io.abort_flag);
    }
    lds_barrier();
    if (s_stop) break;
    if (wave < 8) {
      const int tid = tid_now();
      float v = 0.f;
#pragma unroll
      for (int j = 0; j < LM; ++j)
        if (j < L) v = fmaf(wk[j], s_h[j][tid % 16], v);
      v = gsum16(v);
      if (tid % 16 == 0) s_q[tid / 16] = fmaxf(v + bq, 0.f);
    } else if (hx_on) {
      // x_{j-1}[t] into its slot, and with d = 1 straight to the next step
      const int p = tid_now() - 512;
      const float x = (&s_x[0][0])[p];
      hrow[hslot * R] = x;
      if (hd == 1) (&s_hx[0][0])[p] = x;
      hslot = hslot + 1 == hd ? 0 : hslot + 1;
    }
    lds_barrier();
    {
      const int tid = tid_now();
      const float4 q0 = *reinterpret_cast<const float4*>(&s_q[8 * (tid % 4)]);
      const float4 q1 = *reinterpret_cast<const float4*>(&s_q[8 * (tid % 4) + 4]);
      const float v = gsum4(dot4(make_float4(wz[0], wz[1], wz[2], wz[3]), q0) + dot4(make_float4(wz[4], wz[5], wz[6], wz[7]), q1));
      if (tid % 4 == 0) s_z[tid / 4] = fmaxf(v + bz, 0.f);
    }
    lds_barrier();
    {
      const int tid = tid_now();
      float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 z = *reinterpret_cast<const float4*>(&s_z[4 * (tid % 16 + 16 * k)]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          v[r] = fmaf(wo[r][4 * k + 3], z.w, fmaf(wo[r][4 * k + 2], z.z, fmaf(wo[r][4 * k + 1], z.y, fmaf(wo[r][4 * k], z.x, v[r]))));
      }
      // over 16 lanes: bit 3 keeps rows 0, 1 or 2, 3 (partner 15 - i), bit 2 one of the two (7 - i)
      const bool u3 = (tid & 8) != 0, u2 = (tid & 4) != 0;
      const float k0 = (u3 ? v[2] : v[0]) + dpp<0x140>(u3 ? v[0] : v[2]);
      const float k1 = (u3 ? v[3] : v[1]) + dpp<0x140>(u3 ? v[1] : v[3]);
      const float k = gsum4((u2 ? k1 : k0) + dpp<0x141>(u2 ? k0 : k1));
      if ((tid & 3) == 0) s_lg[4 * (tid / 16) + ((tid >> 3) & 1) * 2 + ((tid >> 2) & 1)] = k + bo;
      if (wave >= 8) pre_of();
    }
    lds_barrier();
    if (wave == 0) {
      const float4 lv = *reinterpret_cast<const float4*>(&s_lg[4 * lane]);
      const float u = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, u64), t & 63));
      const int y = g.w.approx_nl ? wave_draw<true>(lv, u, g.io.smode, g.io.inv_t, g.io.top_k, lane)
                                  : wave_draw<false>(lv, u, g.io.smode, g.io.inv_t, g.io.top_k, lane);
      if (lane == 0) g.io.y_out[(size_t)b * T + t] = y;
      y2 = y1;
      y1 = y;
      ep1 = prev_row(y);
    }
  }
  // after an abort the state stays as it was (the next call must start from zero)
  if (tid == 0 && !s_stop) {
    state[0] = tg0 + T;
    state[1] = y1;
    state[2] = y2;
  }
}

}  // namespace

bool wn_tiny_supported(int R_, int S_, int L) { return R_ == R && S_ == S && L <= LM; }

hipError_t wn_tiny_launch(const WnStreamArgs& g, hipStream_t stream) {
  const dim3 grid(g.io.B), block(NT);
  if (g.w.bf16) hipLaunchKernelGGL(wn_tiny_kernel<uint16_t>, grid, block, 0, stream, g);
  else if (g.w.i8) hipLaunchKernelGGL(wn_tiny_kernel<int8_t>, grid, block, 0, stream, g);
  else hipLaunchKernelGGL(wn_tiny_kernel<float>, grid, block, 0, stream, g);
  return hipGetLastError();
}
