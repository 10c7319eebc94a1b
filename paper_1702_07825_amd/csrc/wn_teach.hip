// Teacher forcing, parallel over time, gfx950.
//
// With the samples given, nothing in a step waits for the step before it: layer j is a width-2 dilated
// causal convolution of the whole sequence (Deep Voice, arXiv 1702.07825, Appendix A.1), so a call is l
// passes over all of its rows (one row per stream and step) instead of T serial steps.  Each pass is
// matrix work on [rows x r] tiles: the gate [2r x 2r], the residual [r x r] and the skip projection
// [s x r] of a tile in one kernel, on fp32 MFMA (v_mfma_f32_16x16x4f32) with every sum in fp32, whatever
// the model's storage (bf16 weights are exact in fp32, int8 ones are code * scale rounded to fp32).
//
// A call runs in chunks of up to 16384 rows (512 tiles of up to 32, two to a CU; at r = 128 12288 rows, 256
// tiles of up to 48), each one launch of teach_pass, which takes its tiles through all layers and the head;
// a call of at most kSmallT steps takes the small_* kernels instead.  Both do a row's sums in the same
// order, so its logits do not depend on how a sequence is cut into calls, chunks or tiles.
//
// The dilation histories in the workspace are read and written in the layout of the kernel family that
// generates with this handle and batch (ring_load, ring_store), so calls of either kind continue each
// other's state.  Layer j reads x_{j-1}[t - d] from the chunk itself, or from the history where t - d lies
// before it.
#include "wn_mfma.h"
#include "wn_teach.h"
#include "wn_wave.h"

#include "wn.h"

#include <algorithm>
#include <type_traits>

namespace {

using namespace wnk;

constexpr int A = WN_A;
constexpr int kSmallT = 16;  // longest call that the small_* kernels take: one tile of rows

__device__ __forceinline__ f32x4 ldg4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ void st4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
// Loads issued before this point stay before it.
__device__ __forceinline__ void issued() { __builtin_amdgcn_sched_barrier(0); }
// This lane's index, anew at each use: as a loop invariant, every address made from it would be computed
// before the layer loop and spilled there (40-180 registers; a reload from scratch memory also waits for
// every load in flight).
__device__ __forceinline__ unsigned lane_now() {
  unsigned l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// What a group-kernel history slot holds of a value: the sum of its two bf16 parts.
__device__ __forceinline__ f32x4 as_pair(f32x4 v) {
  uint2 hi, lo;
  split4(make_float4(v[0], v[1], v[2], v[3]), hi, lo);
  return f32x4{low_bf16(hi.x) + low_bf16(lo.x), high_bf16(hi.x) + high_bf16(lo.x),
               low_bf16(hi.y) + low_bf16(lo.y), high_bf16(hi.y) + high_bf16(lo.y)};
}

// Four channels of a history slot as they lie in memory.  The loads of all layouts are issued alike (some
// twice) and nothing looks at them until take(), so that they can stay in flight.
struct RingRow {
  uint2 w[4];
};
// Channels c .. c + 3 (c a multiple of 4) of slot `slot` of layer j's history of stream b.
__device__ __forceinline__ RingRow ring_load(const WnTeachArgs& g, int b, int j, int slot, int c) {
  const size_t row = (size_t)g.d.hoff[j] + (size_t)slot * g.d.R;  // words (or floats) into the stream's block
  const bool tiles = g.ring_kind == WN_RING_TILES, pair = g.ring_kind == WN_RING_PAIR;
  const int rep = tiles ? b / g.ring_g : b, col = b - rep * g.ring_g;
  const size_t at = tiles ? ((size_t)rep * g.d.hist_len + row) * g.ring_ns + (size_t)(c >> 4) * 16 * g.ring_ns +
                                (((c & 15) >> 2) * g.ring_ns + col) * 4
                          : (size_t)b * g.d.hist_len + row + (pair ? c / 2 : c);
  const bool words = tiles || g.ring_kind == WN_RING_TAGGED;
  const uint2* p = reinterpret_cast<const uint2*>(static_cast<const char*>(g.ring) + at * (words ? 8 : 4));
  // units of 8 bytes: words (value, tag) 0 1 2 3; fp32 pairs 0 1; hi parts 0, lo parts R / 4
  const int s1 = pair ? g.d.R / 4 : 1;
  return RingRow{{p[0], p[s1], p[words ? 2 : 0], p[words ? 3 : 0]}};
}
__device__ __forceinline__ f32x4 take(const WnTeachArgs& g, const RingRow& r) {
  if (g.ring_kind == WN_RING_F32)
    return f32x4{__uint_as_float(r.w[0].x), __uint_as_float(r.w[0].y), __uint_as_float(r.w[1].x), __uint_as_float(r.w[1].y)};
  if (g.ring_kind == WN_RING_PAIR)
    return f32x4{low_bf16(r.w[0].x) + low_bf16(r.w[1].x), high_bf16(r.w[0].x) + high_bf16(r.w[1].x),
                 low_bf16(r.w[0].y) + low_bf16(r.w[1].y), high_bf16(r.w[0].y) + high_bf16(r.w[1].y)};
  return f32x4{__uint_as_float(r.w[0].x), __uint_as_float(r.w[1].x), __uint_as_float(r.w[2].x), __uint_as_float(r.w[3].x)};
}

// The same slot written with x_{j-1} of the step whose tag (step + 1) is `tag`.
__device__ __forceinline__ void ring_store(const WnTeachArgs& g, int b, int j, int slot, int c, f32x4 v, unsigned tag) {
  const size_t row = (size_t)g.d.hoff[j] + (size_t)slot * g.d.R;
  if (g.ring_kind == WN_RING_F32) {
    st4(reinterpret_cast<float*>(g.ring) + (size_t)b * g.d.hist_len + row + c, v);
    return;
  }
  if (g.ring_kind == WN_RING_PAIR) {
    u16* p = reinterpret_cast<u16*>(reinterpret_cast<float*>(g.ring) + (size_t)b * g.d.hist_len + row);
    uint2 hi, lo;
    split4(make_float4(v[0], v[1], v[2], v[3]), hi, lo);
    *reinterpret_cast<uint2*>(p + c) = hi;
    *reinterpret_cast<uint2*>(p + g.d.R + c) = lo;
    return;
  }
  u32x4* p;
  int pad = 0;  // columns after this one that carry no stream
  if (g.ring_kind == WN_RING_TAGGED) {
    p = reinterpret_cast<u32x4*>(reinterpret_cast<unsigned long long*>(g.ring) + (size_t)b * g.d.hist_len + row + c);
  } else {
    const int rep = b / g.ring_g, col = b - rep * g.ring_g;
    if (col == g.ring_g - 1 || b == g.io.B - 1) pad = g.ring_ns - 1 - col;
    p = reinterpret_cast<u32x4*>(reinterpret_cast<unsigned long long*>(g.ring) +
                                 ((size_t)rep * g.d.hist_len + row) * g.ring_ns + (size_t)(c >> 4) * 16 * g.ring_ns +
                                 (((c & 15) >> 2) * g.ring_ns + col) * 4);
  }
  p[0] = u32x4{__float_as_uint(v[0]), tag, __float_as_uint(v[1]), tag};
  p[1] = u32x4{__float_as_uint(v[2]), tag, __float_as_uint(v[3]), tag};
  // the MFMA kernel polls whole tiles, so a replica's last stream also tags the columns without one
  for (int k = 1; k <= pad; ++k) p[2 * k] = p[2 * k + 1] = u32x4{0u, tag, 0u, tag};
}

__device__ __forceinline__ int clamp_y(int y) { return y < 0 ? 0 : (y > A - 1 ? A - 1 : y); }

// Channels c .. c + 3 of x_0 of step `at` (of the call) of stream b: E[y_{t-1}] + B_embed (+ E_prev[y_{t-2}]).
// start: where the call began (its z and w are y_{-1} and y_{-2} of the call).
__device__ __forceinline__ f32x4 embed4(const WnTeachArgs& g, const int4 start, int b, int at, int c) {
  const int32_t* y = g.io.y_in + (size_t)b * g.io.T;
  const int y1 = clamp_y(at >= 1 ? y[at - 1] : start.z);
  f32x4 v = ldg4(static_cast<const float*>(g.w.embed) + (size_t)y1 * g.d.R + c) + ldg4(g.w.b_embed + c);
  if (g.w.embed_prev) {
    const int y2 = at >= 2 ? clamp_y(y[at - 2]) : (at == 1 ? clamp_y(start.z) : min(start.w, A - 1));
    if (y2 >= 0) v += ldg4(static_cast<const float*>(g.w.embed_prev) + (size_t)y2 * g.d.R + c);
  }
  return v;
}

// x_j between tiles: words of a value and the layer's tag, stored and read at agent scope (cache policy sc1,
// as in wn_msg.h).  A word validates itself, so a reader re-reads until the tag it expects appears and
// nothing orders the words among each other (a progress word after them would need a release fence, whose
// write-back of the whole L2 by every tile and layer took as long as the products: 590 against 330 us for
// 16000 rows at l = 20, r = 64).  Offsets in words.
typedef __amdgpu_buffer_rsrc_t wnb_rsrc;
__device__ __forceinline__ wnb_rsrc buffer_of(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 ld_words(wnb_rsrc rs, unsigned at) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at * 8u), 0, 16);
}
__device__ __forceinline__ void st_words(wnb_rsrc rs, unsigned at, f32x4 v, unsigned tag) {
  const u32x4 a = {__float_as_uint(v[0]), tag, __float_as_uint(v[1]), tag};
  const u32x4 b = {__float_as_uint(v[2]), tag, __float_as_uint(v[3]), tag};
  __builtin_amdgcn_raw_buffer_store_b128(a, rs, (int)(at * 8u), 0, 16);
  __builtin_amdgcn_raw_buffer_store_b128(b, rs, (int)(at * 8u + 16u), 0, 16);
}
constexpr int kProgStride = 16;  // one progress word per 64 bytes


// How the W waves of a block share a product with N output channels over NC tiles of 16 rows: wave w
// takes the channel tiles wr + WR i and the row tiles wc + WC k.
template <int N, int NC, int W>
struct Split {
  static constexpr int NR = N / 16;
  static constexpr int WR = NR < W ? NR : W, WC = W / WR;
  static constexpr int NRT = NR / WR, NCT = (NC + WC - 1) / WC;
  int wr, wc;
  __device__ explicit Split(int wave) : wr(wave % WR), wc(wave / WR) {}
  __device__ int rt(int i) const { return wr + WR * i; }
  __device__ int ct(int k) const { return wc + WC * k; }
  // With fewer row tiles than wave columns some waves have none.
  __device__ bool on(int k) const { return NC % WC == 0 || ct(k) < NC; }
};

// Row pitch (floats) of a [rows][K] tile in LDS: 32 bytes mod 64, so that the b128 reads of 16 rows by 4
// lane groups hit every bank equally (a pitch of 16 mod 64 bytes measured half that rate).
constexpr int pitch(int K) { return K + 8; }

// Biases, conditioning, x and the skip sums join a product after it: started from them, the sums' steps
// would round at their size (with b_out of a peaked voice the logits' error was six times as large).
template <int N, int M>
__device__ __forceinline__ void clear(f32x4 (&acc)[N][M]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int k = 0; k < M; ++k) acc[i][k] = zero4();
}

// A wave's weights of N channel tiles and K inputs, as MFMA A operands: lane (n, quad) holds channel n of
// a tile, and of each 16 inputs the four at 4 quad.  They are loaded a phase ahead of their products, so
// that the loads' round trips (L2 or MALL) run beside the phase before.  The matrices are packed in this
// order (pack_tiles), so that a load reads 1 KB in a run: 16 rows of 64 bytes each, as they lie in the
// row-major matrix, made the loads the bound (the skip product's
// phase 7400 clocks per layer against 3300 packed, r = 64, s = 256).
template <int K, int N>
struct Frag {
  f32x4 f[N][K / 16];
  // w: a packed matrix of rows of ld inputs; channel tile i is the matrix's 16 rows from row(i) on, at inputs
  // k .. k + K - 1
  template <class Row>
  __device__ __forceinline__ void load(const float* w, int ld, int k, Row row) {
    const unsigned lane = lane_now();
#pragma unroll
    for (int i = 0; i < N; ++i) {
      // (a wave-uniform pointer and one 32-bit lane offset: per-lane pointers, kept across the layers, spill)
      const float* p = w + (size_t)row(i) * ld + 16 * k;
#pragma unroll
      for (int k0 = 0; k0 < K / 16; ++k0) f[i][k0] = ldg4(p + 256 * k0 + 4 * lane);
    }
  }
};

// [rows][K] row-major to tiles of 16 rows by 16 inputs, lane order (rows a multiple of 16); a matrix per
// blockIdx.y.
struct PackArgs {
  struct {
    const float* src;
    float* dst;
    size_t rows;
    int K;
  } m[6];
};
__global__ __launch_bounds__(256) void pack_tiles(const PackArgs a) {
  const auto& m = a.m[blockIdx.y];
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < m.rows * m.K / 4; i += (size_t)gridDim.x * 256) {  // 16-byte pieces of dst
    const int lane = i & 63, kt = (int)((i >> 6) % (m.K / 16));
    const size_t rt = (i >> 6) / (m.K / 16);
    st4(m.dst + 4 * i, ldg4(m.src + (16 * rt + (lane & 15)) * m.K + 16 * kt + 4 * (lane >> 4)));
  }
}

// acc[i][k] += W[channel tile i] . X[row tile k]: x[k] is row n of the tile at input 4 quad, in LDS.
// Within 16 inputs the lane group `quad` of product e takes input 4 quad + e, in both operands alike, so
// one 16-byte read feeds four products.
template <int K, int N, int NCT>
__device__ __forceinline__ void mma(f32x4 (&acc)[N][NCT], const Frag<K, N>& w, const float* const (&x)[NCT]) {
#pragma unroll
  for (int k0 = 0; k0 < K / 16; ++k0) {
    f32x4 xb[NCT];
#pragma unroll
    for (int k = 0; k < NCT; ++k) xb[k] = *reinterpret_cast<const f32x4*>(x[k] + 16 * k0);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int k = 0; k < NCT; ++k)
          acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.f[i][k0][e], xb[k][e], acc[i][k], 0, 0, 0);
  }
}

// A block's pass over one layer, for tiles of 16 NC rows.
template <int R, int S, int NC, int W, bool AX>
struct Layer {
  static constexpr int P = pitch(R);
  using G = Split<R, NC, W>;  // the gate (each channel tile with its sigmoid half) and the residual
  using K = Split<S, NC, W>;  // the skip projection
  // the gate's product [W_prev | W_cur] . [x[t - d] ; x[t]] goes in runs of KB inputs
  static constexpr int KB = R < 64 ? R : 64, RUNS = 2 * R / KB;
  using GateFrag = Frag<KB, 2 * G::NRT>;
  struct ResFrag {
    Frag<R, G::NRT> w;
    f32x4 b[G::NRT];
  };
  using SkipFrag = Frag<R, 1>;  // one channel tile
  using GateAcc = f32x4[2 * G::NRT][G::NCT];
  struct GateAdd {
    f32x4 b[2 * G::NRT], l[2 * G::NRT][G::NCT];  // B and L of this lane's gate channels
  };
  using SkipAcc = f32x4[K::NRT][K::NCT];

  // run c of the gate's weights, channel tiles tanh 0, sigmoid 0, tanh 1, ..
  static __device__ __forceinline__ void load_gate(GateFrag& f, const WnTeachArgs& g, int j, int c, const G& sp) {
    f.load(c < RUNS / 2 ? g.p.prev : g.p.cur, R, c % (RUNS / 2) * KB,
           [&](int i) { return j * 2 * R + (i & 1) * R + 16 * sp.rt(i >> 1); });
  }
  // acc += runs C0 .. C1 - 1, run c in f[c & 1]; the runs after the first two are loaded here
  template <int C0, int C1>
  static __device__ __forceinline__ void gate_product(GateAcc& acc, GateFrag (&f)[2], const WnTeachArgs& g, int j,
                                                      const float* Xp, const float* Xc, const G& sp) {
#pragma unroll
    for (int c = C0; c < C1; ++c) {
      const float* x[G::NCT];
      rows(x, (c < RUNS / 2 ? Xp : Xc) + c % (RUNS / 2) * KB, sp);
      mma(acc, f[c & 1], x);
      if (c + 2 < RUNS) {
        load_gate(f[c & 1], g, j, c + 2, sp);
        issued();
      }
    }
  }
  static __device__ __forceinline__ void load_res(ResFrag& f, const WnTeachArgs& g, int j, const G& sp) {
    const int quad = lane_now() >> 4;
    f.w.load(g.p.res, R, 0, [&](int i) { return j * R + 16 * sp.rt(i); });
#pragma unroll
    for (int i = 0; i < G::NRT; ++i) f.b[i] = ldg4(g.w.b_res + (size_t)j * R + 16 * sp.rt(i) + 4 * quad);
  }
  static __device__ __forceinline__ void load_skip(SkipFrag& f, const WnTeachArgs& g, int j, int i, const K& sp) {
    f.load(g.p.skip, R, 0, [&](int) { return j * S + 16 * sp.rt(i); });
  }
  // cond: this lane's rows of the conditioning, at layer 0
  static __device__ __forceinline__ void load_add(GateAdd& add, const WnTeachArgs& g, int j, const G& sp,
                                                  const float* const (&cond)[G::NCT]) {
    const int quad = lane_now() >> 4;
    const float* bg = g.w.b_gate + (size_t)j * 2 * R;
#pragma unroll
    for (int i = 0; i < G::NRT; ++i) {
      const int c = 16 * sp.rt(i) + 4 * quad;
      add.b[2 * i] = ldg4(bg + c);
      add.b[2 * i + 1] = ldg4(bg + R + c);
#pragma unroll
      for (int k = 0; k < G::NCT; ++k) {
        const float* cr = cond[k] + (size_t)j * 2 * R + c;
        add.l[2 * i][k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(cr));  // read once
        add.l[2 * i + 1][k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(cr + R));
      }
    }
  }
  // B operand rows of a [16 NC][P] tile for this wave's row tiles
  template <class SP>
  static __device__ __forceinline__ void rows(const float* (&x)[SP::NCT], const float* X, const SP& sp) {
    const int lane = lane_now(), n = lane & 15, quad = lane >> 4;
#pragma unroll
    for (int k = 0; k < SP::NCT; ++k) x[k] = X + (16 * (sp.on(k) ? sp.ct(k) : 0) + n) * P + 4 * quad;
  }
  // H = tanh(a_h) sigmoid(a_g) of the finished sums
  static __device__ __forceinline__ void gate(float* H, const GateAcc& acc, const GateAdd& add, const G& sp) {
    const int lane = lane_now(), n = lane & 15, quad = lane >> 4;
#pragma unroll
    for (int i = 0; i < G::NRT; ++i)
#pragma unroll
      for (int k = 0; k < G::NCT; ++k) {
        const f32x4 ah = acc[2 * i][k] + (add.b[2 * i] + add.l[2 * i][k]);
        const f32x4 ag = acc[2 * i + 1][k] + (add.b[2 * i + 1] + add.l[2 * i + 1][k]);
        f32x4 h;
#pragma unroll
        for (int v = 0; v < 4; ++v) h[v] = tanh_nl<AX>(ah[v]) * sigmoid_nl<AX>(ag[v]);
        if (sp.on(k)) st4(H + (16 * sp.ct(k) + n) * P + 16 * sp.rt(i) + 4 * quad, h);
      }
  }
  // x_j = x_{j-1} + W_res h + B_res; put(m, c, v) takes channels c .. c + 3 of row m
  template <class Put>
  static __device__ __forceinline__ void residual(const ResFrag& w, const float* Xc,
                                                  const float* H, const G& sp, Put put) {
    const int lane = lane_now(), n = lane & 15, quad = lane >> 4;
    f32x4 acc[G::NRT][G::NCT];
    const float* x[G::NCT];
    rows(x, H, sp);
    clear(acc);
    mma(acc, w.w, x);
#pragma unroll
    for (int i = 0; i < G::NRT; ++i) {
      const int c = 16 * sp.rt(i) + 4 * quad;
#pragma unroll
      for (int k = 0; k < G::NCT; ++k)
        if (sp.on(k)) {
          const int m = 16 * sp.ct(k) + n;
          put(m, c, *reinterpret_cast<const f32x4*>(Xc + m * P + c) + (acc[i][k] + w.b[i]));
        }
    }
  }
  // q += W_skip h for channel tile i of this wave
  static __device__ __forceinline__ void skip(SkipAcc& q, int i, const SkipFrag& w, const float* H, const K& sp) {
    f32x4 acc[1][K::NCT];
    const float* x[K::NCT];
    rows(x, H, sp);
    clear(acc);
    mma(acc, w, x);
#pragma unroll
    for (int k = 0; k < K::NCT; ++k) q[i][k] += acc[0][k];
  }
};

// One of the head's products over a tile of 16 NC rows, W [A][K] by X [16 NC][pitch(K)] in LDS, its
// weights streamed in runs of 32 inputs, one run ahead.
template <int K, int NC, int W>
__device__ __forceinline__ void head_product(f32x4 (&acc)[A / 16 / W][NC], const float* w, const float* X, int wave) {
  constexpr int N = A / 16 / W, KB = 32;
  const int lane = threadIdx.x & 63, n = lane & 15, quad = lane >> 4;
  const float* x[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) x[k] = X + (16 * k + n) * pitch(K) + 4 * quad;
  clear(acc);
  Frag<KB, N> f[2];
  auto load = [&](int b) {
    f[b & 1].load(w, K, b * KB, [&](int i) { return 16 * (wave + W * i); });
  };
  load(0);
#pragma unroll
  for (int b = 0; b < K / KB; ++b) {
    if (b + 1 < K / KB) load(b + 1);
    issued();
    const float* xk[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) xk[k] = x[k] + b * KB;
    mma(acc, f[b & 1], xk);
  }
}

// The head of a tile: Z [16 NC][pitch(S)] holds relu(q); ZA [16 NC][pitch(A)] takes z_a.  out(m, c, v)
// takes the logits c .. c + 3 of row m.  The caller's barrier orders Z.
template <int S, int NC, int W, class Out>
__device__ __forceinline__ void head_tile(const WnTeachArgs& g, const float* Z, float* ZA, Out out) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 15, quad = lane >> 4;
  constexpr int N = A / 16 / W;
  f32x4 acc[N][NC], br[N], bo[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    br[i] = ldg4(g.w.b_relu + 16 * (wave + W * i) + 4 * quad);
    bo[i] = ldg4(g.w.b_out + 16 * (wave + W * i) + 4 * quad);
  }
  head_product<S, NC, W>(acc, g.p.relu, Z, wave);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int c = 16 * (wave + W * i) + 4 * quad;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      f32x4 v = acc[i][k] + br[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
      st4(ZA + (16 * k + n) * pitch(A) + c, v);
    }
  }
  lds_barrier();
  head_product<A, NC, W>(acc, g.p.out, ZA, wave);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int c = 16 * (wave + W * i) + 4 * quad;
#pragma unroll
    for (int k = 0; k < NC; ++k) out(16 * k + n, c, acc[i][k] + bo[i]);
  }
}

// A teach_pass block: four waves and tiles of 16 or 32 rows, two blocks to a CU, so that one block's products
// run beside the other's exchange (16000 rows, l = 20, r = 64, s = 256, when it was chosen: 345 us per call
// against 358 for one block of eight waves and 64 rows; now 331).  At r = 128 a wave's weights of a layer
// only fit its registers with eight waves: one block per CU, tiles of 16, 32 or 48 rows.
constexpr int pass_waves(int R) { return R == 128 ? 8 : 4; }
constexpr int pass_blocks(int R) { return R == 128 ? 1 : 2; }

// A chunk's rows: streams b0 .. b0 + nb - 1, steps c0 .. c0 + n - 1 of the call; row m is step m % n of
// stream m / n.
struct Chunk {
  int b0, nb, c0, n;
};

// Before a chunk's pass: one thread reads the host's abort request, the tiles' progress words and the tags
// of the chunk's x words are cleared, and at the first chunk of a stream its state moves to the end of the call; where it started goes to the
// scratch, for every chunk's pass.
__global__ __launch_bounds__(256) void teach_begin(const WnTeachArgs g, const Chunk ch) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0 && abort_requested(g.io.abort_flag)) atomicCAS(g.status, 0, (int)WN_EABORTED);
  if (i < WN_TEACH_TILES) g.prog[i * kProgStride] = 0;
  const size_t words = (size_t)ch.nb * ch.n * g.d.R;
  for (size_t k = 2 * (size_t)i; k < words; k += 2 * (size_t)gridDim.x * 256)
    for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4*>(g.x + ((size_t)s * g.rows * g.d.R + k) * 2) = u32x4{0u, 0u, 0u, 0u};
  if (ch.c0 == 0 && i < ch.nb) {
    const int b = ch.b0 + i, T = g.io.T;
    int64_t* st = g.state + WN_STATE_WORDS * (size_t)b;
    const int32_t* y = g.io.y_in + (size_t)b * T;
    const int64_t tg = g.io.reset ? 0 : st[0];
    const int y1 = g.io.reset ? g.io.init_sample : (int)st[1], y2 = g.io.reset ? -1 : (int)st[2];
    g.start[i] = make_int4((int)(unsigned)tg, (int)(tg >> 32), y1, y2);
    st[2] = T >= 2 ? clamp_y(y[T - 2]) : y1;
    st[1] = clamp_y(y[T - 1]);
    st[0] = tg + T;
  }
}

// A progress word: tile i has read every input of the layers before j once prog[i] >= j.  Waits are
// bounded; a block that gives up stores WN_ETIMEOUT, the others see the status.  The polls count only once
// every block runs (its progress word is 1 or more): while kernels of other streams hold CUs, some blocks
// may start seconds after the others.  (The words are read only then: a count of the blocks that have
// started, one atomic add each, made every launch 3 us longer.)
__device__ __forceinline__ unsigned ld_prog(const WnTeachArgs& g, int tile) {
  return __hip_atomic_load(g.prog + tile * kProgStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool gave_up(const WnTeachArgs& g, int& spins, int* fail) {
  if (++spins <= g.spin_limit && (spins & 63) != 0) return false;
  if (__hip_atomic_load(g.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
    if (spins <= g.spin_limit) return false;
    for (int k = (int)gridDim.x - 1; k >= 0; --k)
      if (ld_prog(g, k) == 0) {
        spins = 0;
        return false;
      }
    atomicCAS(g.status, 0, (int)WN_ETIMEOUT);
  }
  *fail = 1;
  return true;
}
__device__ __forceinline__ void wait_prog(const WnTeachArgs& g, int tile, unsigned need, int* fail) {
  int spins = 0;
  while (ld_prog(g, tile) < need)
    if (gave_up(g, spins, fail)) break;
}

// The chunk's rows through every layer and the head, a tile of 16 NC rows per block.  x and the skip sums
// stay on the CU (LDS and registers); what a layer needs of other tiles, x_{j-1} of d rows earlier, goes
// through three x buffers in the scratch as tagged words.  A tile sends x_j before its skip product and
// looks for its inputs after it, so the exchange runs beside that product.  Before it overwrites x_{j-3} a
// tile waits until the tiles that read it have (their progress words), and before it overwrites a history
// slot until the row that read that has.  Every wait is for a lower layer, or for an earlier tile at the
// same one, and the launch is cooperative (every block resident), so the waits end.
// Bound: the fp32 matrix units (73.7 KFLOP per row and layer at r = 64, s = 256), busy 54 % of the cycles, and
// the latencies between a layer's products.  Measured, l = 20, r = 64, s = 256, one stream of 16000 steps:
// 331 us per call, 84 TFLOP/s (the step-by-step kernels took 178.8 ms); without any exchange (a timing
// build) 306.
template <int R, int S, int NC, bool AX>
__global__ __launch_bounds__(64 * pass_waves(R), pass_blocks(R)) void teach_pass(const WnTeachArgs g, const Chunk ch) {
  extern __shared__ __align__(16) float dyn[];
  constexpr int W = pass_waves(R), NTH = 64 * W;
  using LY = Layer<R, S, NC, W, AX>;
  using GS = typename LY::G;
  using KS = typename LY::K;
  constexpr int MT = 16 * NC, P = LY::P, PS = pitch(S);
  float* X0 = dyn;            // [MT][P] x_{j-1} and x_j, in turn
  float* X1 = X0 + MT * P;
  float* Xp = X1 + MT * P;    // x_{j-1}[t - d]
  float* H = Xp + MT * P;
  float* Z = dyn;             // [MT][PS] after the layers
  float* ZA = Z + MT * PS;    // [MT][pitch(A)]
  __shared__ int s_fail;
  if (*g.status != 0) return;
  const int M = ch.nb * ch.n, tile = blockIdx.x, m0 = tile * MT, tid = threadIdx.x, L = g.d.L;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, quad = lane >> 4;
  const GS gs(wave);
  const KS ks(wave);
  const wnb_rsrc xr = buffer_of(g.x, (size_t)3 * g.rows * R * 8);
  const int4 start0 = g.start[0];
  const int64_t tg = ((int64_t)start0.y << 32 | (unsigned)start0.x) + ch.c0;  // the chunk's first global step
  if (tid == 0) s_fail = 0;

  // This thread's pieces of the tile: row lm of piece k, channels c .. c + 3; step t of stream b of the chunk.
  // Found anew at each use (see lane_now).  Quotients below 2^17 by reciprocal: (v + 1/2) / n is at least
  // 1 / (2 n) from an integer, more than fp32's error there.
  constexpr int NI = (MT * (R / 4) + NTH - 1) / NTH;
  constexpr bool kWhole = MT * (R / 4) % NTH == 0;
  const float inv_n = 1.0f / (float)ch.n;
  struct Piece {
    int lm, c, m, b, t;
    bool in;
  };
  auto piece = [&](int k) {
    unsigned i = threadIdx.x;
    asm volatile("" : "+v"(i));
    i += k * NTH;
    Piece p;
    p.lm = i / (R / 4);
    p.c = 4 * (i % (R / 4));
    p.in = kWhole || p.lm < MT;
    p.m = min(m0 + p.lm, M - 1);
    p.b = (int)(((float)p.m + 0.5f) * inv_n);
    p.t = p.m - p.b * ch.n;
    return p;
  };
  typename LY::GateFrag gf[2];
  LY::load_gate(gf[0], g, 0, 0, gs);
  LY::load_gate(gf[1], g, 0, 1, gs);
  const float* cond[GS::NCT];  // this lane's rows
#pragma unroll
  for (int k = 0; k < GS::NCT; ++k) {
    const int m = min(m0 + 16 * gs.ct(k) + n, M - 1), bi = m / ch.n, t = m - bi * ch.n;
    cond[k] = g.io.cond + ((size_t)(ch.b0 + bi) * g.io.T + ch.c0 + t) * L * 2 * R;
  }
  typename LY::SkipAcc q;
#pragma unroll
  for (int i = 0; i < KS::NRT; ++i)
#pragma unroll
    for (int k = 0; k < KS::NCT; ++k) q[i][k] = ldg4(g.w.b_skip + 16 * ks.rt(i) + 4 * quad);
  // slot (tg + t) mod d of a history, tgm = tg mod d; a chunk has at most 2^14 steps and d is at most 2^16
  struct Ring {
    int d, tgm;
    float inv;
    __device__ int slot(int t) const {
      const int v = tgm + t;
      return v - (int)(((float)v + 0.5f) * inv) * d;
    }
  };
  auto ring_of = [&](int j) {
    Ring r;
    r.d = g.d.dil[j];
    r.tgm = (int)(tg % r.d);
    r.inv = 1.0f / (float)r.d;
    return r;
  };
  Ring rg = ring_of(0);
  for (int k = 0; k < NI; ++k) {
    const Piece p = piece(k);
    if (p.in) {
      const int b = ch.b0 + p.b, at = ch.c0 + p.t;
      st4(X0 + p.lm * P + p.c, embed4(g, g.start[p.b], b, at, p.c));
      f32x4 v;
      if (p.t >= rg.d) {
        v = embed4(g, g.start[p.b], b, at - rg.d, p.c);
        if (g.ring_kind == WN_RING_PAIR) v = as_pair(v);
      } else {
        v = take(g, ring_load(g, b, 0, rg.slot(p.t), p.c));
      }
      st4(Xp + p.lm * P + p.c, v);
    }
  }

  for (int j = 0; j < L; ++j) {
    float* Xc = j & 1 ? X1 : X0;
    float* Xn = j & 1 ? X0 : X1;
    typename LY::GateAdd add;
    LY::load_add(add, g, j, gs, cond);
    issued();
    lds_barrier();
    if (s_fail) return;
    if (tid == 0) __hip_atomic_store(g.prog + tile * kProgStride, (unsigned)(j + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    typename LY::GateAcc acc;
    clear(acc);
    LY::template gate_product<0, LY::RUNS - 1>(acc, gf, g, j, Xp, Xc, gs);
    typename LY::ResFrag wr;
    typename LY::SkipFrag ws[2];
    auto load_next = [&] {
      LY::load_res(wr, g, j, gs);
      LY::load_skip(ws[0], g, j, 0, ks);
      issued();
    };
    constexpr bool kEarly = R * NC < 256;
    if (kEarly) load_next();
    LY::template gate_product<LY::RUNS - 1, LY::RUNS>(acc, gf, g, j, Xp, Xc, gs);
    if (!kEarly) load_next();  // (earlier, they would spill)
    LY::gate(H, acc, add, gs);
    if (j >= 2 && j + 1 < L) {  // x_{j+1} takes the place of x_{j-2}, which rows m + d of layer j - 2 read
      const int dd = g.d.dil[j - 2], last = (int)gridDim.x - 1;
      const int t0 = min((m0 + dd) / MT, last), t1 = min((m0 + dd + MT - 1) / MT, last);
      const unsigned p0 = ld_prog(g, t0), p1 = ld_prog(g, t1);  // (at the end of the chunk the last tile's: at worst a longer wait)
      if (p0 < (unsigned)(j - 1)) wait_prog(g, t0, j - 1, &s_fail);
      if (p1 < (unsigned)(j - 1)) wait_prog(g, t1, j - 1, &s_fail);
    }
    lds_barrier();
    RingRow past[NI];  // what the next layer looks back on beyond the chunk
    const Ring rc = rg;
    if (j + 1 < L) {
      rg = ring_of(j + 1);
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const Piece p = piece(k);
        if (p.t < rg.d) past[k] = ring_load(g, ch.b0 + p.b, j + 1, rg.slot(p.t), p.c);
      }
      const unsigned base = (unsigned)((j + 1) % 3) * g.rows * R;
      LY::residual(wr, Xc, H, gs, [&](int lm, int c, f32x4 v) {
        st4(Xn + lm * P + c, v);
        if (m0 + lm < M) st_words(xr, base + (unsigned)(m0 + lm) * R + c, v, (unsigned)(j + 1));
      });
#pragma unroll
      for (int k = 0; k < NI; ++k)
      {
        const Piece p = piece(k);
        if (p.t < rg.d && p.in) st4(Xp + p.lm * P + p.c, take(g, past[k]));
      }
    }
    // (at the last layer too: a load that some path leaves out makes every wait after it count for the
    // shortest path, i.e. wait for newer loads)
    LY::load_gate(gf[0], g, min(j + 1, L - 1), 0, gs);
    LY::load_gate(gf[1], g, min(j + 1, L - 1), 1, gs);
#pragma unroll
    for (int i = 0; i < KS::NRT; ++i) {  // tile i of W_skip in ws[i & 1], the next one loaded beside it
      if (i + 1 < KS::NRT) LY::load_skip(ws[(i + 1) & 1], g, j, i + 1, ks);
      issued();
      if (ks.on(0)) LY::skip(q, i, ws[i & 1], H, ks);
    }
    // the history of layer j: its input x_j of the chunk's last d steps; slot t mod d was read by row t mod d
    // of the stream
    for (int k = 0; k < NI; ++k) {
      const Piece p = piece(k);
      if (p.in && m0 + p.lm < M && p.t + rc.d >= ch.n) {
        const int back = (int)(((float)p.t + 0.5f) * rc.inv);
        const int reader = (p.m - back * rc.d) / MT;
        if (reader != tile) wait_prog(g, reader, j + 1, &s_fail);
        ring_store(g, ch.b0 + p.b, j, rc.slot(p.t), p.c, *reinterpret_cast<const f32x4*>(Xc + p.lm * P + p.c),
                   (unsigned)(tg + p.t + 1));
      }
    }
    if (j + 1 < L) {
      // the next layer's x[t - d] from the tiles before or from this one
      lds_barrier();  // x_{j+1} of every wave is in Xn
      const unsigned base = (unsigned)((j + 1) % 3) * g.rows * R;
      u32x4 w[NI][2];
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const Piece p = piece(k);
        const unsigned at = base + (unsigned)max(p.m - rg.d, 0) * R + p.c;
        w[k][0] = ld_words(xr, at);
        w[k][1] = ld_words(xr, at + 2);
      }
      auto put = [&](const Piece& p, f32x4 v) {
        if (g.ring_kind == WN_RING_PAIR) v = as_pair(v);
        st4(Xp + p.lm * P + p.c, v);
      };
      auto here = [&](const u32x4 (&x)[2]) {
        const unsigned tag = (unsigned)(j + 1);
        return x[0][1] == tag && x[0][3] == tag && x[1][1] == tag && x[1][3] == tag;
      };
      auto value = [&](const u32x4 (&x)[2]) {
        return f32x4{__uint_as_float(x[0][0]), __uint_as_float(x[0][2]), __uint_as_float(x[1][0]), __uint_as_float(x[1][2])};
      };
      unsigned late = 0;  // pieces that were not there yet
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const Piece p = piece(k);
        if (p.t >= rg.d && p.in) {
          const int m = p.m - rg.d;
          if (m >= m0) put(p, *reinterpret_cast<const f32x4*>(Xn + (m - m0) * P + p.c));
          else if (here(w[k])) put(p, value(w[k]));
          else late |= 1u << k;
        }
      }
#pragma unroll 1
      for (int k = 0; late >> k != 0; ++k)
        if (late >> k & 1) {
          const Piece p = piece(k);
          const unsigned at = base + (unsigned)(p.m - rg.d) * R + p.c;
          u32x4 x[2];
          int spins = 0;
          do {
            asm volatile("" ::: "memory");  // (the loads stay in the loop)
            x[0] = ld_words(xr, at);
            x[1] = ld_words(xr, at + 2);
          } while (!here(x) && !gave_up(g, spins, &s_fail));
          put(p, value(x));
        }
    }
  }
  lds_barrier();
  if (s_fail) return;
#pragma unroll
  for (int i = 0; i < KS::NRT; ++i)
#pragma unroll
    for (int k = 0; k < KS::NCT; ++k) {
      f32x4 v = q[i][k];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
      if (ks.on(k)) st4(Z + (16 * ks.ct(k) + n) * PS + 16 * ks.rt(i) + 4 * quad, v);
    }
  lds_barrier();
  head_tile<S, NC, W>(g, Z, ZA, [&](int lm, int c, f32x4 v) {
    const int m = m0 + lm;
    if (m >= M) return;
    const int bi = m / ch.n, t = m - bi * ch.n;
    st4(g.io.logits + ((size_t)(ch.b0 + bi) * g.io.T + ch.c0 + t) * A + c, v);
  });
}

// ------------------------------------------------------------------------------------------
// Calls of at most kSmallT steps: every stream's steps fit one 16-row tile, whose rows take their dilated
// inputs from the history (or, for d < T, from the tile itself).  One CU per tile could not read a layer's
// weights fast enough (147 KB at r = 64, s = 256 against ~125 GB/s of a CU), so only the chain of gates
// and residuals stays on it: W_prev x[t - d] of the layers with d >= T is computed before (small_pre, a
// block per layer), the skip projection and the head after (small_skip and small_head, a block per 16
// channels), all in the sums' order of teach_pass.
// ------------------------------------------------------------------------------------------
struct Small {
  int tiles;          // of `per` streams
  float *pre, *h;     // [L][16 tiles][2R], [L][16 tiles][R]
  float *z, *za;      // [16 tiles][S] relu(q), [16 tiles][A]
};
// Row m of a tile: step m % T of its stream m / T.
struct SmallTile {
  int b0, M;
  __device__ SmallTile(const WnTeachArgs& g, int tile) {
    const int per = kSmallT / g.io.T;
    b0 = tile * per;
    M = min(per, g.io.B - b0) * g.io.T;
  }
};
// A tile's row of [.][R] channels as B operands straight from memory or LDS.
template <int K>
__device__ __forceinline__ void mma_rows(f32x4& acc, const Frag<K, 1>& w, const f32x4 (&x)[K / 16]) {
#pragma unroll
  for (int k0 = 0; k0 < K / 16; ++k0)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.f[0][k0][e], x[k0][e], acc, 0, 0, 0);
}

// pre_j = W_prev_j x_{j-1}[t - d_j] of the layers whose rows all lie in the history; one wave per 16 channels.
template <int R>
__global__ __launch_bounds__(64) void small_pre(const WnTeachArgs g, const Small s) {
  const int j = blockIdx.x, ct = blockIdx.y, tile = blockIdx.z, T = g.io.T;
  if (j == 0 && ct == 0 && tile == 0 && threadIdx.x == 0 && abort_requested(g.io.abort_flag))
    atomicCAS(g.status, 0, (int)WN_EABORTED);
  const int d = g.d.dil[j];
  if (d < T) return;
  const SmallTile st(g, tile);
  const int lane = threadIdx.x, n = lane & 15, quad = lane >> 4, m = min(n, st.M - 1), t = m % T, b = st.b0 + m / T;
  const int64_t tg = g.io.reset ? 0 : g.state[WN_STATE_WORDS * (size_t)st.b0];
  const int slot = (int)((tg + t) % d);
  RingRow raw[R / 16];
#pragma unroll
  for (int k = 0; k < R / 16; ++k) raw[k] = ring_load(g, b, j, slot, 16 * k + 4 * quad);
  Frag<R, 1> w;
  w.load(g.p.prev, R, 0, [&](int) { return j * 2 * R + 16 * ct; });
  issued();
  f32x4 x[R / 16], acc = zero4();
#pragma unroll
  for (int k = 0; k < R / 16; ++k) x[k] = take(g, raw[k]);
  mma_rows<R>(acc, w, x);
  st4(s.pre + (((size_t)j * s.tiles + tile) * 16 + n) * 2 * R + 16 * ct + 4 * quad, acc);
}

// Four waves cover the channels at r <= 64 (more would read the same weights again: a CU reads ~53 bytes per
// clock from L2).
constexpr int small_waves(int R) { return R == 128 ? 8 : 4; }

// The chain of a tile, and its streams' state.
// BACK: some layer has d < T.
template <int R, bool AX, bool BACK>
__global__ __launch_bounds__(64 * small_waves(R), 1) void small_chain(const WnTeachArgs g, const Small s) {
  extern __shared__ __align__(16) float dyn[];
  constexpr int NTH = 64 * small_waves(R);
  using LY = Layer<R, 128, 1, small_waves(R), AX>;
  using GS = typename LY::G;
  constexpr int P = LY::P;
  static_assert(16 * (R / 4) <= NTH, "one piece of a tile's rows per thread");
  float* X0 = dyn;  // x_{j-1} and x_j, in turn
  float* X1 = X0 + 16 * P;
  float* Xp = X1 + 16 * P;  // x_{j-1}[t - d] of the layers with d < T
  float* H = Xp + 16 * P;
  if (*g.status != 0) return;
  const int T = g.io.T, L = g.d.L, tid = threadIdx.x, tile = blockIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, quad = lane >> 4;
  const SmallTile st(g, tile);
  const int M = st.M, b0 = st.b0;
  const GS gs(wave);
  const bool on = gs.on(0);
  int64_t* const state = g.state + WN_STATE_WORDS * (size_t)b0;
  const int64_t tg = g.io.reset ? 0 : state[0];
  // this thread's piece of the tile: row pm (step pt of stream pb), channels pc .. pc + 3
  const int pm = tid / (R / 4), pc = 4 * (tid % (R / 4)), pb = min(b0 + pm / T, g.io.B - 1), pt = pm % T;
  const bool mine = pm < M;
  const float* cond[1];
  {
    const int m = min(n, M - 1);
    cond[0] = g.io.cond + ((size_t)(b0 + m / T) * T + m % T) * L * 2 * R;
  }
  __shared__ int s_tgm[WN_MAX_LAYERS];  // the first step mod d of every layer (a 64-bit quotient each)
  if (tid < L) s_tgm[tid] = (int)(tg % g.d.dil[tid]);
  // What a layer's step on the chain reads from memory, loaded DEEP layers ahead (a load takes up to ~2 us
  // here, more than a layer; at r = 128 two layers' would spill).
  constexpr int DEEP = R < 128 ? 2 : 1;
  struct Stage {
    Frag<R, 2 * GS::NRT> wc;
    typename LY::GateAdd add;
    typename LY::ResFrag wr;
    f32x4 pre[2 * GS::NRT];
  } stage[DEEP];
  auto row_of = [&](int j) { return [&gs, j](int i) { return j * 2 * R + (i & 1) * R + 16 * gs.rt(i >> 1); }; };
  auto fetch_gate = [&](Stage& f, int j) {
    f.wc.load(g.p.cur, R, 0, row_of(j));
    LY::load_add(f.add, g, j, gs, cond);
#pragma unroll
    for (int i = 0; i < 2 * GS::NRT; ++i)  // (not written, and not used, where d < T)
      f.pre[i] = ldg4(s.pre + (((size_t)j * s.tiles + tile) * 16 + n) * 2 * R + (i & 1) * R + 16 * gs.rt(i >> 1) + 4 * quad);
    issued();
  };
  auto fetch_res = [&](Stage& f, int j) {
    LY::load_res(f.wr, g, j, gs);
    issued();
  };
#pragma unroll
  for (int k = 0; k < DEEP; ++k) {
    fetch_gate(stage[k], min(k, L - 1));
    fetch_res(stage[k], min(k, L - 1));
  }
  lds_barrier();
  RingRow past{};
  int d = 1, slot = 0;
  auto look = [&](int j) {  // layer j's dilation, and its look beyond the call where it is not in `pre`
    d = g.d.dil[j];
    const int v = s_tgm[j] + pt;  // below 2^17: see Piece
    slot = v - (int)(((float)v + 0.5f) * (1.0f / (float)d)) * d;
    if (BACK && d < T) past = ring_load(g, pb, j, slot, pc);
  };
  look(0);
  // a row of x goes to its own place and, where t + d is a step of the call, to the row that looks back on it
  auto put_past = [&](int m, int c, f32x4 v) {
    if (BACK && d < T && m < M && m % T + d < T) st4(Xp + (m + d) * P + c, g.ring_kind == WN_RING_PAIR ? as_pair(v) : v);
  };
  if (pm < 16) {
    int4 start = make_int4(0, 0, g.io.init_sample, -1);
    if (!g.io.reset) {
      const int64_t* ps = g.state + WN_STATE_WORDS * (size_t)pb;
      start.z = (int)ps[1];
      start.w = (int)ps[2];
    }
    const f32x4 v = mine ? embed4(g, start, pb, pt, pc) : zero4();
    st4(X0 + pm * P + pc, v);
    if (mine) put_past(pm, pc, v);
    if (BACK && d < T && (!mine || pt < d)) st4(Xp + pm * P + pc, mine ? take(g, past) : zero4());
  }
  auto layer = [&](int j, float* Xc, float* Xn, Stage& f) {
    lds_barrier();
    typename LY::GateAcc acc;
    const float* x[1];
    if (BACK && d < T) {
      Frag<R, 2 * GS::NRT> wp;
      wp.load(g.p.prev, R, 0, row_of(j));
      LY::rows(x, Xp, gs);
      clear(acc);
      mma(acc, wp, x);
    } else {
#pragma unroll
      for (int i = 0; i < 2 * GS::NRT; ++i) acc[i][0] = f.pre[i];
    }
    LY::rows(x, Xc, gs);
    if (on) {
      mma(acc, f.wc, x);
      LY::gate(H, acc, f.add, gs);
    }
    const bool keep = mine && pt + d >= T;
    const int jslot = slot;
    lds_barrier();
    // (the next loads are issued at the last layers too: a load that some path leaves out makes every wait
    // after it count for the shortest path, i.e. wait for newer loads)
    fetch_gate(f, min(j + DEEP, L - 1));
    if (j + 1 < L) {
      look(j + 1);
      if (on)
        LY::residual(f.wr, Xc, H, gs, [&](int m, int c, f32x4 v) {
          st4(Xn + m * P + c, v);
          put_past(m, c, v);
        });
      if (BACK && d < T && mine && pt < d) st4(Xp + pm * P + pc, take(g, past));
    }
    fetch_res(f, min(j + DEEP, L - 1));
    // stores last: a wait for loads issued after them would wait for them too
    if (pm < 16) st4(s.h + (((size_t)j * s.tiles + tile) * 16 + pm) * R + pc, *reinterpret_cast<const f32x4*>(H + pm * P + pc));
    // this block is the only one that uses these streams' histories, and the slots have been read
    if (keep)
      ring_store(g, pb, j, jslot, pc, *reinterpret_cast<const f32x4*>(Xc + pm * P + pc), (unsigned)(tg + pt + 1));
  };
  for (int j = 0;;) {
    layer(j, X0, X1, stage[0]);
    if (++j == L) break;
    layer(j, X1, X0, stage[DEEP - 1]);
    if (++j == L) break;
  }
  if (tid < M / T) {
    int64_t* ps = state + WN_STATE_WORDS * (size_t)tid;
    const int32_t* y = g.io.y_in + (size_t)(b0 + tid) * T;
    ps[2] = T >= 2 ? clamp_y(y[T - 2]) : (g.io.reset ? g.io.init_sample : ps[1]);
    ps[1] = clamp_y(y[T - 1]);
    ps[0] = tg + T;
  }
}

// relu(b_skip + W_skip_0 h_0 + W_skip_1 h_1 + ..) of 16 channels of a tile: the layers' products over the
// waves, their sum in layer order.
template <int R, int S>
__global__ __launch_bounds__(1024) void small_skip(const WnTeachArgs g, const Small s) {
  __shared__ __align__(16) float part[WN_MAX_LAYERS][64][4];
  if (*g.status != 0) return;
  const int ct = blockIdx.x, tile = blockIdx.y, L = g.d.L, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, quad = lane >> 4;
  for (int j = wave; j < L; j += 16) {
    Frag<R, 1> w;
    w.load(g.p.skip, R, 0, [&](int) { return j * S + 16 * ct; });
    f32x4 x[R / 16], acc = zero4();
#pragma unroll
    for (int k = 0; k < R / 16; ++k) x[k] = ldg4(s.h + (((size_t)j * s.tiles + tile) * 16 + n) * R + 16 * k + 4 * quad);
    issued();
    mma_rows<R>(acc, w, x);
    st4(part[j][lane], acc);
  }
  __syncthreads();
  if (wave == 0) {
    f32x4 q = ldg4(g.w.b_skip + 16 * ct + 4 * quad);
    for (int j = 0; j < L; ++j) q += *reinterpret_cast<const f32x4*>(part[j][lane]);
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = fmaxf(q[e], 0.f);
    st4(s.z + ((size_t)tile * 16 + n) * S + 16 * ct + 4 * quad, q);
  }
}

// 16 channels of one of the head's products: z_a (LAST = false) or the logits.
template <int K, bool LAST>
__global__ __launch_bounds__(64) void small_head(const WnTeachArgs g, const Small s) {
  if (*g.status != 0) return;
  const int ct = blockIdx.x, tile = blockIdx.y, lane = threadIdx.x, n = lane & 15, quad = lane >> 4;
  const int c = 16 * ct + 4 * quad;
  const float* src = (LAST ? s.za : s.z) + ((size_t)tile * 16 + n) * K + 4 * quad;
  Frag<K, 1> w;
  w.load(LAST ? g.p.out : g.p.relu, K, 0, [&](int) { return 16 * ct; });
  f32x4 x[K / 16], acc = zero4();
#pragma unroll
  for (int k = 0; k < K / 16; ++k) x[k] = ldg4(src + 16 * k);
  const f32x4 b = ldg4((LAST ? g.w.b_out : g.w.b_relu) + c);
  issued();
  mma_rows<K>(acc, w, x);
  f32x4 v = acc + b;
  if (LAST) {
    const SmallTile st(g, tile);
    const int T = g.io.T;
    if (n < st.M) st4(g.io.logits + ((size_t)(st.b0 + n / T) * T + n % T) * A + c, v);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
    st4(s.za + ((size_t)tile * 16 + n) * A + c, v);
  }
}

// The same at r = 16, where a CU reads a layer's weights in a fraction of its latency: one launch, a tile per
// block.  Wave 0 runs the chain alone: with 16 channels the result layout of one product (lane (n, quad):
// channels 4 quad .. of row n) is the operand layout of the next, so x and h stay in its registers, a row
// looks back on another by a shuffle, and no barrier stands in the chain.  Then two waves take the skip sums
// and all of them the head.  Bound: latencies, one after the other.  Measured, l = 4, one stream: 14.1 us a
// call of one step, 14.3 of 16 (in the five launches above 24.6 and 24.5; on the per-stream kernel 12.2 and
// 118).  (With the head's weights loaded into registers beside the chain: 14.7, and one block to a CU.)
// More than kOneTiles tiles go to teach_pass: l = 4, 512 tiles 49 against 53 us, 1024 tiles 85 against 68;
// l = 20 83 against 118 and 147 against 135.
//
// Tile t is block t + 4: block b runs on XCD b mod 8, and a single stream's generation, one block, on XCD 0.
// There its tile's weights, another copy of the matrices, would take from that L2 what the generating calls
// between keep there (three voices in turn, l = 4, 1600 steps and one forced: 4.58 ms a turn on XCD 0, 4.43
// so, 4.52 in five launches).
constexpr int kOneWaves = 8, kOneTiles = 512, kOneFirst = 4;
template <int R, int S, bool AX>
__global__ __launch_bounds__(64 * kOneWaves, 4) void small_one(const WnTeachArgs g) {
  static_assert(R == 16 && S == 32 && A == 256, "layouts below");
  extern __shared__ __align__(16) float dyn[];
  constexpr int PZ = pitch(S), DEEP = 2;
  float* H = dyn;                   // [L][16][R] h of every layer
  float* Z = H + g.d.L * 16 * R;    // [16][PZ] relu(q)
  float* ZA = Z + 16 * PZ;          // [16][pitch(A)]
  __shared__ int s_stop;
  const int T = g.io.T, L = g.d.L;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 15, quad = lane >> 4;
  const int c = 4 * quad;
  if ((int)blockIdx.x < kOneFirst) return;
  const SmallTile st(g, blockIdx.x - kOneFirst);
  int64_t tg = 0;
  if (wave == 0) {
    struct Stage {
      Frag<R, 2> wp, wc;
      Frag<R, 1> wr;
      f32x4 b[2], l[2], br, past;
      int d;
      float* slot;  // this lane's channels of the history slot its row reads
    } stage[DEEP];
    const int m = min(n, st.M - 1), t = m % T, b = st.b0 + m / T;
    const bool mine = n < st.M;
    const float* cond = g.io.cond + ((size_t)b * T + t) * L * 2 * R + c;
    int64_t* const state = g.state + WN_STATE_WORDS * (size_t)st.b0;
    tg = g.io.reset ? 0 : state[0];
    const int tgm = (int)(tg % g.d.dil[min(lane, L - 1)]);  // of layer `lane`
    float* const ring = static_cast<float*>(g.ring) + (size_t)b * g.d.hist_len + c;  // (WN_RING_F32)
    auto fetch = [&](Stage& f, int j) {
      auto pair = [&](int i) { return j * 2 * R + i * R; };
      f.wp.load(g.p.prev, R, 0, pair);
      f.wc.load(g.p.cur, R, 0, pair);
      f.wr.load(g.p.res, R, 0, [&](int) { return j * R; });
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f.b[i] = ldg4(g.w.b_gate + pair(i) + c);
        f.l[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(cond + pair(i)));
      }
      f.br = ldg4(g.w.b_res + j * R + c);
      f.d = g.d.dil[j];
      const int v = __builtin_amdgcn_readlane(tgm, j) + t;  // below 2^17: see Piece
      f.slot = ring + g.d.hoff[j] + (size_t)(v - (int)(((float)v + 0.5f) * (1.0f / (float)f.d)) * f.d) * R;
      f.past = ldg4(f.slot);
      issued();
    };
#pragma unroll
    for (int k = 0; k < DEEP; ++k) fetch(stage[k], min(k, L - 1));
    int4 start = make_int4(0, 0, g.io.init_sample, -1);
    if (!g.io.reset) {
      const int64_t* ps = g.state + WN_STATE_WORDS * (size_t)b;
      start.z = (int)ps[1];
      start.w = (int)ps[2];
    }
    f32x4 x = mine ? embed4(g, start, b, t, c) : zero4();
    auto layer = [&](int j, Stage& f) {
      f32x4 xp, acc[2] = {zero4(), zero4()};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float back = __shfl(x[e], (lane & 48) | ((n - f.d) & 15), 64);
        xp[e] = t >= f.d ? back : f.past[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.wp.f[i][0][e], xp[e], acc[i], 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.wc.f[i][0][e], x[e], acc[i], 0, 0, 0);
      const f32x4 ah = acc[0] + (f.b[0] + f.l[0]), ag = acc[1] + (f.b[1] + f.l[1]);
      f32x4 h, res = zero4();
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = tanh_nl<AX>(ah[e]) * sigmoid_nl<AX>(ag[e]);
      st4(H + (j * 16 + n) * R + c, h);
#pragma unroll
      for (int e = 0; e < 4; ++e) res = __builtin_amdgcn_mfma_f32_16x16x4f32(f.wr.f[0][0][e], h[e], res, 0, 0, 0);
      // the history of layer j: the slot was read (by this wave, above) before row t of the last d writes it
      if (mine && t + f.d >= T) st4(f.slot, x);
      x = x + (res + f.br);
      fetch(f, min(j + DEEP, L - 1));
    };
    for (int j = 0;;) {
      layer(j, stage[0]);
      if (++j == L) break;
      layer(j, stage[1]);
      if (++j == L) break;
    }
  } else if (wave == kOneWaves - 1) {
    int stop = __hip_atomic_load(g.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    if (!stop && abort_requested(g.io.abort_flag)) {
      stop = 1;
      if (lane == 0) atomicCAS(g.status, 0, (int)WN_EABORTED);
    }
    if (lane == 0) s_stop = stop;
  }
  lds_barrier();
  if (s_stop) return;
  if (wave == 1 || wave == 2) {
    const int ct = wave - 1;
    f32x4 q = ldg4(g.w.b_skip + 16 * ct + c);
    constexpr int U = 4;
    for (int j0 = 0; j0 < L; j0 += U) {
      Frag<R, 1> w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) w[u].load(g.p.skip, R, 0, [&](int) { return min(j0 + u, L - 1) * S + 16 * ct; });
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (j0 + u >= L) break;
        const f32x4 h = *reinterpret_cast<const f32x4*>(H + ((j0 + u) * 16 + n) * R + c);
        f32x4 acc = zero4();
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u].f[0][0][e], h[e], acc, 0, 0, 0);
        q += acc;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = fmaxf(q[e], 0.f);
    st4(Z + n * PZ + 16 * ct + c, q);
  }
  lds_barrier();
  head_tile<S, 1, kOneWaves>(g, Z, ZA, [&](int m, int ch, f32x4 v) {
    if (m < st.M) st4(g.io.logits + ((size_t)(st.b0 + m / T) * T + m % T) * A + ch, v);
  });
  if (wave == 0 && lane < st.M / T) {
    int64_t* ps = g.state + WN_STATE_WORDS * (size_t)(st.b0 + lane);
    const int32_t* y = g.io.y_in + (size_t)(st.b0 + lane) * T;
    ps[2] = T >= 2 ? clamp_y(y[T - 2]) : (g.io.reset ? g.io.init_sample : ps[1]);
    ps[1] = clamp_y(y[T - 1]);
    ps[0] = tg + T;
  }
}

template <class K>
hipError_t with_lds(K k, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int R, int S, int NC, bool AX>
hipError_t run_chunk(const WnTeachArgs& g, const Chunk ch, hipStream_t st) {
  const int MT = 16 * NC, tiles = (ch.nb * ch.n + MT - 1) / MT;
  const size_t lds = (size_t)MT * 4 * std::max(4 * pitch(R), pitch(S) + pitch(A));
  hipError_t e = with_lds(teach_pass<R, S, NC, AX>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(teach_begin, dim3(std::max((std::max(ch.nb, WN_TEACH_TILES) + 255) / 256, 2 * tiles)), dim3(256), 0, st, g, ch);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  void* args[] = {const_cast<WnTeachArgs*>(&g), const_cast<Chunk*>(&ch)};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(teach_pass<R, S, NC, AX>), dim3(tiles), dim3(64 * pass_waves(R)),
                                    args, (unsigned)lds, st);
}

template <int R, int S, bool AX>
hipError_t run_small(const WnTeachArgs& g, Small s, hipStream_t st) {
  const size_t lds = (size_t)16 * 4 * pitch(R) * 4;
  hipLaunchKernelGGL(small_pre<R>, dim3(g.d.L, 2 * R / 16, s.tiles), dim3(64), 0, st, g, s);
  const bool back = *std::min_element(g.d.dil, g.d.dil + g.d.L) < g.io.T;
  if (back) hipLaunchKernelGGL((small_chain<R, AX, true>), dim3(s.tiles), dim3(64 * small_waves(R)), lds, st, g, s);
  else hipLaunchKernelGGL((small_chain<R, AX, false>), dim3(s.tiles), dim3(64 * small_waves(R)), lds, st, g, s);
  hipLaunchKernelGGL((small_skip<R, S>), dim3(S / 16, s.tiles), dim3(1024), 0, st, g, s);
  hipLaunchKernelGGL((small_head<S, false>), dim3(A / 16, s.tiles), dim3(64), 0, st, g, s);
  hipLaunchKernelGGL((small_head<A, true>), dim3(A / 16, s.tiles), dim3(64), 0, st, g, s);
  return hipGetLastError();
}

template <int R, int S, bool AX>
hipError_t run(const WnTeachArgs& g, hipStream_t st) {
  const int B = g.io.B, T = g.io.T, L = g.d.L;
  if constexpr (R == 16) {
    const int tiles = T <= kSmallT ? (B + kSmallT / T - 1) / (kSmallT / T) : 0;
    if (T <= kSmallT && tiles <= kOneTiles) {
      const size_t lds = (size_t)16 * 4 * (L * R + pitch(S) + pitch(A));
      const hipError_t e = with_lds(small_one<R, S, AX>, lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((small_one<R, S, AX>), dim3(tiles + kOneFirst), dim3(64 * kOneWaves), lds, st, g);
      return hipGetLastError();
    }
  } else if (T <= kSmallT) {
    const size_t tile_floats = (size_t)16 * (L * 3 * R + S + A), have = (size_t)6 * g.rows * R;
    const int tiles = (B + kSmallT / T - 1) / (kSmallT / T);
    if (tiles * tile_floats <= have) {
      Small s{tiles, g.x, nullptr, nullptr, nullptr};
      s.h = s.pre + (size_t)L * 16 * tiles * 2 * R;
      s.z = s.h + (size_t)L * 16 * tiles * R;
      s.za = s.z + (size_t)16 * tiles * S;
      return run_small<R, S, AX>(g, s, st);
    }
  }
  // Chunks of up to `rows` rows: whole calls of as many streams as fit, or else runs of steps, at least 256 of a
  // stream.  Full chunks cost the same with runs of 64 to 1024 steps; what differs is the short launches that a
  // call's remainder adds (100 streams of 1000 steps, l = 20, r = 64: 2.68 ms, 2.17 with runs of 1024; 32 of 1500
  // at r = 128: 2.39 and 2.70), so no one length is best.
  const int rows = std::min(g.rows, WN_TEACH_TILES / 2 * pass_blocks(R) * (R == 128 ? 48 : 32));
  const int steps = std::min(T, rows);
  const int nb = std::max(1, std::min(B, rows / std::min(steps, 256)));
  const int n = std::min(T, rows / nb);
  for (int b0 = 0; b0 < B; b0 += nb) {
    for (int c0 = 0; c0 < T; c0 += n) {
      const Chunk ch{b0, std::min(nb, B - b0), c0, std::min(n, T - c0)};
      const int M = ch.nb * ch.n;
      hipError_t e;
      // tiles of as few rows as fit beside each other: a layer's time on a CU goes with its rows
      const int tiles16 = (M + 15) / 16, most = WN_TEACH_TILES / 2 * pass_blocks(R);
      if (tiles16 <= most) e = run_chunk<R, S, 1, AX>(g, ch, st);
      else if (tiles16 <= 2 * most) e = run_chunk<R, S, 2, AX>(g, ch, st);
      else e = run_chunk<R, S, R == 128 ? 3 : 2, AX>(g, ch, st);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <int R, int S>
hipError_t run_rs(const WnTeachArgs& g, hipStream_t st) {
  return g.w.approx_nl ? run<R, S, true>(g, st) : run<R, S, false>(g, st);
}

size_t up256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

size_t wn_teach_scratch_bytes(int R, int B, int rows) {
  return (size_t)WN_TEACH_TILES * kProgStride * 4 + up256((size_t)std::min(B, rows) * sizeof(int4)) + (size_t)3 * rows * R * 8;
}

size_t wn_teach_packed_floats(int L, int R, int S) {
  return (size_t)L * R * (2 * R + 2 * R + R + S) + (size_t)A * S + (size_t)A * A;
}

hipError_t wn_teach_pack(int L, int R, int S, const WnDevWeights& w, float* dst, WnTeachWeights* out) {
  const struct { const void* src; const float** at; size_t rows; int K; } m[] = {
      {w.w_prev, &out->prev, (size_t)L * 2 * R, R}, {w.w_cur, &out->cur, (size_t)L * 2 * R, R},
      {w.w_res, &out->res, (size_t)L * R, R},       {w.w_skip, &out->skip, (size_t)L * S, R},
      {w.w_relu, &out->relu, (size_t)A, S},         {w.w_out, &out->out, (size_t)A, A}};
  PackArgs a;
  for (int k = 0; k < 6; ++k) {
    a.m[k] = {static_cast<const float*>(m[k].src), dst, m[k].rows, m[k].K};
    *m[k].at = dst;
    dst += m[k].rows * m[k].K;
  }
  hipLaunchKernelGGL(pack_tiles, dim3(256, 6), dim3(256), 0, nullptr, a);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? hipStreamSynchronize(nullptr) : e;
}

// LDS of a CU at the largest tiles.
size_t wn_teach_lds_bytes(int R, int S) {
  return (size_t)(R == 128 ? 48 : 2 * 32) * 4 * std::max(4 * pitch(R), pitch(S) + pitch(A)) + 256;
}

hipError_t wn_teach_launch(WnTeachArgs g, void* scratch, int rows, hipStream_t stream) {
  char* p = static_cast<char*>(scratch);
  g.rows = rows;
  g.prog = reinterpret_cast<unsigned*>(p);
  g.start = reinterpret_cast<int4*>(p + (size_t)WN_TEACH_TILES * kProgStride * 4);
  g.x = reinterpret_cast<float*>(reinterpret_cast<char*>(g.start) + up256((size_t)std::min(g.io.B, rows) * sizeof(int4)));
  const int R = g.d.R, S = g.d.S;
  if (R == 16 && S == 32) return run_rs<16, 32>(g, stream);
  if (R == 32 && S == 128) return run_rs<32, 128>(g, stream);
  if (R == 64 && S == 128) return run_rs<64, 128>(g, stream);
  if (R == 64 && S == 256) return run_rs<64, 256>(g, stream);
  if (R == 128 && S == 256) return run_rs<128, 256>(g, stream);
  return hipErrorInvalidValue;
}
