// Interface of the teacher forcing that takes every step of a call at once (gfx950).
#pragma once
#include "wn_internal.h"

// Teacher forcing, parallel over time (wn_teach.hip): every product in fp32 on fp32 weights, the
// histories in the layout of the family that generates with the same handle and batch.
enum {
  WN_RING_F32 = 0,     // [B][hist_len] fp32 (per-stream kernel)
  WN_RING_TAGGED = 1,  // [B][hist_len] tagged words (fp32 multi-CU kernel)
  WN_RING_PAIR = 2,    // [B][hist_len], a slot's R values as R bf16 hi parts, then R lo parts (batched kernel)
  WN_RING_TILES = 3    // [nrep][hist_len][NS] tagged words in blocks of NS-column tiles (MFMA multi-CU kernel)
};
// Its weights: the fp32 matrices in tiles of 16 rows by 16 inputs, in the lane order of the MFMA operands
// (wn_teach_pack).
struct WnTeachWeights {
  const float *prev, *cur, *res, *skip, *relu, *out;
};
struct WnTeachArgs {
  WnDims d;
  WnDevWeights w;      // fp32 embeddings, biases
  WnTeachWeights p;
  WnIO io;
  int32_t* status;
  int64_t* state;      // [B][WN_STATE_WORDS]
  void* ring;
  int ring_kind, ring_g, ring_ns;  // WN_RING_TILES: streams per replica and columns of a tile
  int spin_limit;      // polls before a wait gives up with WN_ETIMEOUT
  // scratch, filled in by wn_teach_launch
  int rows;            // rows (one per stream and step) of a chunk
  unsigned* prog;      // the tiles' progress words
  int4* start;         // per stream: the global step a call began at (low, high word), y_{-1}, y_{-2}
  float* x;            // [3][rows][R] words (value, tag): x_{j-1}, x_j, x_{j+1} of a chunk's rows
};
#define WN_TEACH_TILES 512               // tiles of a chunk, two per CU
#define WN_TEACH_ROWS (WN_TEACH_TILES * 32)
size_t wn_teach_scratch_bytes(int R, int B, int rows);
size_t wn_teach_lds_bytes(int R, int S);  // of a CU
// `scratch`: wn_teach_scratch_bytes(R, B, rows) bytes, 256-byte aligned.
hipError_t wn_teach_launch(WnTeachArgs g, void* scratch, int rows, hipStream_t stream);

size_t wn_teach_packed_floats(int L, int R, int S);
// Packs the fp32 matrices of w into dst (wn_teach_packed_floats floats on the device) and waits for it.
hipError_t wn_teach_pack(int L, int R, int S, const WnDevWeights& w, float* dst, WnTeachWeights* out);
