// Interface of the generation kernel of the smallest models (gfx950).
#pragma once
#include "wn_internal.h"

#define WN_TINY_MAX_LAYERS 8
bool wn_tiny_supported(int R, int S, int L);
// Generation only; the per-stream kernel's arguments, histories and state.
hipError_t wn_tiny_launch(const WnStreamArgs& g, hipStream_t stream);
