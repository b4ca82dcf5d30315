// The product of several tokens with deployed layers (lut_gemm.hip), as lut_matvec.hip calls it.
#pragma once
#include "common.h"

// Whether a layer's product with m tokens runs here (otherwise token by token in lut_matvec.hip).
// Depends on nothing but these sizes, so that a layer gives the same bits in any group.
bool lut_gemm_takes(int64_t d_in, int64_t d_out, int64_t m);

// Scratch for a layer's product with m tokens on the matrix cores: what is enough for any layer of
// these sizes, and what this layer's plan takes.
size_t lut_gemm_ws_bytes(int64_t d_in, int64_t d_out, int64_t m);
size_t lut_gemm_need(const cmpq_deployed_layer &layer, int64_t m);

// Enqueues the products of `layers` (checked by the caller, d_out > 0, m > 0).  `ws` holds the
// sum of lut_gemm_need over the layers.
int launch_lut_gemm(const cmpq_deployed_layer *const *layers, int n_layers, int64_t m, void *ws, hipStream_t s);
