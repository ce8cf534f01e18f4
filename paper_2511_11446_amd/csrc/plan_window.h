// Which layers of a plan go together, decided on the host before anything is launched (tests ask it without a GPU).
// Not part of the public ABI.
#pragma once
#include "../../include/diffpro_qlinear.h"
#include "ql_internal.h"

namespace ql {

struct PlanWindow {
    GemmArgs g[PLAN_WINDOW];
    DaqMany daq;   // the quantized ones among them
    int n;         // layers of the window; 0: fewer than two quantized ones, the first layer runs alone
    const GemmArgs *together[PLAN_WINDOW];   // those whose GEMMs share a launch, ahead of the others, which follow in order
    int count;
};

// Do the GEMMs of these layers give the same in any order?
bool any_order(const GemmArgs *g, size_t n);

// The next layers of a plan from `first` on in one go, where their inputs are there already: their activations are quantized by
// the launches of one layer (each layer's codes, scales and scratch in a part of its own of the workspace), then the GEMMs follow in order.  Takes
// layers as long as no input of one is written by another one before it, they fit the workspace and PLAN_WINDOW_BYTES together, and none
// quantizes its own rows inside its GEMM on one 16x16 tile per workgroup (those of two to five tiles would, on their own; here they share the DAQ launches).
void plan_window(const ql_layer_desc *layers, size_t n_layers, size_t first, const void *const *x_in, void *const *y_out, int64_t M, int64_t R,
                 const ql_daq_params *dp, void *workspace, size_t workspace_bytes, PlanWindow &w);

}  // namespace ql
