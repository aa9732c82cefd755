// multi.hpp -- host entry points of the kernels that take several steps per
// launch (lbm_multi.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "enthalpy.hpp"
#include "model.hpp"
#include "shapes.hpp"

namespace lbm {

// Untyped population regions of one state (see Store in kernels.hpp).
struct StateRegions {
  void *mf, *mg, *rs, *r0;
};

// `steps` <= shape.steps time steps of an enthalpy lattice.
void launch_brick_enthalpy(const KParams<float>& kp, const EnthalpyConsts<float>& ec, const BrickShape& shape,
                           int steps, const StateRegions& src, const StateRegions& dst, hipStream_t stream);
void launch_brick_enthalpy(const KParams<double>& kp, const EnthalpyConsts<double>& ec, const BrickShape& shape,
                           int steps, const StateRegions& src, const StateRegions& dst, hipStream_t stream);

// Two time steps of a large enthalpy lattice; variant: its march_variant.
void launch_march2(const KParams<float>& kp, const EnthalpyConsts<float>& ec, const StateRegions& src,
                   const StateRegions& dst, int variant, int ncu, hipStream_t stream);
void launch_march2(const KParams<double>& kp, const EnthalpyConsts<double>& ec, const StateRegions& src,
                   const StateRegions& dst, int variant, int ncu, hipStream_t stream);

// Two time steps src -> dst (natural layout) of a lattice with q = 19 or 15
// flow populations; params: its KParams in device memory; clk, slot: its step
// count, which an FP16 pass reads in clk[slot] and writes, two more, to the other slot.
// macro1, macro2 (or null): where u and T before each step go (4 planes of nodes
// in the compute type).
void launch_brick2(int q, int prec, const void* params, const int dim[3], const BrickShape& shape,
                   const StateRegions& src, const StateRegions& dst, uint32_t* clk, int slot, void* macro1, void* macro2,
                   hipStream_t stream);

// Residual check of u and T in `cur` against `snap` (as a compare step and k_fold
// make it with blocks of 256), into res and its host mirror.
void launch_compare(int prec, const void* params, int nodes, const void* snap, const void* cur, double* part,
                    uint32_t* done, double* res, double* host, hipStream_t stream);

}  // namespace lbm
