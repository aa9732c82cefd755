// shapes.hpp -- which lattices take several steps per launch, and in what pieces
// (host rules of lbm_multi.hip).
#pragma once

namespace lbm {

// Brick edges a lattice of this shape is cut into (0: it is not).
struct BrickShape {
  int b[3] = {0, 0, 0};
  int threads = 0;
  int steps = 0;  // most time steps per pass
};

// prec: lbm_precision; ncu: compute units of the device.
BrickShape brick_shape(const int dim[3], int prec, int ncu);
BrickShape brick_shape_enthalpy(const int dim[3], int prec, int ncu);

// Variant of the two-step pass that a large enthalpy lattice takes, 0 if it takes
// none (launch_march2 makes the pass).
int march_variant(const int dim[3], int prec, int ncu);

}  // namespace lbm
