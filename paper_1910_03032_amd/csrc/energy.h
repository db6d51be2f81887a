// The energy at a quadrature point as the float32 CG's element kernels add it up for p.Ap.
#pragma once

#include "eo.h"

namespace sfem {

// dot + v u (the mass term) and dot + g . d (the gradient term).  Every product is formed and added
// in float64, as in the vector kernels' dot products: a product of two float32 is exact there, and
// the terms of a sheared element have both signs.  (Summed in float32 per point and then widened, an
// iteration is 0 to 2 % shorter.)
SFEM_HD double add_energy(double dot, float v, float u) { return dot + (double)v * (double)u; }
SFEM_HD double add_energy(double dot, float g1, float d1, float g2, float d2, float g3, float d3) {
  return add_energy(add_energy(add_energy(dot, g1, d1), g2, d2), g3, d3);
}

}  // namespace sfem
