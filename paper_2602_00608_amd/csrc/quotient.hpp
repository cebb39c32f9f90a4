// Division by a count whose reciprocal is at hand.
#pragma once

namespace wmdec {

// a / n, where rcp is 1 / n up to an ulp (what the reciprocal instruction gives): the remainder of a * rcp is exact in a fused
// multiply-add, and adding its share leaves half an ulp, as a division would.  Where n is a power of two rcp is exact and so is a * rcp.
template <typename F>   // (float; a template, as a fused multiply-add is no constant expression)
constexpr F quotient(F a, F n, F rcp) {
  const F q = a * rcp;
  return __builtin_fmaf(__builtin_fmaf(-q, n, a), rcp, q);
}

}  // namespace wmdec
