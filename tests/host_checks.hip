// Host-side functions of the library's headers behind a C interface, for
// test_host_checks.py: compiled for the host alone, no device is touched.
#include "../paper_2604_26823_amd/csrc/fixed.h"

extern "C" {

// unit of the scale for amax, and the integer of the contribution w v
double hc_unit(double amax) { return ic::fx::scale_for(amax).inv; }
long long hc_rounded(double amax, double w, double v) {
  const ic::fx::Scale sc = ic::fx::scale_for(amax);
  return ic::fx::rounded(w, v * sc.s);
}

}
