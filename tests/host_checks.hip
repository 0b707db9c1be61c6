// Host-side functions of the library's headers behind a C interface, for
// test_host_checks.py: compiled for the host alone, no device is touched.
#include "../paper_2604_26823_amd/csrc/blocks.h"
#include "../paper_2604_26823_amd/csrc/fft.h"
#include "../paper_2604_26823_amd/csrc/sort.h"

extern "C" {

// unit of the scale for amax, and the integer of the contribution w v
double hc_unit(double amax) { return ic::fx::scale_for(amax).inv; }
long long hc_rounded(double amax, double w, double v) {
  const ic::fx::Scale sc = ic::fx::scale_for(amax);
  return ic::fx::rounded(w, v * sc.s);
}

// the eight integers that an FP32 paint adds for a particle displaced by d
// (cells of side 1) with value v, in a work item whose largest |v| is amax
void hc_particle(float d, double v, double amax, long long* out) {
  using A = ic::bk::FixAcc;
  const A::Scale sc = ic::fx::scale_for(amax);
  const double x = A::scaled(v, sc);
  const int idx[3] = {0, 0, 0};
  const float dsp[3] = {0.25f, d, 0.25f};
  const ic::pk::Stencil<float> s = ic::pk::stencil(idx, 1, dsp, 1.0f, 1.0f);
  for (int k = 0; k < 8; ++k) out[k] = 0;
  if (!A::takes(s)) return;
  int k = 0;
  ic::pk::for_corners_xyz(s, [&](int, int, int, float w, float, float, float) {
    out[k++] = ic::fx::rounded(static_cast<double>(w), x);
  });
}

// passes that a sort of n values launches
int hc_sort_passes(int bytes, long long n) {
  return bytes == 4 ? ic::sort_passes<uint32_t>(n) : ic::sort_passes<uint64_t>(n);
}

// status of an x scatter from spectra 0 and 1 to outputs o0 and o1 (numbers of spectra):
// 0 if it is launched, else the refusal's code
int hc_x_scatter(int o0, int o1) {
  ic::cx<float> spectra[4];
  const ic::cx<float>* in[2] = {spectra, spectra + 1};
  const ic::XOut<float> out[2] = {{spectra + o0, 1.0, 0.0, 0}, {spectra + o1, 1.0, 0.0, 1}};
  try {
    ic::require_apart<float>(in, 2, out, 2);
  } catch (const ic::ApiError& e) {
    return e.code;
  }
  return 0;
}

// whether a gather of m inputs by `blocks` workgroups of `threads` per input takes its
// inputs side by side, with `lds` bytes of tile per input
int hc_gather_wide(unsigned blocks, int m, int threads, long long lds) {
  return ic::gather_wide(blocks, m, threads, static_cast<size_t>(lds) * m);
}

}
