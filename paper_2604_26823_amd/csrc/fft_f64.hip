// FP64 instantiations of the FFT passes.
#include "fft_impl.h"

namespace ic {
template void fft_r2c_z<double>(const FftArgs<double>&, const double*, double, const double*, double,
                               cx<double>*, const double*);
template void fft_c2r_z<double>(const FftArgs<double>&, const cx<double>*, double*, double,
                               const double*, double, bool);
template void fft_y<double>(const FftArgs<double>&, cx<double>*, bool);
template void fft_y_inv<double>(const FftArgs<double>&, const cx<double>*, cx<double>*, const YZMul<double>&);
template bool fft_zy_fused<double>(int, bool);
template void fft_r2c_zy<double>(const FftArgs<double>&, const PlaneFwd<double>*, int);
template void fft_c2r_yz<double>(const FftArgs<double>&, const PlaneInv<double>*, int, bool);
template void fft_x<double>(const FftArgs<double>&, const cx<double>*, cx<double>*, bool, double);
template void spectrum_pack<double>(const FftArgs<double>&, const cx<double>*, cx<double>*);
template void spectrum_unpack<double>(const FftArgs<double>&, const cx<double>*, cx<double>*);
template void fft_x_scatter<double>(const FftArgs<double>&, const cx<double>* const*, const int*, int,
                                   int, const XOut<double>*, int);
template void fft_x_gather<double>(const FftArgs<double>&, const cx<double>* const*, const Mul*, int,
                                  cx<double>*);
template void fft_x_embed<double>(const FftArgs<double>&, cx<double>*, const cx<double>*, int, double, double);
template bool fft_halo_x_apart<double>(int);
}  // namespace ic
