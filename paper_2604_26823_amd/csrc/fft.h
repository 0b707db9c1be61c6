// Host interface of the LDS-staged Stockham FFT passes (gfx950).
//
// A 3D real transform of an n^3 cube is three axis passes: a real-to-complex
// pass along the contiguous z axis (half-length complex FFT plus the
// even/odd split), and complex passes along y and x over the half spectrum
// [n][n][n/2+1], stored with each z row padded to kp >= n/2+1 entries so
// that rows start on 128-byte boundaries and the strided passes move whole
// cache lines (the y and x passes load and transform the pad entries with the
// others, and store none of them).  The x pass is the last forward axis
// and the first inverse one, so k-space multipliers are applied inside it:
// one kernel runs the forward x FFT, multiplies by m multipliers and runs m
// inverse x FFTs (scatter), or the reverse for m inputs summed into one
// output (gather).  Inverse passes are unnormalised; the 1/n^3 of the
// inverse real DFT is folded into the multiplier scale.  Where an x plane of the
// half spectrum fits a workgroup the z and y passes run fused, several fields
// per launch.
#pragma once

#include "common.h"
#include "halo.h"

namespace ic {

// One k-space multiplier, factored along the axes:
//   scale w(k)^white |k|^(-2 div) k~x^px k~y^py k~z^pz i^imag,
// wave numbers in units of the fundamental mode, k~ their derivative versions
// (0 at the Nyquist index); it vanishes at k = 0 when white or div is set.  The
// x passes apply w, |k|^-2 and the power of k~x, which need the transform along
// x, and the inverse y pass the rest: outputs that differ only in k~y and k~z
// share one spectrum (the three force components two, the nine fields of 2LPT
// three).
struct Mul {
  double scale = 1.0;
  int white = 0, div = 0;  // 0 or 1; 0, 1 or 2
  int px = 0, py = 0, pz = 0;  // 0..3
  int imag = 0;
};

constexpr int kMaxMul = 9;
// Depth of a slab, the block side of the particle orders.
constexpr int kSlab = 8;

// The y and z part of a multiplier with a real scale: c(k~y) d(k~z) i^imag, the
// powers as polynomials with one term.
template <typename T>
struct YZMul {
  T c[4], d[4];
  int imag;
};
template <typename T>
inline YZMul<T> yz_mul(double scale, int py, int pz, int imag) {
  YZMul<T> m{};
  m.c[py] = static_cast<T>(scale);
  m.d[pz] = static_cast<T>(1);
  m.imag = imag;
  return m;
}
template <typename T>
inline YZMul<T> yz_one() {
  return yz_mul<T>(1.0, 0, 0, 0);
}

// One output of a scatter x pass: k~x^px (a V0 + b V1), V the inputs' spectra
// times w^white |k|^(-2 div).
template <typename T>
struct XOut {
  cx<T>* S;
  double a, b;
  int px;
};

// Row pitch of the stored half spectrum: n/2+1 rounded up to a multiple of
// 128 bytes.
template <typename T>
inline int spectrum_pitch(int n) {
  const int q = 128 / static_cast<int>(sizeof(cx<T>));
  const int k = n / 2 + 1;
  return (k + q - 1) / q * q;
}

template <typename T>
struct FftArgs {
  int n = 0;                    // grid side
  int kp = 0;                   // stored row pitch of the half spectrum (spectrum_pitch)
  const cx<T>* tw = nullptr;    // device table exp(-2 pi i m / n), m < n
  const T* wtab = nullptr;      // whitening multiplier indexed by |k|^2 / kf^2 (particle grid)
  hipStream_t stream = nullptr;
};

// Real fields are [x][y][z] or in the slab layout
// [z / 8][x][y][z mod 8] of the fields that particles paint and read: inputs with a halo hl (HaloMap) are in slabs,
// outputs with slab set.

// out = forward rfft along z of (alpha a + beta b); b may be null.
template <typename T>
void fft_r2c_z(const FftArgs<T>& f, const T* a, T alpha, const T* b, T beta, cx<T>* out,
               const T* hl = nullptr);

// out = alpha * (unnormalised inverse rfft along z of in) + beta * aux (aux may be null).
template <typename T>
void fft_c2r_z(const FftArgs<T>& f, const cx<T>* in, T* out, T alpha, const T* aux, T beta,
               bool slab = false);

// One field of a fused z and y pass: forward, the half spectrum S of
// alpha (a + hl) + beta b transformed along z and y; inverse, the real field
// out = (inverse of mul S) + beta_aux aux.
template <typename T>
struct PlaneFwd {
  const T* a;
  T alpha;
  const T* b;    // nullable (all fields of one call alike)
  T beta;
  const T* hl;   // the halo of a paint, a then in slabs (nullable, all alike)
  cx<T>* S;
};
template <typename T>
struct PlaneInv {
  const cx<T>* S;
  YZMul<T> mul;  // applied to S
  T* out;
  const T* aux;  // nullable
  T beta_aux;
};

// Whether the fused z and y passes below serve grid side n at this precision
// (n <= 128, and 256 in FP32); with_aux: also with fields added to the result
// (n <= 128).
template <typename T>
bool fft_zy_fused(int n, bool with_aux = false);

// Whether a field with a halo must have the x part of it added before its forward
// passes (k_add_halo_x).  At n = 256 in FP32 the fused planes hold their field in all
// registers of a CU, one plane each: the one plane in eight with an x halo took
// 33 us longer and set the time of the launch, where adding it first takes 8.
template <typename T>
bool fft_halo_x_apart(int n);

// fft_r2c_z then the forward fft_y of m fields in one launch (where fft_zy_fused).
template <typename T>
void fft_r2c_zy(const FftArgs<T>& f, const PlaneFwd<T>* fields, int m);

// The inverse fft_y then fft_c2r_z of m fields in one launch (where
// fft_zy_fused), for spectra of real fields: their kz = 0 and kz = n/2
// columns must be Hermitian along y (their inverse along y real).
template <typename T>
void fft_c2r_yz(const FftArgs<T>& f, const PlaneInv<T>* fields, int m, bool slab);

// In-place complex FFT along y of the half spectrum (forward or inverse, unnormalised).
template <typename T>
void fft_y(const FftArgs<T>& f, cx<T>* data, bool forward);
// out = inverse FFT along y of mul in.
template <typename T>
void fft_y_inv(const FftArgs<T>& f, const cx<T>* in, cx<T>* out, const YZMul<T>& mul);

// Complex FFT along x, out = scale * FFT(in); in may equal out.
template <typename T>
void fft_x(const FftArgs<T>& f, const cx<T>* in, cx<T>* out, bool forward, T scale);

// Copies between the stored half spectrum and the contiguous n x n x (n/2+1) layout.
template <typename T>
void spectrum_pack(const FftArgs<T>& f, const cx<T>* stored, cx<T>* dense);
template <typename T>
void spectrum_unpack(const FftArgs<T>& f, const cx<T>* dense, cx<T>* stored);

// The x passes' outputs at most, and inputs of a scatter.
constexpr int kMaxXOut = 4;

// The outputs of a scatter must not share storage with its inputs or with each
// other: on small grids every output is a row of workgroups of its own, which
// reads the inputs again.
template <typename T>
inline void require_apart(const cx<T>* const* in, int nin, const XOut<T>* outs, int m) {
  for (int j = 0; j < m; ++j) {
    bool apart = true;
    for (int q = 0; q < nin; ++q) apart = apart && outs[j].S != in[q];
    for (int k = 0; k < j; ++k) apart = apart && outs[j].S != outs[k].S;
    if (!apart) throw ApiError(-7, "outputs of an x scatter share storage");
  }
}

// Forward x FFT of the nin (1 or 2) inputs, then for each j < m the inverse x
// FFT of outs[j]; white[q] per input, div for both.  The outputs must be apart
// (require_apart).
template <typename T>
void fft_x_scatter(const FftArgs<T>& f, const cx<T>* const* in, const int* white, int nin,
                   int div, const XOut<T>* outs, int m);

// White-noise upsampling (section 3, the resolution schedule): forward x FFT of
// S, whose modes with every wave index strictly inside (-nl/2, nl/2) are
// replaced by scale times those of the coarse spectrum lo ([nl][nl][nl/2+1],
// dense; its Nyquist rows are not used), then norm times the inverse x FFT, in
// place.  scale = (n/nl)^{3/2}: the unnormalised DFT of unit white noise grows
// as the root of the cell count.
template <typename T>
void fft_x_embed(const FftArgs<T>& f, cx<T>* S, const cx<T>* lo, int nl, T scale, T norm);

// Workgroups of an x pass up to which it counts as small: the chip has 256 CUs,
// and a pass over m fields then spreads them over more workgroups or threads.
// Grids up to 64^3 have at most 320, 128^3 at least 640.  Below the line the
// spread is faster (64^3, scatters of two and three outputs 5.4 and 6.4 us against
// 6.0 of one row of workgroups in FP32, of four from two inputs 8.6 against 9.9; 32^3
// FP64 6.9 against 9.6), above it slower (128^3, three outputs 11.6 -> 16.3 us
// in FP32 and 16.1 -> 24.3 in FP64, the three-input gather 13.4 -> 26.7 and 19.9 -> 33.1).
constexpr unsigned kSmallGrid = 512;
constexpr unsigned kCus = 256;
constexpr size_t kCuLds = 160 * 1024;

// Whether a gather of m inputs, `blocks` workgroups of `threads` each, takes its
// inputs side by side (lds: bytes of the m tiles): on small grids, where the CUs
// hold all its workgroups at once.  Three inputs take 8.2 us instead of 9.0 at
// 64^3 in FP64 and 6.0 instead of 8.7 at 32^3, nine 7.9 instead of 18.0 at 32^3;
// at 64^3 nine would fill a CU's LDS with each of 320 workgroups, a second round
// for 64 of them: 20.6 us against 18.7 one after the other.
inline bool gather_wide(unsigned blocks, int m, int threads, size_t lds) {
  return m > 1 && threads * m <= 1024 && blocks <= kSmallGrid && blocks <= kCus * (kCuLds / lds);
}

// out = inverse x FFT of sum_j mult_j * forward x FFT of ins[j]; out may equal
// ins[0].  The multipliers share white and div.
template <typename T>
void fft_x_gather(const FftArgs<T>& f, const cx<T>* const* ins, const Mul* muls, int m,
                  cx<T>* out);

}  // namespace ic
