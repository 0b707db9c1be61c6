// Stockham FFT passes staged in LDS for gfx950 (64-wide wavefronts).
//
// Each 1D transform of length n is done by n / R_max threads ("lanes") that
// hold R_max points in registers; a stage is one radix-R butterfly per
// (lane, batch) with the Stockham autosort index map, so data stays in
// natural order and every stage reads contiguous element runs.  Stages
// exchange data through LDS; the first stage reads global memory and the
// last one writes it, so each pass touches HBM once per element in and out.
//
// Strided passes (y, x) put consecutive lines of the batch on consecutive
// threads, so every global access of a wavefront covers LINES consecutive
// complex values (128 B in FP32); the z pass keeps lanes of one line on
// consecutive threads because its lines are contiguous.
#pragma once

#include <type_traits>

#include "fft.h"

namespace ic {
namespace fftk {

// Radix plan (up to three stages) for complex length n.
template <int n> struct Plan;
#define IC_FFT_PLAN(N, A, B, C)                                 \
  template <> struct Plan<N> {                                  \
    static constexpr int R0 = A, R1 = B, R2 = C;                \
    static constexpr int S = (B == 1) ? 1 : ((C == 1) ? 2 : 3); \
    static constexpr int RMAX = (A > B ? (A > C ? A : C) : (B > C ? B : C)); \
    static constexpr int TPL = N / RMAX;                        \
  };
IC_FFT_PLAN(2, 2, 1, 1)
IC_FFT_PLAN(4, 4, 1, 1)
IC_FFT_PLAN(8, 8, 1, 1)
IC_FFT_PLAN(16, 16, 1, 1)
IC_FFT_PLAN(32, 8, 4, 1)
IC_FFT_PLAN(64, 8, 8, 1)
IC_FFT_PLAN(128, 16, 8, 1)
IC_FFT_PLAN(256, 16, 16, 1)
IC_FFT_PLAN(512, 8, 8, 8)
IC_FFT_PLAN(1024, 16, 8, 8)
#undef IC_FFT_PLAN

// Radix plans of the fused x passes, which hold a line's spectrum in
// registers across several transforms.  At n = 128 and 256 they take radix 8
// first, so a thread holds 8 values instead of 16 and twice the waves fit per
// SIMD (x scatter of two outputs: 128^3 FP64 24.7 -> 15.6 us, 256^3 FP64 111 ->
// 88; the gather 116 -> 100 and 235 -> 175 in FP32 and FP64 at 256^3).
template <int n> struct PlanX : Plan<n> {};
template <> struct PlanX<128> {
  static constexpr int R0 = 8, R1 = 4, R2 = 4, S = 3, RMAX = 8, TPL = 128 / RMAX;
};
template <> struct PlanX<256> {
  static constexpr int R0 = 8, R1 = 8, R2 = 4, S = 3, RMAX = 8, TPL = 256 / RMAX;
};

// cos and sin of 2 pi m / 16, m = 0..7.
__device__ constexpr double kC16[8] = {1.0,
                                       0.92387953251128675613,
                                       0.70710678118654752440,
                                       0.38268343236508977173,
                                       0.0,
                                       -0.38268343236508977173,
                                       -0.70710678118654752440,
                                       -0.92387953251128675613};
__device__ constexpr double kS16[8] = {0.0,
                                       0.38268343236508977173,
                                       0.70710678118654752440,
                                       0.92387953251128675613,
                                       1.0,
                                       0.92387953251128675613,
                                       0.70710678118654752440,
                                       0.38268343236508977173};

// x * exp(-+ 2 pi i k / R) (forward: minus), k < R/2.
template <typename T, int R, bool FWD>
__device__ __forceinline__ cx<T> rot(cx<T> x, int k) {
  if (k == 0) return x;
  if (4 * k == R) return FWD ? mkc<T>(x.y, -x.x) : mkc<T>(-x.y, x.x);
  const int m = k * (16 / R);
  const T c = static_cast<T>(kC16[m]);
  const T s = FWD ? -static_cast<T>(kS16[m]) : static_cast<T>(kS16[m]);
  return mkc<T>(x.x * c - x.y * s, x.x * s + x.y * c);
}

// In-register DFT of length R (R a power of two <= 16), decimation in time.
template <typename T, int R, bool FWD>
__device__ __forceinline__ void dft(cx<T>* v) {
  if constexpr (R == 1) {
    return;
  } else if constexpr (R == 2) {
    cx<T> a = v[0];
    v[0] = cadd<T>(a, v[1]);
    v[1] = csub<T>(a, v[1]);
  } else {
    cx<T> e[R / 2], o[R / 2];
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      e[i] = v[2 * i];
      o[i] = v[2 * i + 1];
    }
    dft<T, R / 2, FWD>(e);
    dft<T, R / 2, FWD>(o);
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      cx<T> t = rot<T, R, FWD>(o[k], k);
      v[k] = cadd<T>(e[k], t);
      v[k + R / 2] = csub<T>(e[k], t);
    }
  }
}

// One Stockham stage of radix R on a length-n transform whose sub-transforms
// have size Ns.  Butterfly j reads elements j + r n/R, twiddles them by
// W_{Ns R}^{(j mod Ns) r} and writes (j - j mod Ns) R + j mod Ns + r Ns.
// tw is the table exp(-2 pi i m / (n * tws)).  All reads of the stage
// happen before the (optional) barrier and all writes after it, so a stage
// may write the buffer it read.
template <typename T, int n, int R, int TPL, bool FWD, class Load, class Store>
__device__ __forceinline__ void stage(int lane, int Ns, const cx<T>* __restrict__ tw, int tws,
                                      Load&& load, Store&& store, bool sync_before_store) {
  constexpr int NB = n / R;
  static_assert(NB % TPL == 0, "butterflies must divide evenly over lanes");
  constexpr int BPT = NB / TPL;
  cx<T> v[BPT][R];
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    const int jb = lane + b * TPL;
    const int k = jb & (Ns - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) v[b][r] = load(jb + r * NB);
    if (Ns > 1) {
      const int step = (n / (Ns * R)) * k;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        cx<T> w = tw[step * r * tws];
        if (!FWD) w.y = -w.y;
        v[b][r] = cmul<T>(v[b][r], w);
      }
    }
    dft<T, R, FWD>(v[b]);
  }
  if (sync_before_store) __syncthreads();
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    const int jb = lane + b * TPL;
    const int k = Ns == NB ? jb : jb & (Ns - 1);  // (last stage: jb < Ns)
    const int base = (jb - k) * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) store(base + r * Ns, v[b][r]);
  }
}

// Full length-n transform: first stage from load0, intermediate stages in
// the LDS buffer buf (element e of this thread's line at buf[lidx(e)]), last
// stage to storeL.
template <typename T, int n, bool FWD, class P = Plan<n>, class Load, class Store, class LIdx>
__device__ __forceinline__ void fft_line(int lane, cx<T>* buf, LIdx lidx,
                                         const cx<T>* __restrict__ tw, int tws, Load&& load0,
                                         Store&& storeL) {
  constexpr int TPL = P::TPL;
  auto ld = [&](int e) { return buf[lidx(e)]; };
  auto st = [&](int e, cx<T> v) { buf[lidx(e)] = v; };
  if constexpr (P::S == 1) {
    stage<T, n, P::R0, TPL, FWD>(lane, 1, tw, tws, load0, storeL, true);
  } else if constexpr (P::S == 2) {
    stage<T, n, P::R0, TPL, FWD>(lane, 1, tw, tws, load0, st, true);
    __syncthreads();
    stage<T, n, P::R1, TPL, FWD>(lane, P::R0, tw, tws, ld, storeL, true);
  } else {
    stage<T, n, P::R0, TPL, FWD>(lane, 1, tw, tws, load0, st, true);
    __syncthreads();
    stage<T, n, P::R1, TPL, FWD>(lane, P::R0, tw, tws, ld, st, true);
    __syncthreads();
    stage<T, n, P::R2, TPL, FWD>(lane, P::R0 * P::R1, tw, tws, ld, storeL, true);
  }
}

// Transforms that keep the last stage in registers.  The last stage of a
// Stockham plan writes element jb + r n / R_last from butterfly jb, and the
// first stage (sub-size 1) of a plan that starts with radix R_last reads
// exactly those elements into butterfly jb.  So a forward transform can end
// in registers and an inverse transform in the reversed radix order can
// start from them, with no LDS round trip in between: the fused x passes
// hold a line's spectrum in registers while it is multiplied (and summed),
// and need one LDS tile instead of two.
template <int n>
struct XPlan {
  using P = PlanX<n>;
  static constexpr int S = P::S;
  static constexpr int RL = S == 1 ? P::R0 : (S == 2 ? P::R1 : P::R2);  // last forward radix
  static constexpr int Q1 = S == 1 ? 1 : (S == 2 ? P::R0 : P::R1);      // inverse radices
  static constexpr int Q2 = S == 3 ? P::R0 : 1;                         // after RL
  static constexpr int TPL = P::TPL;
  static constexpr int NBL = n / RL;
  static constexpr int BPT = NBL / TPL;
};

// A stage whose outputs stay in registers: v[b][r] holds element
// lane + b TPL + r n / R (valid as the last stage, sub-size n / R).
template <typename T, int n, int R, int TPL, bool FWD, class Load>
__device__ __forceinline__ void stage_to_regs(int lane, int Ns, const cx<T>* __restrict__ tw,
                                              Load&& load, cx<T> (&v)[n / R / TPL][R]) {
  constexpr int NB = n / R;
  constexpr int BPT = NB / TPL;
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    const int jb = lane + b * TPL;
    const int k = jb & (Ns - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) v[b][r] = load(jb + r * NB);
    if (Ns > 1) {
      const int step = (n / (Ns * R)) * k;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        cx<T> w = tw[step * r];
        if (!FWD) w.y = -w.y;
        v[b][r] = cmul<T>(v[b][r], w);
      }
    }
    dft<T, R, FWD>(v[b]);
  }
}

// A first stage (sub-size 1) from registers: butterfly jb = lane + b TPL
// takes v[b][r] as its element jb + r n / R and stores element jb R + r.
// With sync, a barrier precedes the stores (earlier readers of the LDS
// tile are done).
template <typename T, int n, int R, int TPL, bool FWD, class Store>
__device__ __forceinline__ void stage_from_regs(int lane, cx<T> (&v)[n / R / TPL][R],
                                                Store&& store, bool sync) {
  constexpr int BPT = n / R / TPL;
#pragma unroll
  for (int b = 0; b < BPT; ++b) dft<T, R, FWD>(v[b]);
  if (sync) __syncthreads();
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    const int jb = lane + b * TPL;
#pragma unroll
    for (int r = 0; r < R; ++r) store(jb * R + r, v[b][r]);
  }
}

// Forward length-n transform from load0 ending in registers (XPlan layout);
// the first store into buf follows a barrier.
template <typename T, int n, class Load, class LIdx>
__device__ __forceinline__ void fft_fwd_to_regs(int lane, cx<T>* buf, LIdx lidx,
                                                const cx<T>* __restrict__ tw, Load&& load0,
                                                cx<T> (&v)[XPlan<n>::BPT][XPlan<n>::RL]) {
  using P = PlanX<n>;
  constexpr int TPL = P::TPL;
  auto ld = [&](int e) { return buf[lidx(e)]; };
  auto st = [&](int e, cx<T> x) { buf[lidx(e)] = x; };
  if constexpr (P::S == 1) {
    stage_to_regs<T, n, P::R0, TPL, true>(lane, 1, tw, load0, v);
  } else if constexpr (P::S == 2) {
    stage<T, n, P::R0, TPL, true>(lane, 1, tw, 1, load0, st, true);
    __syncthreads();
    stage_to_regs<T, n, P::R1, TPL, true>(lane, P::R0, tw, ld, v);
  } else {
    stage<T, n, P::R0, TPL, true>(lane, 1, tw, 1, load0, st, true);
    __syncthreads();
    stage<T, n, P::R1, TPL, true>(lane, P::R0, tw, 1, ld, st, true);
    __syncthreads();
    stage_to_regs<T, n, P::R2, TPL, true>(lane, P::R0 * P::R1, tw, ld, v);
  }
}

// Inverse length-n transform starting from registers in the XPlan layout,
// radices in the reversed order, last stage to storeL; the first store into
// buf follows a barrier.  v is consumed.
template <typename T, int n, class Store, class LIdx>
__device__ __forceinline__ void fft_inv_from_regs(int lane, cx<T>* buf, LIdx lidx,
                                                  const cx<T>* __restrict__ tw,
                                                  cx<T> (&v)[XPlan<n>::BPT][XPlan<n>::RL],
                                                  Store&& storeL) {
  using X = XPlan<n>;
  constexpr int TPL = X::TPL;
  auto ld = [&](int e) { return buf[lidx(e)]; };
  auto st = [&](int e, cx<T> x) { buf[lidx(e)] = x; };
  if constexpr (X::S == 1) {
    stage_from_regs<T, n, X::RL, TPL, false>(lane, v, storeL, false);
  } else if constexpr (X::S == 2) {
    stage_from_regs<T, n, X::RL, TPL, false>(lane, v, st, true);
    __syncthreads();
    stage<T, n, X::Q1, TPL, false>(lane, X::RL, tw, 1, ld, storeL, true);
  } else {
    stage_from_regs<T, n, X::RL, TPL, false>(lane, v, st, true);
    __syncthreads();
    stage<T, n, X::Q1, TPL, false>(lane, X::RL, tw, 1, ld, st, true);
    __syncthreads();
    stage<T, n, X::Q2, TPL, false>(lane, X::RL * X::Q1, tw, 1, ld, storeL, true);
  }
}

// ---------------------------------------------------------------- sizing
template <typename T, int N> struct ZCfg {
  static constexpr int n = N / 2;
  static constexpr int TPL = Plan<n>::TPL;
  static constexpr int LINES0 = 256 / TPL;
  static constexpr int LINES = LINES0 > 64 ? 64 : (LINES0 < 1 ? 1 : LINES0);
  static constexpr int THREADS = LINES * TPL;
  // LDS line stride (complex): one pad element per 16 (zl) plus two, so
  // the stride-16 accesses of the radix-16 stage fall in different banks.
  static constexpr int LS = n + n / 16 + 2;
};

// Padded LDS position of element e of a z line.
__device__ __forceinline__ int zl(int e) { return e + (e >> 4); }

template <typename T, int N> struct SCfg {  // strided C2C passes
  static constexpr int TPL = Plan<N>::TPL;
  static constexpr int LINES0 = sizeof(T) == 4 ? 16 : (N >= 1024 ? 4 : 8);
  static constexpr int LINES = (N <= 16) ? 64 : LINES0;
  static constexpr int THREADS = LINES * TPL;
  static constexpr int LP = LINES + 1;  // padded LDS element stride
};

template <typename T, int N> struct FCfg {  // fused x passes
  static constexpr int TPL = PlanX<N>::TPL;
  // waves per SIMD the register allocation must allow
  static constexpr int MINW = (sizeof(T) == 4 && N <= 512) ? 2 : 1;
  // Lines of a workgroup.  At n >= 256 in FP32 eight (64 bytes of a row): the
  // workgroups get half as large and overlap their loads with the others'
  // transforms, and their neighbours on the same XCD (x_line) use the other
  // half of each cache line: 512^3 x scatter of two outputs 545 -> 486 us,
  // 256^3 gather 77 -> 70.  (Without the neighbours sixteen lines were better.)
  static constexpr int LINES = (N <= 16) ? 64
                               : (sizeof(T) == 4 ? (N <= 128 ? 16 : 8)
                                                 : (N <= 512 ? 8 : 2));
  static constexpr int THREADS = LINES * TPL;
  static constexpr int LP = LINES + 1;
};

// First line of this workgroup in an x pass: consecutive groups of lines go to
// workgroups of one XCD (workgroup w runs on XCD w mod 8), which share the cache
// lines that the groups split (x gather at 256^3 in FP64 132 -> 122 us).
template <typename T, int N>
__device__ __forceinline__ int x_line() {
  const int nb = gridDim.x, w = blockIdx.x;
  return (nb % 8 == 0 ? w % 8 * (nb / 8) + w / 8 : w) * FCfg<T, N>::LINES;
}

// Elements e of one line of a strided pass, `stride` complex values apart.  A lane
// touches e = lane + constants, so an element's address is a base common to the
// workgroup, a constant multiple of the stride, and one 32-bit byte offset per
// lane; 64-bit addresses per element took a third of the x passes' registers.
template <typename T>
struct StridedLine {
  char* p;
  uint32_t off;
  int lane;
  long long sb;
  __device__ __forceinline__ StridedLine(const cx<T>* data, long long first, long long stride,
                                         int lane_)
      : p(const_cast<char*>(reinterpret_cast<const char*>(data))), lane(lane_),
        sb(stride * static_cast<long long>(sizeof(cx<T>))) {
    off = static_cast<uint32_t>((first + lane_ * stride) * static_cast<long long>(sizeof(cx<T>)));
  }
  __device__ __forceinline__ cx<T>& operator()(int e) const {
    return *reinterpret_cast<cx<T>*>(p + (e - lane) * sb + off);
  }
};

template <typename T>
__device__ __forceinline__ void load_table(cx<T>* dst, const cx<T>* __restrict__ src, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

// The cell pairs (z = 2e, 2e + 1) of one z row `line` = x N + y of a real field:
// [x][y][z], or the slab layout of the fields that particles read and paint
// (cell_at in blocks.h), [z / 8][x][y][z mod 8].  In the latter a
// wavefront that handles a few consecutive rows moves runs of 32 bytes (64 in
// FP64) per row side by side.
//
// A pair is addressed by a base that is the same for the whole workgroup
// (that of row line0 <= line, on the same or a lower plane), a constant of the
// element, and one 32-bit byte offset per lane: with TPL a multiple of the
// slab's four pairs, a lane's elements are lane + multiples of TPL and
// share that offset.  Addresses of their own for every element cost the
// fused passes, which hold a plane in all their registers, spills.
template <typename T, int N, bool SLAB, int TPL>
struct RowPairs {
  static constexpr int kP = kSlab / 2;
  static constexpr bool kShared = !SLAB || TPL % kP == 0;
  char* p;
  uint32_t off;
  int lane;
  static __device__ __forceinline__ size_t pair(size_t line, int e) {
    if (!SLAB) return line * (N / 2) + e;
    return (static_cast<size_t>(e / kP) * (N * N) + line) * kP + e % kP;
  }
  __device__ __forceinline__ RowPairs(const T* field, size_t line0, size_t line, int lane_)
      : lane(lane_) {
    p = const_cast<char*>(reinterpret_cast<const char*>(field)) + pair(line0, 0) * sizeof(cx<T>);
    off = static_cast<uint32_t>((pair(line, kShared ? lane_ : 0) - pair(line0, 0)) *
                                sizeof(cx<T>));
  }
  __device__ __forceinline__ cx<T>& operator()(int e) const {
    if constexpr (!SLAB)
      return *reinterpret_cast<cx<T>*>(p + (e - lane) * static_cast<int>(sizeof(cx<T>)) + off);
    if constexpr (kShared)
      return *reinterpret_cast<cx<T>*>(
          p + (e - lane) / kP * static_cast<long long>(N * N * kP * sizeof(cx<T>)) + off);
    return *reinterpret_cast<cx<T>*>(
        p + static_cast<uint32_t>(off + (e / kP * (N * N * kP) + e % kP) * sizeof(cx<T>)));
  }
};

// The halo of a paint (HaloMap) for ROWS rows y0.. of plane x, staged in LDS by a
// workgroup of THREADS: what the cells z = 0 mod 8 of every row take along z and its
// edges, then what the rows y = 0 mod 8 take along y.  Rows of a plane x = 0 mod
// 8 also take the x halo, laid out as the rows themselves, from memory.  A load
// per element and kind of halo, selected by the lanes that need it, would double
// the loads of the pass.
// XIN: the x halo is added here; else it is in the field already (fft_halo_x_apart).
template <typename T, int N, int ROWS, int THREADS, bool XIN>
struct HaloRows {
  static constexpr int NB = N / 8;
  static constexpr int RR = ROWS >= 8 ? ROWS / 8 : 1;
  static constexpr int Z = NB * ROWS, R = RR * N;
  static constexpr int kReals = Z + R;
  static __device__ __forceinline__ HaloMap map() {
    constexpr int lm = N == 8 ? 3 : N == 16 ? 4 : N == 32 ? 5 : N == 64 ? 6 : N == 128 ? 7
                     : N == 256 ? 8 : N == 512 ? 9 : 10;
    static_assert(1 << lm == N, "sides 8 to 1024");
    return HaloMap(lm);
  }
  // row0: first row, x N + y0
  static __device__ __forceinline__ void stage(const T* __restrict__ h, size_t row0, T* lds) {
    const HaloMap m = map();
    const unsigned x = static_cast<unsigned>(row0 / N), y0 = static_cast<unsigned>(row0 % N);
    const unsigned bx = x >> 3;
    const bool on_x = XIN && (x & 7u) == 0;
    constexpr int QZ = (Z + THREADS - 1) / THREADS, QR = (R + THREADS - 1) / THREADS;
    // all loads out before the first wait; indices past the end take the last entry
    auto iz = [](int q) { return min(static_cast<int>(threadIdx.x) + q * THREADS, Z - 1); };
    auto ir = [](int q) { return min(static_cast<int>(threadIdx.x) + q * THREADS, R - 1); };
    auto zrow = [&](int i) { return y0 + i % ROWS; };
    auto rby = [&](int i) { return (y0 >> 3) + i / N; };
    T zv[QZ], yv[QR], ev[QR];
#pragma unroll
    for (int q = 0; q < QZ; ++q) zv[q] = h[m.z(iz(q) / ROWS, x, zrow(iz(q)))];
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      const unsigned i = ir(q), z = i % N;
      yv[q] = h[m.y(rby(i), x, z)];
      ev[q] = h[m.yz(rby(i), z >> 3, x)];
    }
    if (on_x) {
#pragma unroll
      for (int q = 0; q < QZ; ++q) zv[q] += h[m.xz(bx, iz(q) / ROWS, zrow(iz(q)))];
#pragma unroll
      for (int q = 0; q < QR; ++q) {
        const unsigned i = ir(q), z = i % N;
        yv[q] += h[m.xy(bx, rby(i), z)];
        ev[q] += h[m.xyz(bx, rby(i), z >> 3)];
      }
    }
#pragma unroll
    for (int q = 0; q < QZ; ++q) lds[iz(q)] = zv[q];
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      const unsigned i = ir(q);
      lds[Z + i] = yv[q] + ((i & 7u) == 0 ? ev[q] : T(0));
    }
  }
  // raw[j], the pair of cells at element lane + j TPL of row `row` (rr after row0),
  // plus its halo.
  template <int TPL, int RAW>
  static __device__ __forceinline__ void add(const T* __restrict__ h, const T* lds, size_t row,
                                             int rr, int lane, cx<T> (&raw)[RAW]) {
    const HaloMap m = map();
    const unsigned x = static_cast<unsigned>(row / N), y = static_cast<unsigned>(row % N);
    if (XIN && (x & 7u) == 0) {
      cx<T> v[RAW];
#pragma unroll
      for (int j = 0; j < RAW; ++j)
        v[j] = *reinterpret_cast<const cx<T>*>(
            h + m.x(x >> 3, y, 2 * static_cast<unsigned>(lane + j * TPL)));
#pragma unroll
      for (int j = 0; j < RAW; ++j) raw[j] = cadd<T>(raw[j], v[j]);
    }
    if ((y & 7u) == 0) {
      const T* p = lds + Z + (rr >> 3) * N;
#pragma unroll
      for (int j = 0; j < RAW; ++j) {
        const int z = 2 * (lane + j * TPL);
        raw[j] = mkc<T>(raw[j].x + p[z], raw[j].y + p[z + 1]);
      }
    }
#pragma unroll
    for (int j = 0; j < RAW; ++j) {
      const int e = lane + j * TPL;
      const T z = lds[(e >> 2) * ROWS + rr];
      raw[j].x += (e & 3) == 0 ? z : T(0);
    }
  }
};

// ------------------------------------------------------------ z pass R2C
// Loads out before the first wait: HL and B are compile-time.
template <typename T, int N, bool HL, bool B>
__global__ __launch_bounds__((ZCfg<T, N>::THREADS)) void k_r2c_z(
    const T* __restrict__ a, T alpha, const T* __restrict__ b, T beta,
    cx<T>* __restrict__ out, const cx<T>* __restrict__ twg, int kp,
    const T* __restrict__ hl) {
  using C = ZCfg<T, N>;
  constexpr int n = C::n;
  static_assert(N * N % C::LINES == 0, "whole workgroups of rows");
  __shared__ cx<T> buf[C::LINES * C::LS];
  __shared__ cx<T> tw[N];
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const int lane = threadIdx.x % C::TPL;
  const int l = threadIdx.x / C::TPL;
  const size_t line0 = static_cast<size_t>(blockIdx.x) * C::LINES, line = line0 + l;
  const RowPairs<T, N, HL, C::TPL> ra(a, line0, line, lane);
  const RowPairs<T, N, false, C::TPL> rb(b, line0, line, lane);
  constexpr int RAW = n / C::TPL;
  cx<T> raw[RAW];
#pragma unroll
  for (int r = 0; r < RAW; ++r) raw[r] = ra(lane + r * C::TPL);
  if constexpr (HL) {
    using H = HaloRows<T, N, C::LINES, C::THREADS, true>;
    static_assert(N % C::LINES == 0 && H::kReals <= 2 * C::LINES * C::LS, "rows of one plane");
    T* st = reinterpret_cast<T*>(buf);
    H::stage(hl, line0, st);
    __syncthreads();
    H::template add<C::TPL>(hl, st, line, l, lane, raw);
  }
  auto load0 = [&](int e) -> cx<T> {
    cx<T> v = cscale<T>(raw[(e - lane) / C::TPL], alpha);
    if constexpr (B) {
      const cx<T> w = rb(e);
      v.x += beta * w.x;
      v.y += beta * w.y;
    }
    return v;
  };
  cx<T>* lb = buf + l * C::LS;
  auto lidx = [&](int e) { return l * C::LS + zl(e); };
  auto storeL = [&](int e, cx<T> v) { lb[zl(e)] = v; };
  fft_line<T, n, true>(lane, buf, lidx, tw, 2, load0, storeL);
  __syncthreads();
  cx<T>* o = out + line * kp;
  const T half = static_cast<T>(0.5);
  for (int k = lane; k <= n; k += C::TPL) {
    cx<T> zk = lb[zl(k == n ? 0 : k)];
    cx<T> zc = cconj<T>(lb[zl(k == 0 ? 0 : n - k)]);
    cx<T> e = cscale<T>(cadd<T>(zk, zc), half);
    cx<T> d = cscale<T>(csub<T>(zk, zc), half);
    // X[k] = E + W^k (-i D), W = exp(-2 pi i / N)
    cx<T> mid = mkc<T>(d.y, -d.x);
    o[k] = cadd<T>(e, cmul<T>(tw[k], mid));
  }
}

// ------------------------------------------------------------ z pass C2R
template <typename T, int N, bool SLAB>
__global__ __launch_bounds__((ZCfg<T, N>::THREADS)) void k_c2r_z(
    const cx<T>* __restrict__ in, T* __restrict__ out, T alpha, const T* __restrict__ aux,
    T beta, const cx<T>* __restrict__ twg, int kp) {
  using C = ZCfg<T, N>;
  constexpr int n = C::n;
  static_assert(N * N % C::LINES == 0, "whole workgroups of rows");
  __shared__ cx<T> buf[C::LINES * C::LS];
  __shared__ cx<T> tw[N];
  load_table<T>(tw, twg, N);
  const int lane = threadIdx.x % C::TPL;
  const int l = threadIdx.x / C::TPL;
  const size_t line0 = static_cast<size_t>(blockIdx.x) * C::LINES, line = line0 + l;
  cx<T>* lb = buf + l * C::LS;
  // the row's n + 1 values, all loads out before the first wait (no branch:
  // indices clamped)
  const cx<T>* src = in + line * kp;
  constexpr int KS = n / C::TPL + 1;
  cx<T> rv[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) rv[j] = src[min(lane + j * C::TPL, n)];
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    const int k = lane + j * C::TPL;
    if (k > n) continue;
    cx<T> v = rv[j];
    if (k == 0 || k == n) v.y = 0;  // the real transform ignores these imaginary parts
    lb[zl(k)] = v;
  }
  __syncthreads();
  auto load0 = [&](int e) -> cx<T> {
    cx<T> xk = lb[zl(e)];
    cx<T> xc = cconj<T>(lb[zl(n - e)]);
    cx<T> s = cadd<T>(xk, xc);
    cx<T> d = csub<T>(xk, xc);
    cx<T> w = cconj<T>(tw[e]);  // exp(+2 pi i e / N)
    cx<T> wd = cmul<T>(w, d);
    return mkc<T>(s.x - wd.y, s.y + wd.x);  // s + i w d
  };
  auto lidx = [&](int e) { return l * C::LS + zl(e); };
  const RowPairs<T, N, SLAB, C::TPL> dst(out, line0, line, lane);
  const cx<T>* ax = aux ? reinterpret_cast<const cx<T>*>(aux + line * N) : nullptr;
  auto storeL = [&](int e, cx<T> v) {
    cx<T> r = cscale<T>(v, alpha);
    if (ax) {
      cx<T> u = ax[e];
      r.x += beta * u.x;
      r.y += beta * u.y;
    }
    dst(e) = r;
  };
  fft_line<T, n, false>(lane, buf, lidx, tw, 2, load0, storeL);
}

// Integer wavenumber of index i on a full axis of side N.
__device__ __forceinline__ int wave_index(int i, int N) { return i < N / 2 ? i : i - N; }
// Its derivative version (0 at the Nyquist index).
template <typename T>
__device__ __forceinline__ T wave_deriv(int i, int N) {
  return static_cast<T>(i == N / 2 ? 0 : wave_index(i, N));
}
// The one-term polynomial c at k (exact where the power is: zero terms add
// nothing).
template <typename T>
__device__ __forceinline__ T one_term(const T (&c)[4], T k) {
  return fma(fma(fma(c[3], k, c[2]), k, c[1]), k, c[0]);
}
// v times the y and z part of a multiplier: ky index e of side N, dz = one_term
// of the line's k~z.
template <typename T>
__device__ __forceinline__ cx<T> times_yz(cx<T> v, const YZMul<T>& m, int e, int N, T dz) {
  const T s = one_term(m.c, wave_deriv<T>(e, N)) * dz;
  return mkc<T>(s * (m.imag ? -v.y : v.x), s * (m.imag ? v.x : v.y));
}

// The fields of one fused launch, one per blockIdx.y.
template <typename T>
struct FwdSet {
  PlaneFwd<T> f[kMaxMul];
};
template <typename T>
struct InvSet {
  PlaneInv<T> f[kMaxMul];
};

// ------------------------------------------ fused z and y passes (FP32, n = 256)
// One workgroup transforms a whole x plane along z and y, so the plane's half
// spectrum crosses HBM once instead of three times.  The plane (256 rows y of
// 129 values kz) does not fit in LDS, so two identities shrink it:
//  * the columns kz = 0 and kz = n/2 are real along y (the z transform of a
//    real row is real there), so they travel as one complex column
//    c(y) = X(y, 0) + i X(y, n/2): 128 complex columns;
//  * one radix-2 step of the length-256 y transform splits it into two
//    length-128 transforms: the even outputs are the transform of
//    u(y) + u(y + 128), the odd ones that of (u(y) - u(y + 128)) W^y.
// A 128 x 128 LDS tile plus 16 values per thread in registers then hold the
// plane.  Forward: z transforms of rows 0-127 (through the tile, into
// registers), of rows 128-255 (into the tile); the radix-2 step (sums to the
// tile, differences to registers); the 128 even-output column transforms,
// then the odd ones; the packed column's outputs are separated last
// (X0 = (C[k] + conj C[-k]) / 2, X_{n/2} = (C[k] - conj C[-k]) / 2i).  The
// inverse mirrors it; its packed column needs the kz = 0 and n/2 columns to
// be Hermitian along y, which holds for the spectrum of any real field and
// for the k-space multipliers applied to one (even ones real, odd ones
// imaginary, the derivative ones zero at the Nyquist index).
template <typename T, int N>
struct ZYCfg {
  static constexpr bool ok = false;
};
template <>
struct ZYCfg<float, 256> {
  static constexpr bool ok = true;
  static constexpr int n = 128;                  // z row (complex), tile rows and columns
  static constexpr int TPL = Plan<n>::TPL;       // threads per row or column transform
  static constexpr int THREADS = n * TPL;        // 1024
  static constexpr int LS = n + n / 16 + 2;      // tile row stride, as the z pass
  static constexpr int OWN = THREADS / n;        // thread t owns rows t / n + OWN j of column t % n
  static constexpr int PER = n / OWN;            // 16 held values per thread
};

template <typename T, int N, bool HL, bool B>
__global__ __launch_bounds__((ZYCfg<T, N>::THREADS)) void k_r2c_zy(
    FwdSet<T> fields, const cx<T>* __restrict__ twg, int kp) {
  using C = ZYCfg<T, N>;
  constexpr int n = C::n;
  const T* __restrict__ a = fields.f[blockIdx.y].a;
  const T* __restrict__ b = fields.f[blockIdx.y].b;
  const T* __restrict__ hl = fields.f[blockIdx.y].hl;
  const T alpha = fields.f[blockIdx.y].alpha, beta = fields.f[blockIdx.y].beta;
  cx<T>* __restrict__ out = fields.f[blockIdx.y].S;
  __shared__ cx<T> buf[n * C::LS];
  __shared__ cx<T> tw[N];
  __shared__ cx<T> pk[2 * n];  // the packed column's even and odd outputs
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const int t = threadIdx.x;
  const size_t x = blockIdx.x;
  const int lane = t % C::TPL, l = t / C::TPL;  // z phase: lane of tile row l
  const int c = t % n, r0 = t / n;              // column phase and held values
  const T half = static_cast<T>(0.5);
  // held values: PER - SPARE in registers, the rest in LDS (the register
  // file is full)
  constexpr int SPARE = 1;
  __shared__ cx<T> spare[SPARE * C::THREADS];
  cx<T> keep[C::PER - SPARE];
  auto held = [&](int j) -> cx<T>& {
    return j < C::PER - SPARE ? keep[j] : spare[(j - (C::PER - SPARE)) * C::THREADS + t];
  };
  cx<T>* lb = buf + l * C::LS;
  T* st = reinterpret_cast<T*>(buf);  // the half's halo
  using H = HaloRows<T, N, n, C::THREADS, false>;
  static_assert(H::kReals <= 2 * n * C::LS, "the halo fits the tile");
  for (int h = 0; h < 2; ++h) {
    const size_t line = x * N + h * n + l;
    const RowPairs<T, N, HL, C::TPL> ra(a, x * N, line, lane);
    const RowPairs<T, N, false, C::TPL> rb(b, x * N, line, lane);
    constexpr int RAW = n / C::TPL;
    cx<T> raw[RAW];  // all loads out before the first wait
    if constexpr (HL) {
      if (h == 1) __syncthreads();  // the first half's held values are read
      H::stage(hl, x * N + h * n, st);
    }
#pragma unroll
    for (int r = 0; r < RAW; ++r) raw[r] = ra(lane + r * C::TPL);
    if constexpr (HL) {
      __syncthreads();
      H::template add<C::TPL>(hl, st, line, l, lane, raw);
    }
    auto load0 = [&](int e) -> cx<T> {
      cx<T> v = cscale<T>(raw[(e - lane) / C::TPL], alpha);
      if constexpr (B) {
        const cx<T> w = rb(e);
        v.x += beta * w.x;
        v.y += beta * w.y;
      }
      return v;
    };
    auto lidx = [&](int e) { return l * C::LS + zl(e); };
    auto storeL = [&](int e, cx<T> v) { lb[zl(e)] = v; };
    fft_line<T, n, true>(lane, buf, lidx, tw, 2, load0, storeL);
    __syncthreads();
    // the real transform's split, in place, pair (k, n - k) by one thread:
    // X[k] = E + W^k (-i D), E, D = (Z[k] +- conj Z[n - k]) / 2; X[0] and
    // X[n] (both real) packed into slot 0
    for (int k = lane; k <= n / 2; k += C::TPL) {
      const cx<T> zk = lb[zl(k)];
      if (k == 0) {
        lb[zl(0)] = mkc<T>(zk.x + zk.y, zk.x - zk.y);
        continue;
      }
      const cx<T> zm = lb[zl(n - k)];
      auto split = [&](cx<T> p, cx<T> q, int j) {
        const cx<T> qc = cconj<T>(q);
        const cx<T> e = cscale<T>(cadd<T>(p, qc), half);
        const cx<T> d = cscale<T>(csub<T>(p, qc), half);
        return cadd<T>(e, cmul<T>(tw[j], mkc<T>(d.y, -d.x)));
      };
      lb[zl(k)] = split(zk, zm, k);
      if (k != n / 2) lb[zl(n - k)] = split(zm, zk, n - k);
    }
    __syncthreads();
    if (h == 0) {
#pragma unroll
      for (int j = 0; j < C::PER; ++j) held(j) = buf[(r0 + C::OWN * j) * C::LS + zl(c)];
    }
    // the second half's first tile store follows a barrier in fft_line
  }
  // radix-2 step along y: rows y (held) and y + n (tile)
#pragma unroll
  for (int j = 0; j < C::PER; ++j) {
    const int y = r0 + C::OWN * j;
    cx<T>* q = buf + y * C::LS + zl(c);
    const cx<T> lo = held(j), hi = *q;
    *q = cadd<T>(lo, hi);
    held(j) = cmul<T>(csub<T>(lo, hi), tw[y]);
  }
  __syncthreads();
  auto cidx = [&](int e) { return e * C::LS + zl(c); };
  auto cload = [&](int e) { return buf[cidx(e)]; };
  for (int par = 0; par < 2; ++par) {
    if (par == 1) {
      // the even transforms' tile reads preceded their final barrier
#pragma unroll
      for (int j = 0; j < C::PER; ++j) buf[(r0 + C::OWN * j) * C::LS + zl(c)] = held(j);
      __syncthreads();
    }
    auto storeC = [&](int e, cx<T> v) {
      if (c == 0)
        pk[par * n + e] = v;
      else
        out[(x * N + 2 * e + par) * kp + c] = v;
    };
    fft_line<T, n, true>(r0, buf, cidx, tw, 2, cload, storeC);
  }
  __syncthreads();
  for (int i = t; i < 2 * n; i += C::THREADS) {
    const int par = i / n, e = i % n;
    const int em = par == 0 ? ((n - e) & (n - 1)) : (n - 1 - e);  // output -k
    const cx<T> cc = pk[i], cm = cconj<T>(pk[par * n + em]);
    const cx<T> s = cadd<T>(cc, cm), d = csub<T>(cc, cm);
    cx<T>* o = out + (x * N + 2 * e + par) * kp;
    o[0] = cscale<T>(s, half);
    o[n] = mkc<T>(half * d.y, -half * d.x);
  }
}

template <typename T, int N, bool SLAB>
__global__ __launch_bounds__((ZYCfg<T, N>::THREADS)) void k_c2r_yz(
    InvSet<T> fields, const cx<T>* __restrict__ twg, int kp) {
  using C = ZYCfg<T, N>;
  constexpr int n = C::n;
  const cx<T>* __restrict__ in = fields.f[blockIdx.y].S;
  T* __restrict__ out = fields.f[blockIdx.y].out;
  __shared__ cx<T> buf[n * C::LS];
  __shared__ cx<T> tw[N];
  __shared__ cx<T> edge[N];  // the column kz = n/2
  const int t = threadIdx.x;
  const size_t x = blockIdx.x;
  const int c = t % n, r0 = t / n;
  if (t < N) {
    tw[t] = twg[t];
    edge[t] = in[(x * N + t) * kp + n];
  }
  // held values: PER - 1 in registers, the last in LDS (the register file
  // is full)
  __shared__ cx<T> spare[C::THREADS];
  cx<T> keep[C::PER - 1];
  auto held = [&](int j) -> cx<T>& { return j < C::PER - 1 ? keep[j] : spare[t]; };
  auto cidx = [&](int e) { return e * C::LS + zl(c); };
  auto cstore = [&](int e, cx<T> v) { buf[cidx(e)] = v; };
  // inverse y transforms of the even and odd rows ky, the packed column
  // read as X(ky, 0) + i X(ky, n/2) (k~z is 0 for both).  The column kz = n/2
  // comes through LDS: a second load per element, needed by column 0 only, took
  // three fields from 116 to 140 us.
  const YZMul<T>& mul = fields.f[blockIdx.y].mul;
  const T dz = one_term(mul.d, static_cast<T>(c));
  for (int par = 0; par < 2; ++par) {
    constexpr int RAW = n / C::TPL;  // element r0 + r TPL
    cx<T> raw[RAW];
#pragma unroll
    for (int r = 0; r < RAW; ++r)
      raw[r] = in[(x * N + 2 * (r0 + r * C::TPL) + par) * kp + c];
    if (par == 0) __syncthreads();  // edge
    if (c == 0) {
#pragma unroll
      for (int r = 0; r < RAW; ++r) {
        const cx<T> v = edge[2 * (r0 + r * C::TPL) + par];
        raw[r] = mkc<T>(raw[r].x - v.y, raw[r].y + v.x);
      }
    }
    auto load0 = [&](int e) -> cx<T> {
      return times_yz<T>(raw[(e - r0) / C::TPL], mul, 2 * e + par, N, dz);
    };
    fft_line<T, n, false>(r0, buf, cidx, tw, 2, load0, cstore);
    __syncthreads();
    if (par == 0) {
#pragma unroll
      for (int j = 0; j < C::PER; ++j) held(j) = buf[(r0 + C::OWN * j) * C::LS + zl(c)];
    }
    // the odd transforms' first tile store follows a barrier in fft_line
  }
  // radix-2 step: u(y) = E(y) + W^-y O(y), u(y + n) = E(y) - W^-y O(y)
#pragma unroll
  for (int j = 0; j < C::PER; ++j) {
    const int y = r0 + C::OWN * j;
    cx<T>* q = buf + y * C::LS + zl(c);
    const cx<T> o = cmul<T>(*q, cconj<T>(tw[y]));
    const cx<T> e = held(j);
    *q = cadd<T>(e, o);
    held(j) = csub<T>(e, o);
  }
  __syncthreads();
  const int lane = t % C::TPL, l = t / C::TPL;
  cx<T>* lb = buf + l * C::LS;
  // the real inverse's merge Z[e] = S + i W^-e D, S, D = X[e] +- conj X[n - e]
  auto merge = [&](cx<T> xk, cx<T> xc, int e) {
    const cx<T> s = cadd<T>(xk, xc);
    const cx<T> d = csub<T>(xk, xc);
    const cx<T> wd = cmul<T>(cconj<T>(tw[e]), d);
    return mkc<T>(s.x - wd.y, s.y + wd.x);
  };
  auto lidx = [&](int e) { return l * C::LS + zl(e); };
  auto lload = [&](int e) { return lb[zl(e)]; };
  for (int h = 0; h < 2; ++h) {
    if (h == 1) {
      // the first half's tile reads preceded the final barrier of its transform
#pragma unroll
      for (int j = 0; j < C::PER; ++j) buf[(r0 + C::OWN * j) * C::LS + zl(c)] = held(j);
      __syncthreads();
    }
    // merge in place, pair (k, n - k) by one thread; X[0] and X[n] (real)
    // packed in slot 0
    for (int k = lane; k <= n / 2; k += C::TPL) {
      const cx<T> xk = lb[zl(k)];
      if (k == 0) {
        lb[zl(0)] = merge(mkc<T>(xk.x, 0), mkc<T>(xk.y, 0), 0);
        continue;
      }
      const cx<T> xm = lb[zl(n - k)];
      lb[zl(k)] = merge(xk, cconj<T>(xm), k);
      if (k != n / 2) lb[zl(n - k)] = merge(xm, cconj<T>(xk), n - k);
    }
    __syncthreads();
    const size_t line = x * N + h * n + l;
    const RowPairs<T, N, SLAB, C::TPL> dst(out, x * N, line, lane);
    auto storeL = [&](int e, cx<T> v) { dst(e) = v; };
    fft_line<T, n, false>(lane, buf, lidx, tw, 2, lload, storeL);
  }
}

// ------------------------------------------- fused z and y passes (n <= 128)
// A plane x = const of the half spectrum, N rows of N/2 complex values with the
// columns kz = 0 and N/2 packed into one as above, fits the LDS of one
// workgroup (143 KiB at N = 128 in FP64), so the z and y passes of a field are
// one kernel that crosses HBM once each way, and all fields of a chain go in
// one launch.  At 32^3 and 64^3 every launch takes 3-4 us whatever it does:
// there the launches saved count (nine per force chain become three); at
// 128^3 the two passes saved do as well: three fields take 37 us instead of 55
// in FP64.  A 32^3 FP64 evaluation went from 1244 to 790 us, a 64^3 FP32 forward
// run from 1245 to 832, a 128^3 FP64 forward run and gradient from 10.25 to
// 9.47 ms.
//
// PlanY: the radix plan of the y transforms.  In FP64 at N = 128 one workgroup
// fills a CU's LDS, so it takes 1024 threads (eight values each, radix 8 4 4).
template <typename T, int N> struct PlanY : Plan<N> {};
template <> struct PlanY<double, 128> {
  static constexpr int R0 = 8, R1 = 4, R2 = 4;
  static constexpr int S = 3;
  static constexpr int RMAX = 8;
  static constexpr int TPL = 128 / RMAX;
};
template <typename T, int N>
struct PlCfg {
  static constexpr int n = N / 2;
  static constexpr int TZ = Plan<n>::TPL, TY = PlanY<T, N>::TPL;
  static constexpr int T0 = N * TZ > n * TY ? N * TZ : n * TY;
  static constexpr int TMAX = TY * n > 512 ? TY * n : 512;
  static constexpr int THREADS = T0 > TMAX ? TMAX : T0;
  static constexpr int ROWS = THREADS / TZ;                  // z transforms per round
  static constexpr int ROUNDS = N > ROWS ? N / ROWS : 1;
  static constexpr int TROWS = ROWS > N ? ROWS : N;          // tile rows (idle lanes have theirs)
  static constexpr int COLS = THREADS / TY;                  // y transforms at a time
  static constexpr int W = COLS > n ? COLS : n;
  static constexpr int LS = W + W / 16 + 2;                  // tile row stride
  static_assert(COLS >= n, "all columns in one round");
};

template <typename T, int N, bool HL, bool B>
__global__ __launch_bounds__((PlCfg<T, N>::THREADS)) void k_plane_fwd(
    FwdSet<T> fields, const cx<T>* __restrict__ twg, int kp) {
  using C = PlCfg<T, N>;
  constexpr int n = C::n;
  __shared__ cx<T> buf[C::TROWS * C::LS];
  __shared__ cx<T> tw[N];
  __shared__ cx<T> pk[N];  // the packed column's outputs
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const PlaneFwd<T>& fl = fields.f[blockIdx.y];
  const T* __restrict__ hl = fl.hl;
  const T alpha = fl.alpha, beta = fl.beta;
  cx<T>* __restrict__ out = fl.S;
  const int t = threadIdx.x;
  const size_t x = blockIdx.x;
  const int lane = t % C::TZ, l0 = t / C::TZ;
  const T half = static_cast<T>(0.5);
  // the plane's halo, staged where the last round's rows go
  T* st = reinterpret_cast<T*>(buf + (C::TROWS - C::ROWS) * C::LS);
  using H = HaloRows<T, N, N, C::THREADS, true>;
  static_assert(H::kReals <= 2 * C::ROWS * C::LS, "the halo fits the tile");
  for (int h = 0; h < C::ROUNDS; ++h) {
    const int l = h * C::ROWS + l0;                       // tile row
    const size_t line = x * N + (l < N ? l : 0);          // idle lanes transform row 0 again
    const RowPairs<T, N, HL, C::TZ> ra(fl.a, x * N, line, lane);
    const RowPairs<T, N, false, C::TZ> rb(fl.b, x * N, line, lane);
    constexpr int RAW = n / C::TZ;
    cx<T> raw[RAW];
#pragma unroll
    for (int r = 0; r < RAW; ++r) raw[r] = ra(lane + r * C::TZ);
    if constexpr (HL) {
      if (h == 0) {
        H::stage(hl, x * N, st);
        __syncthreads();
      }
      H::template add<C::TZ>(hl, st, line, static_cast<int>(line % N), lane, raw);
    }
    auto load0 = [&](int e) -> cx<T> {
      cx<T> v = cscale<T>(raw[(e - lane) / C::TZ], alpha);
      if constexpr (B) {
        const cx<T> w = rb(e);
        v.x += beta * w.x;
        v.y += beta * w.y;
      }
      return v;
    };
    cx<T>* lb = buf + l * C::LS;
    auto lidx = [&](int e) { return l * C::LS + zl(e); };
    auto storeL = [&](int e, cx<T> v) { lb[zl(e)] = v; };
    fft_line<T, n, true>(lane, buf, lidx, tw, 2, load0, storeL);
  }
  __syncthreads();
  // the real transforms' split, in place (see k_r2c_zy)
  for (int h = 0; h < C::ROUNDS; ++h) {
    cx<T>* lb = buf + (h * C::ROWS + l0) * C::LS;
    for (int k = lane; k <= n / 2; k += C::TZ) {
      const cx<T> zk = lb[zl(k)];
      if (k == 0) {
        lb[zl(0)] = mkc<T>(zk.x + zk.y, zk.x - zk.y);
        continue;
      }
      const cx<T> zm = lb[zl(n - k)];
      auto split = [&](cx<T> p, cx<T> q, int j) {
        const cx<T> qc = cconj<T>(q);
        const cx<T> e = cscale<T>(cadd<T>(p, qc), half);
        const cx<T> d = cscale<T>(csub<T>(p, qc), half);
        return cadd<T>(e, cmul<T>(tw[j], mkc<T>(d.y, -d.x)));
      };
      lb[zl(k)] = split(zk, zm, k);
      if (k != n / 2) lb[zl(n - k)] = split(zm, zk, n - k);
    }
  }
  __syncthreads();
  const int c = t % C::COLS, r0 = t / C::COLS;
  auto cidx = [&](int e) { return e * C::LS + zl(c); };
  auto cload = [&](int e) { return buf[cidx(e)]; };
  auto storeC = [&](int e, cx<T> v) {
    if (c == 0)
      pk[e] = v;
    else if (c < n)
      out[(x * N + e) * kp + c] = v;
  };
  fft_line<T, N, true, PlanY<T, N>>(r0, buf, cidx, tw, 1, cload, storeC);
  __syncthreads();
  for (int e = t; e < N; e += C::THREADS) {
    const cx<T> cc = pk[e], cm = cconj<T>(pk[(N - e) & (N - 1)]);
    const cx<T> s = cadd<T>(cc, cm), d = csub<T>(cc, cm);
    cx<T>* o = out + (x * N + e) * kp;
    o[0] = cscale<T>(s, half);
    o[n] = mkc<T>(half * d.y, -half * d.x);
  }
}

template <typename T, int N, bool SLAB>
__global__ __launch_bounds__((PlCfg<T, N>::THREADS)) void k_plane_inv(
    InvSet<T> fields, const cx<T>* __restrict__ twg, int kp) {
  using C = PlCfg<T, N>;
  constexpr int n = C::n;
  __shared__ cx<T> buf[C::TROWS * C::LS];
  __shared__ cx<T> tw[N];
  __shared__ cx<T> edge[N];  // the column kz = n (see k_c2r_yz)
  const PlaneInv<T>& fl = fields.f[blockIdx.y];
  const int t = threadIdx.x;
  const size_t x = blockIdx.x;
  {
    const int c = t % C::COLS, r0 = t / C::COLS;
    const int ci = c < n ? c : n - 1;
    const cx<T>* __restrict__ in = fl.S + x * N * kp;
    const T dz = one_term(fl.mul.d, static_cast<T>(ci));
    for (int i = t; i < N; i += C::THREADS) {
      tw[i] = twg[i];
      edge[i] = in[i * kp + n];
    }
    constexpr int TPL = PlanY<T, N>::TPL, RAW = N / TPL;  // element r0 + r TPL
    cx<T> raw[RAW];
#pragma unroll
    for (int r = 0; r < RAW; ++r) raw[r] = in[(r0 + r * TPL) * kp + ci];
    __syncthreads();  // edge
    if (c == 0) {
#pragma unroll
      for (int r = 0; r < RAW; ++r) {
        const cx<T> v = edge[r0 + r * TPL];
        raw[r] = mkc<T>(raw[r].x - v.y, raw[r].y + v.x);
      }
    }
    auto load0 = [&](int e) -> cx<T> {
      return times_yz<T>(raw[(e - r0) / TPL], fl.mul, e, N, dz);
    };
    auto cidx = [&](int e) { return e * C::LS + zl(c); };
    auto cstore = [&](int e, cx<T> v) { buf[cidx(e)] = v; };
    fft_line<T, N, false, PlanY<T, N>>(r0, buf, cidx, tw, 1, load0, cstore);
  }
  __syncthreads();
  const int lane = t % C::TZ, l0 = t / C::TZ;
  // the real inverse's merge Z[e] = S + i W^-e D, S, D = X[e] +- conj X[n - e]
  auto merge = [&](cx<T> xk, cx<T> xc, int e) {
    const cx<T> s = cadd<T>(xk, xc);
    const cx<T> d = csub<T>(xk, xc);
    const cx<T> wd = cmul<T>(cconj<T>(tw[e]), d);
    return mkc<T>(s.x - wd.y, s.y + wd.x);
  };
  for (int h = 0; h < C::ROUNDS; ++h) {
    cx<T>* lb = buf + (h * C::ROWS + l0) * C::LS;
    for (int k = lane; k <= n / 2; k += C::TZ) {
      const cx<T> xk = lb[zl(k)];
      if (k == 0) {
        lb[zl(0)] = merge(mkc<T>(xk.x, 0), mkc<T>(xk.y, 0), 0);
        continue;
      }
      const cx<T> xm = lb[zl(n - k)];
      lb[zl(k)] = merge(xk, cconj<T>(xm), k);
      if (k != n / 2) lb[zl(n - k)] = merge(xm, cconj<T>(xk), n - k);
    }
  }
  __syncthreads();
  const T* __restrict__ aux = fl.aux;
  const T beta = fl.beta_aux;
  for (int h = 0; h < C::ROUNDS; ++h) {
    const int l = h * C::ROWS + l0;
    const size_t line = x * N + (l < N ? l : 0);
    const cx<T>* lb = buf + l * C::LS;
    const RowPairs<T, N, SLAB, C::TZ> dst(fl.out, x * N, line, lane);
    auto lidx = [&](int e) { return l * C::LS + zl(e); };
    auto lload = [&](int e) { return lb[zl(e)]; };
    auto storeL = [&](int e, cx<T> v) {
      if (l >= N) return;
      if (aux) {
        const cx<T> u = reinterpret_cast<const cx<T>*>(aux)[line * n + e];
        v.x += beta * u.x;
        v.y += beta * u.y;
      }
      dst(e) = v;
    };
    fft_line<T, n, false>(lane, buf, lidx, tw, 2, lload, storeL);
  }
}

// ------------------------------------------------- strided C2C (y or x)
// Line L of the batch starts at (L / group) * gstride + L % group and its
// elements are estride apart; lines with L mod vmod >= vcnt are row padding
// and are skipped.
// MUL (the inverse y pass of a chain): elements are multiplied by mul on load, e
// being their ky and L mod vmod their kz.
template <typename T, int N, bool FWD, bool MUL>
__global__ __launch_bounds__((SCfg<T, N>::THREADS)) void k_strided(
    const cx<T>* in, cx<T>* out, T scale, const cx<T>* __restrict__ twg, int nlines, int group,
    long long gstride, long long estride, int vmod, int vcnt, YZMul<T> mul) {
  using C = SCfg<T, N>;
  __shared__ cx<T> buf[N * C::LP];
  __shared__ cx<T> tw[N];
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const int l = threadIdx.x % C::LINES;
  const int lane = threadIdx.x / C::LINES;
  const int line = blockIdx.x * C::LINES + l;
  const bool valid = (line % vmod) < vcnt;  // row padding is transformed too, and not stored
  const int g0 = blockIdx.x * C::LINES / group;
  const long long first = (long long)(line / group - g0) * gstride + line % group;
  const StridedLine<T> src(in + g0 * gstride, first, estride, lane);
  const StridedLine<T> dst(out + g0 * gstride, first, estride, lane);
  const T dz = MUL ? one_term(mul.d, line % vmod == N / 2 ? T(0) : static_cast<T>(line % vmod))
                   : T(1);
  auto load0 = [&](int e) -> cx<T> {
    const cx<T> v = src(e);
    if constexpr (MUL) return times_yz<T>(v, mul, e, N, dz);
    return v;
  };
  auto storeL = [&](int e, cx<T> v) {
    if (valid) dst(e) = cscale<T>(v, scale);
  };
  auto lidx = [&](int e) { return e * C::LP + l; };
  fft_line<T, N, FWD>(lane, buf, lidx, tw, 1, load0, storeL);
}

// ------------------------------------------------- x passes
template <typename T>
struct InPtrs {
  const cx<T>* p[kMaxMul];
};

// w(k)^white |k|^(-2 div) at the squared integer wave number n2 (0 at n2 = 0 when
// either is set).
template <typename T>
__device__ __forceinline__ T k_factor(int n2, int white, int div, const T* __restrict__ wtab) {
  const T inv = static_cast<T>(1) / static_cast<T>(n2);
  T f = white ? wtab[n2] : static_cast<T>(1);
  f *= div == 0 ? static_cast<T>(1) : (div == 1 ? inv : inv * inv);
  return n2 == 0 && (white || div) ? static_cast<T>(0) : f;
}

// Outputs of a scatter: coefficients of the one-term polynomials in k~x.
template <typename T>
struct XOutSet {
  cx<T>* p[kMaxXOut];
  T a[kMaxXOut][4], b[kMaxXOut][4];
};

// Forward x FFT of the inputs, times w and |k|^-2 in place, then m inverse x FFTs
// of their combinations with powers of k~x; the forward results stay in
// registers (XPlan layout) across the m inverses.  On grids too small to
// fill the chip (fft_x_scatter) the outputs are dealt over blockIdx.y and each
// workgroup repeats the forward transform.
//
// With whole multipliers per output (a division, a table and index arithmetic
// per element and output) the pass was bound by its arithmetic at two waves per
// SIMD; factored, an output costs one multiplication per part.
template <typename T, int N, int NIN>
__global__ __launch_bounds__((FCfg<T, N>::THREADS),
                             (FCfg<T, N>::MINW)) void k_x_scatter(
    InPtrs<T> ins, int white0, int white1, int div, XOutSet<T> outs, int m,
    const T* __restrict__ wtab, const cx<T>* __restrict__ twg, int nlines, int K, int kp) {
  using C = FCfg<T, N>;
  using X = XPlan<N>;
  __shared__ cx<T> B[N * C::LP];
  __shared__ cx<T> tw[N];
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const int l = threadIdx.x % C::LINES;
  const int lane = threadIdx.x / C::LINES;
  const int line = x_line<T, N>() + l;
  const int ky = line / kp, kz = line % kp;
  const bool valid = kz < K;  // row padding is transformed too, and not stored
  const long long stride = (long long)nlines;  // = N * kp
  const int iy = wave_index(ky, N), iz = kz;
  auto lidx = [&](int e) { return e * C::LP + l; };
  cx<T> V[NIN][X::BPT][X::RL];
#pragma unroll
  for (int q = 0; q < NIN; ++q) {
    const StridedLine<T> in(ins.p[q], line, stride, lane);
    auto load_in = [&](int e) -> cx<T> { return in(e); };
    fft_fwd_to_regs<T, N>(lane, B, lidx, tw, load_in, V[q]);
#pragma unroll
    for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
      for (int r = 0; r < X::RL; ++r) {
        const int ix = wave_index(lane + b * X::TPL + r * X::NBL, N);
        const int n2 = valid ? ix * ix + iy * iy + iz * iz : 0;
        V[q][b][r] = cscale<T>(V[q][b][r], k_factor<T>(n2, q ? white1 : white0, div, wtab));
      }
    }
  }
  for (int j = blockIdx.y; j < m; j += gridDim.y) {
    cx<T> W[X::BPT][X::RL];
#pragma unroll
    for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
      for (int r = 0; r < X::RL; ++r) {
        const T dx = wave_deriv<T>(lane + b * X::TPL + r * X::NBL, N);
        const T sa = one_term(outs.a[j], dx);
        cx<T> w = cscale<T>(V[0][b][r], sa);
        if constexpr (NIN == 2) {
          const T sb = one_term(outs.b[j], dx);
          w.x = fma(sb, V[1][b][r].x, w.x);
          w.y = fma(sb, V[1][b][r].y, w.y);
        }
        W[b][r] = w;
      }
    }
    const StridedLine<T> dst(outs.p[j], line, stride, lane);
    auto store_o = [&](int e, cx<T> v) {
      if (valid) dst(e) = v;
    };
    fft_inv_from_regs<T, N>(lane, B, lidx, tw, W, store_o);
  }
}

// The polynomial parts of a gather's multipliers; white and div are common.
template <typename T>
struct GatherSet {
  T cx[kMaxMul][4], cy[kMaxMul][4], cz[kMaxMul][4];
  int imag[kMaxMul];
};

// s_j k~x^px k~y^py k~z^pz i^imag of input j applied to v (dyz: its y and z part).
template <typename T>
__device__ __forceinline__ cx<T> gather_term(cx<T> v, const T (&c)[4], int imag, T dx, T dyz) {
  const T s = one_term(c, dx) * dyz;
  return mkc<T>(s * (imag ? -v.y : v.x), s * (imag ? v.x : v.y));
}

// Sum over m inputs of multiplier * forward x FFT (accumulated in
// registers), then one inverse x FFT.
template <typename T, int N>
__global__ __launch_bounds__((FCfg<T, N>::THREADS)) void k_x_gather(
    InPtrs<T> ins, GatherSet<T> gs, int white, int div, int m, cx<T>* out,
    const T* __restrict__ wtab, const cx<T>* __restrict__ twg, int nlines, int K, int kp) {
  using C = FCfg<T, N>;
  using X = XPlan<N>;
  __shared__ cx<T> B[N * C::LP];
  __shared__ cx<T> tw[N];
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const int l = threadIdx.x % C::LINES;
  const int lane = threadIdx.x / C::LINES;
  const int line = x_line<T, N>() + l;
  const int ky = line / kp, kz = line % kp;
  const bool valid = kz < K;  // row padding is transformed too, and not stored
  const long long stride = (long long)nlines;  // = N * kp
  const int iy = wave_index(ky, N), iz = kz;
  const T dy = wave_deriv<T>(ky, N), dz = static_cast<T>(kz == N / 2 ? 0 : kz);
  auto lidx = [&](int e) { return e * C::LP + l; };
  cx<T> acc[X::BPT][X::RL];
  for (int j = 0; j < m; ++j) {
    const StridedLine<T> src(ins.p[j], line, stride, lane);
    auto load_in = [&](int e) -> cx<T> { return src(e); };
    cx<T> V[X::BPT][X::RL];
    fft_fwd_to_regs<T, N>(lane, B, lidx, tw, load_in, V);
    const T dyz = one_term(gs.cy[j], dy) * one_term(gs.cz[j], dz);
#pragma unroll
    for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
      for (int r = 0; r < X::RL; ++r) {
        const T dx = wave_deriv<T>(lane + b * X::TPL + r * X::NBL, N);
        const cx<T> t = gather_term<T>(V[b][r], gs.cx[j], gs.imag[j], dx, dyz);
        acc[b][r] = j == 0 ? t : cadd<T>(acc[b][r], t);
      }
    }
  }
#pragma unroll
  for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
    for (int r = 0; r < X::RL; ++r) {
      const int ix = wave_index(lane + b * X::TPL + r * X::NBL, N);
      const int n2 = valid ? ix * ix + iy * iy + iz * iz : 0;
      acc[b][r] = cscale<T>(acc[b][r], k_factor<T>(n2, white, div, wtab));
    }
  }
  const StridedLine<T> dst(out, line, stride, lane);
  auto store_o = [&](int e, cx<T> v) {
    if (valid) dst(e) = v;
  };
  fft_inv_from_regs<T, N>(lane, B, lidx, tw, acc, store_o);
}

// The gather of grids too small to fill the chip: thread group j of the
// workgroup takes input j through its forward transform in an LDS tile of its
// own, every group then sums all tiles (in the order of the inputs, as above)
// and inverts, and the first one stores.  The m transforms run side by side
// instead of one after the other.
template <typename T, int N>
__global__ __launch_bounds__(1024) void k_x_gather_wide(
    InPtrs<T> ins, GatherSet<T> gs, int white, int div, int m, cx<T>* out,
    const T* __restrict__ wtab, const cx<T>* __restrict__ twg, int nlines, int K, int kp) {
  using C = FCfg<T, N>;
  using X = XPlan<N>;
  extern __shared__ char smem[];
  cx<T>* tw = reinterpret_cast<cx<T>*>(smem);
  cx<T>* tiles = tw + N;
  load_table<T>(tw, twg, N);
  const int j = threadIdx.x / C::THREADS, t = threadIdx.x % C::THREADS;
  cx<T>* B = tiles + j * N * C::LP;
  const int l = t % C::LINES;
  const int lane = t / C::LINES;
  const int line = x_line<T, N>() + l;
  const int ky = line / kp, kz = line % kp;
  const bool valid = kz < K;  // row padding is transformed too, and not stored
  const long long stride = (long long)nlines;  // = N * kp
  const int iy = wave_index(ky, N), iz = kz;
  const T dy = wave_deriv<T>(ky, N), dz = static_cast<T>(kz == N / 2 ? 0 : kz);
  auto lidx = [&](int e) { return e * C::LP + l; };
  const cx<T>* src = ins.p[j];
  auto load_in = [&](int e) -> cx<T> { return src[line + e * stride]; };
  cx<T> V[X::BPT][X::RL];
  fft_fwd_to_regs<T, N>(lane, B, lidx, tw, load_in, V);
  __syncthreads();
  const T dyz = one_term(gs.cy[j], dy) * one_term(gs.cz[j], dz);
#pragma unroll
  for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
    for (int r = 0; r < X::RL; ++r) {
      const int e = lane + b * X::TPL + r * X::NBL;
      B[lidx(e)] = gather_term<T>(V[b][r], gs.cx[j], gs.imag[j], wave_deriv<T>(e, N), dyz);
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
    for (int r = 0; r < X::RL; ++r) {
      const int e = lane + b * X::TPL + r * X::NBL, i = lidx(e);
      cx<T> a = tiles[i];
      for (int q = 1; q < m; ++q) a = cadd<T>(a, tiles[q * N * C::LP + i]);
      const int ix = wave_index(e, N);
      const int n2 = valid ? ix * ix + iy * iy + iz * iz : 0;
      V[b][r] = cscale<T>(a, k_factor<T>(n2, white, div, wtab));
    }
  }
  __syncthreads();
  auto store_o = [&](int e, cx<T> v) {
    if (valid && j == 0) out[line + e * stride] = v;
  };
  fft_inv_from_regs<T, N>(lane, B, lidx, tw, V, store_o);
}

// The x passes of the white-noise upsampling (fft_x_embed): one pass over the
// spectrum, where two transforms and a kernel that wrote the coarse modes between
// them took three (25 + 12 + 25 us at 256^3 in FP32).
template <typename T, int N>
__global__ __launch_bounds__((FCfg<T, N>::THREADS)) void k_x_embed(
    cx<T>* S, const cx<T>* __restrict__ lo, int nl, T scale, T norm,
    const cx<T>* __restrict__ twg, int nlines, int K, int kp) {
  using C = FCfg<T, N>;
  using X = XPlan<N>;
  __shared__ cx<T> B[N * C::LP];
  __shared__ cx<T> tw[N];
  load_table<T>(tw, twg, N);  // visible after the first stage's barrier, before any use
  const int l = threadIdx.x % C::LINES;
  const int lane = threadIdx.x / C::LINES;
  const int line = x_line<T, N>() + l;
  const int ky = line / kp, kz = line % kp;
  const long long stride = (long long)nlines;  // = N * kp
  auto lidx = [&](int e) { return e * C::LP + l; };
  const StridedLine<T> io(S, line, stride, lane);
  auto load_in = [&](int e) -> cx<T> { return io(e); };
  cx<T> V[X::BPT][X::RL];
  fft_fwd_to_regs<T, N>(lane, B, lidx, tw, load_in, V);
  // coarse index of fine index i, and whether the band holds it
  const int h = nl / 2;
  auto coarse = [&](int i) { return i < h ? i : i - (N - nl); };
  auto inside = [&](int i) { return i < h || i > N - h; };
  if (kz < h && inside(ky)) {
    const cx<T>* row = lo + static_cast<long long>(coarse(ky)) * (h + 1) + kz;
    const long long plane = static_cast<long long>(nl) * (h + 1);
#pragma unroll
    for (int b = 0; b < X::BPT; ++b) {
#pragma unroll
      for (int r = 0; r < X::RL; ++r) {
        const int e = lane + b * X::TPL + r * X::NBL;
        if (inside(e)) V[b][r] = cscale<T>(row[coarse(e) * plane], scale);
      }
    }
  }
  auto store_o = [&](int e, cx<T> v) {
    if (kz < K) io(e) = cscale<T>(v, norm);  // row padding is transformed too, and not stored
  };
  fft_inv_from_regs<T, N>(lane, B, lidx, tw, V, store_o);
}

// ------------------------------------------------- layout conversion
// Copies between the stored half spectrum (row pitch kp) and the contiguous
// [n][n][n/2+1] layout; pack = stored -> contiguous.
template <typename T, bool PACK>
__global__ void k_spec_copy(const cx<T>* __restrict__ src, cx<T>* __restrict__ dst, int K,
                            int kp, long long H) {
  for (long long f = blockIdx.x * (long long)blockDim.x + threadIdx.x; f < H;
       f += (long long)gridDim.x * blockDim.x) {
    const long long s = (f / K) * kp + f % K;
    if (PACK)
      dst[f] = src[s];
    else
      dst[s] = src[f];
  }
}

// ------------------------------------------------------------ dispatch
// f(HL, B) with the two flags as compile-time constants (a painted field, which
// has a halo, has no second input).
template <class F>
void with_flags(bool hl, bool b, F&& f) {
  using Y = std::true_type;
  using No = std::false_type;
  if (hl && b) throw ApiError(-2, "a field with a halo has no second input");
  if (hl)
    f(Y{}, No{});
  else if (b)
    f(No{}, Y{});
  else
    f(No{}, No{});
}

template <typename T, class F>
void dispatch_n(int n, F&& f) {
  switch (n) {
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    case 256: f(std::integral_constant<int, 256>{}); break;
    case 512: f(std::integral_constant<int, 512>{}); break;
    case 1024: f(std::integral_constant<int, 1024>{}); break;
    default: throw ApiError(-2, "FFT size must be a power of two in [8, 1024]");
  }
}

// Whether the chains' fields of side N always take the fused z and y passes (without
// aux), so that the separate passes need no slab, halo or second-input form.
template <typename T, int N>
constexpr bool planes() {
  return N <= 128 || ZYCfg<T, N>::ok;
}

}  // namespace fftk

template <typename T>
bool fft_zy_fused(int n, bool with_aux) {
  return n <= 128 || (!with_aux && fftk::ZYCfg<T, 256>::ok && n == 256);
}

template <typename T>
void fft_r2c_z(const FftArgs<T>& f, const T* a, T alpha, const T* b, T beta, cx<T>* out,
               const T* hl) {
  if ((hl || b) && fft_zy_fused<T>(f.n)) throw ApiError(-2, "chains go through the fused planes");
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::ZCfg<T, N>;
    const int nlines = f.n * f.n;
    fftk::with_flags(hl != nullptr, b != nullptr, [&](auto HL, auto B) {
      fftk::k_r2c_z<T, N, HL.value && !fftk::planes<T, N>(),
                    B.value && !fftk::planes<T, N>()>
          <<<blocks_for(nlines, C::LINES), C::THREADS, 0, f.stream>>>(a, alpha, b, beta, out,
                                                                      f.tw, f.kp, hl);
    });
  });
  IC_LAUNCHED();
}

template <typename T>
void fft_c2r_z(const FftArgs<T>& f, const cx<T>* in, T* out, T alpha, const T* aux, T beta,
               bool slab) {
  if (slab && fft_zy_fused<T>(f.n)) throw ApiError(-2, "slabs come out of the fused planes");
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::ZCfg<T, N>;
    const int nlines = f.n * f.n;
    const unsigned grid = blocks_for(nlines, C::LINES);
    if (slab)
      fftk::k_c2r_z<T, N, !fftk::planes<T, N>()><<<grid, C::THREADS, 0, f.stream>>>(in, out, alpha, aux, beta,
                                                                   f.tw, f.kp);
    else
      fftk::k_c2r_z<T, N, false><<<grid, C::THREADS, 0, f.stream>>>(in, out, alpha, aux, beta,
                                                                    f.tw, f.kp);
  });
  IC_LAUNCHED();
}

// f(integral_constant<N>) for the sides of the fused planes.
template <class F>
void dispatch_plane(int n, F&& f) {
  switch (n) {
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    default: throw ApiError(-2, "fused z and y passes: n <= 128, and 256 in FP32");
  }
}

template <typename T>
bool fft_halo_x_apart(int n) {
  return fftk::ZYCfg<T, 256>::ok && n == 256;
}

template <typename T>
void fft_r2c_zy(const FftArgs<T>& f, const PlaneFwd<T>* fields, int m) {
  if (m < 1 || m > kMaxMul) throw ApiError(-1, "field count out of range");
  fftk::FwdSet<T> set{};
  for (int j = 0; j < m; ++j) set.f[j] = fields[j];
  const dim3 grid(f.n, m);
  fftk::with_flags(fields[0].hl != nullptr, fields[0].b != nullptr, [&](auto HL, auto B) {
    if constexpr (fftk::ZYCfg<T, 256>::ok) {
      if (f.n == 256) {
        using C = fftk::ZYCfg<T, 256>;
        fftk::k_r2c_zy<T, 256, HL.value, B.value>
            <<<grid, C::THREADS, 0, f.stream>>>(set, f.tw, f.kp);
        return;
      }
    }
    dispatch_plane(f.n, [&](auto NC) {
      constexpr int N = decltype(NC)::value;
      fftk::k_plane_fwd<T, N, HL.value, B.value>
          <<<grid, fftk::PlCfg<T, N>::THREADS, 0, f.stream>>>(set, f.tw, f.kp);
    });
  });
  IC_LAUNCHED();
}

template <typename T>
void fft_c2r_yz(const FftArgs<T>& f, const PlaneInv<T>* fields, int m, bool slab) {
  if (m < 1 || m > kMaxMul) throw ApiError(-1, "field count out of range");
  fftk::InvSet<T> set{};
  bool aux = false;
  for (int j = 0; j < m; ++j) {
    set.f[j] = fields[j];
    aux = aux || fields[j].aux;
  }
  if (!fft_zy_fused<T>(f.n, aux)) throw ApiError(-2, "fused y and z passes: unsupported");
  const dim3 grid(f.n, m);
  auto launch = [&](auto SL) {
    if constexpr (fftk::ZYCfg<T, 256>::ok) {
      if (f.n == 256) {
        using C = fftk::ZYCfg<T, 256>;
        fftk::k_c2r_yz<T, 256, SL.value><<<grid, C::THREADS, 0, f.stream>>>(set, f.tw, f.kp);
        return;
      }
    }
    dispatch_plane(f.n, [&](auto NC) {
      constexpr int N = decltype(NC)::value;
      fftk::k_plane_inv<T, N, SL.value>
          <<<grid, fftk::PlCfg<T, N>::THREADS, 0, f.stream>>>(set, f.tw, f.kp);
    });
  };
  if (slab)
    launch(std::true_type{});
  else
    launch(std::false_type{});
  IC_LAUNCHED();
}

template <typename T>
void fft_y(const FftArgs<T>& f, cx<T>* data, bool forward) {
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::SCfg<T, N>;
    const int K = N / 2 + 1, kp = f.kp;
    const int nlines = N * kp;
    const unsigned grid = blocks_for(nlines, C::LINES);
    if (forward)
      fftk::k_strided<T, N, true, false><<<grid, C::THREADS, 0, f.stream>>>(
          data, data, T(1), f.tw, nlines, kp, (long long)N * kp, kp, kp, K, yz_one<T>());
    else
      fftk::k_strided<T, N, false, false><<<grid, C::THREADS, 0, f.stream>>>(
          data, data, T(1), f.tw, nlines, kp, (long long)N * kp, kp, kp, K, yz_one<T>());
  });
  IC_LAUNCHED();
}

template <typename T>
void fft_y_inv(const FftArgs<T>& f, const cx<T>* in, cx<T>* out, const YZMul<T>& mul) {
  if (f.n <= 128) throw ApiError(-2, "multipliers of n <= 128 go through the fused planes");
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::SCfg<T, N>;
    const int K = N / 2 + 1, kp = f.kp;
    const int nlines = N * kp;
    fftk::k_strided<T, N, false, (N > 128)><<<blocks_for(nlines, C::LINES), C::THREADS, 0, f.stream>>>(
        in, out, T(1), f.tw, nlines, kp, (long long)N * kp, kp, kp, K, mul);
  });
  IC_LAUNCHED();
}

template <typename T>
void fft_x(const FftArgs<T>& f, const cx<T>* in, cx<T>* out, bool forward, T scale) {
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::SCfg<T, N>;
    const int K = N / 2 + 1, kp = f.kp;
    const int nlines = N * kp;
    const unsigned grid = blocks_for(nlines, C::LINES);
    if (forward)
      fftk::k_strided<T, N, true, false><<<grid, C::THREADS, 0, f.stream>>>(
          in, out, scale, f.tw, nlines, nlines, 0, nlines, kp, K, yz_one<T>());
    else
      fftk::k_strided<T, N, false, false><<<grid, C::THREADS, 0, f.stream>>>(
          in, out, scale, f.tw, nlines, nlines, 0, nlines, kp, K, yz_one<T>());
  });
  IC_LAUNCHED();
}

template <typename T>
void spectrum_pack(const FftArgs<T>& f, const cx<T>* stored, cx<T>* dense) {
  const int K = f.n / 2 + 1;
  const long long H = (long long)f.n * f.n * K;
  fftk::k_spec_copy<T, true><<<grid_for(H, 256), 256, 0, f.stream>>>(stored, dense, K, f.kp, H);
  IC_LAUNCHED();
}

template <typename T>
void spectrum_unpack(const FftArgs<T>& f, const cx<T>* dense, cx<T>* stored) {
  const int K = f.n / 2 + 1;
  const long long H = (long long)f.n * f.n * K;
  fftk::k_spec_copy<T, false><<<grid_for(H, 256), 256, 0, f.stream>>>(dense, stored, K, f.kp, H);
  IC_LAUNCHED();
}

template <typename T, int NIN>
void x_scatter(const FftArgs<T>& f, const fftk::InPtrs<T>& ip, const int* white, int div,
               const fftk::XOutSet<T>& set, int m) {
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::FCfg<T, N>;
    const int K = N / 2 + 1;
    const int nlines = N * f.kp;
    const unsigned blocks = blocks_for(nlines, C::LINES);
    const dim3 grid(blocks, blocks <= kSmallGrid ? m : 1);
    fftk::k_x_scatter<T, N, NIN><<<grid, C::THREADS, 0, f.stream>>>(
        ip, white[0], NIN == 2 ? white[1] : 0, div, set, m, f.wtab, f.tw, nlines, K, f.kp);
  });
  IC_LAUNCHED();
}

template <typename T>
void fft_x_scatter(const FftArgs<T>& f, const cx<T>* const* in, const int* white, int nin,
                   int div, const XOut<T>* outs, int m) {
  if (m < 1 || m > kMaxXOut || nin < 1 || nin > 2) throw ApiError(-1, "x pass out of range");
  require_apart<T>(in, nin, outs, m);
  fftk::InPtrs<T> ip{};
  for (int q = 0; q < nin; ++q) ip.p[q] = in[q];
  fftk::XOutSet<T> set{};
  for (int j = 0; j < m; ++j) {
    set.p[j] = outs[j].S;
    set.a[j][outs[j].px] = static_cast<T>(outs[j].a);
    set.b[j][outs[j].px] = static_cast<T>(outs[j].b);
  }
  if (nin == 1)
    x_scatter<T, 1>(f, ip, white, div, set, m);
  else
    x_scatter<T, 2>(f, ip, white, div, set, m);
}

template <typename T>
void fft_x_gather(const FftArgs<T>& f, const cx<T>* const* ins, const Mul* muls, int m,
                  cx<T>* out) {
  if (m < 1 || m > kMaxMul) throw ApiError(-1, "multiplier count out of range");
  fftk::InPtrs<T> ip{};
  fftk::GatherSet<T> gs{};
  const int white = muls[0].white, div = muls[0].div;
  for (int j = 0; j < m; ++j) {
    if (muls[j].white != white || muls[j].div != div)
      throw ApiError(-1, "multipliers of a gather share w and |k|^-2");
    ip.p[j] = ins[j];
    gs.cx[j][muls[j].px] = static_cast<T>(muls[j].scale);
    gs.cy[j][muls[j].py] = static_cast<T>(1);
    gs.cz[j][muls[j].pz] = static_cast<T>(1);
    gs.imag[j] = muls[j].imag;
  }
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::FCfg<T, N>;
    const int K = N / 2 + 1;
    const int nlines = N * f.kp;
    const unsigned blocks = blocks_for(nlines, C::LINES);
    if constexpr (N <= 64) {  // (128 and above: too many workgroups)
      const size_t lds = sizeof(cx<T>) * (N + (size_t)m * N * C::LP);
      if (gather_wide(blocks, m, C::THREADS, lds)) {
        fftk::k_x_gather_wide<T, N><<<blocks, C::THREADS * m, lds, f.stream>>>(
            ip, gs, white, div, m, out, f.wtab, f.tw, nlines, K, f.kp);
        return;
      }
    }
    fftk::k_x_gather<T, N><<<blocks, C::THREADS, 0, f.stream>>>(
        ip, gs, white, div, m, out, f.wtab, f.tw, nlines, K, f.kp);
  });
  IC_LAUNCHED();
}

template <typename T>
void fft_x_embed(const FftArgs<T>& f, cx<T>* S, const cx<T>* lo, int nl, T scale, T norm) {
  const int nlines = f.n * f.kp;
  fftk::dispatch_n<T>(f.n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    using C = fftk::FCfg<T, N>;
    fftk::k_x_embed<T, N><<<blocks_for(nlines, C::LINES), C::THREADS, 0, f.stream>>>(
        S, lo, nl, scale, norm, f.tw, nlines, f.n / 2 + 1, f.kp);
  });
  IC_LAUNCHED();
}

}  // namespace ic
