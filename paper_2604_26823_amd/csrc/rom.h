// Rank-order matching kernels (paper section 2.3.2): the elements of the
// real-space set (cells with R >= r_min) and of the Fourier-space k bins as
// sources and digits of the radix passes (sort.h), target draws, and the
// matched values' way back into the field (gfx950).
//
// The targets are values, and a descending key gives its value back, so they
// are sorted as keys alone and the last pass writes each one where the element
// of its rank lies: no orders of targets, no gathers through them.
#pragma once

#include "common.h"
#include "fields.h"
#include "sort.h"

namespace ic {
namespace rk {

// Real space, the stable partition that compacts the matched set: cell i with
// its descending value key; digit 0 on the set (R >= r_min), 1 (dropped) elsewhere.
template <typename T>
struct InSet {
  static constexpr int kDrop = 1;
  const T* R;
  T r_min;
  template <typename K>
  __device__ __forceinline__ unsigned operator()(K, uint32_t i) const {
    return R[i] >= r_min ? 0u : 1u;
  }
};

// Rank order: element index and value at each rank.
template <typename T>
struct ToRanks {
  uint32_t* idx;
  T* value;
  __device__ __forceinline__ void operator()(long long p, sk::key_t<T> key, uint32_t val,
                                             unsigned) const {
    idx[p] = val;
    value[p] = sk::key_value(key);
  }
};
// The same with the element's bin (the pass's digit).
template <typename T>
struct ToRanksAndBins {
  uint32_t* idx;
  T* value;
  uint32_t* bin;
  __device__ __forceinline__ void operator()(long long p, sk::key_t<T> key, uint32_t val,
                                             unsigned d) const {
    idx[p] = val;
    value[p] = sk::key_value(key);
    bin[p] = d;
  }
};
// out[idx[p]] = the value at rank p: the j-th largest target to the element
// of rank j.
template <typename T>
struct ToElements {
  T* out;
  const uint32_t* idx;
  __device__ __forceinline__ void operator()(long long p, sk::key_t<T> key, uint32_t,
                                             unsigned) const {
    out[idx[p]] = sk::key_value(key);
  }
};

// Descending keys of the real-space set's targets: N(0,1) draw j.
template <typename T>
__global__ void k_real_targets(uint64_t event, uint64_t seed, sk::key_t<T>* __restrict__ keys,
                               long long n) {
  for (long long j = blockIdx.x * (long long)blockDim.x + threadIdx.x; j < n;
       j += (long long)gridDim.x * blockDim.x)
    keys[j] =
        sk::descending_key<T>(static_cast<T>(fk::philox_draw(0, (uint64_t)j, 0, 2, event, seed)));
}

// k bin of every squared wave number n2 (in units of the fundamental mode):
// equal widths dk from k_min, 255 below k_min.
static __global__ void k_bin_table(int len, double kf, double kmin, double dk, int nbins,
                                   uint8_t* __restrict__ tab) {
  const int n2 = blockIdx.x * blockDim.x + threadIdx.x;
  if (n2 >= len) return;
  const double k = kf * sqrt(static_cast<double>(n2));
  int b = 255;
  if (!(k < kmin)) {
    b = static_cast<int>(floor((k - kmin) / dk));
    b = b < nbins - 1 ? b : nbins - 1;
  }
  tab[n2] = static_cast<uint8_t>(b);
}

// Half-spectrum modes f = (kx n + ky) K + kz, K = n/2 + 1.
constexpr int kModeBits = 28;  // f < 2^kModeBits
struct Modes {
  int n, K;
  uint64_t magic;      // ceil(2^40 / K): f / K = f magic >> 40 for f < 2^kModeBits
  const uint8_t* tab;  // k_bin_table
  struct At {
    uint32_t r, kz;  // f = r K + kz
    int kx, ky;
  };
  __device__ __forceinline__ At at(uint32_t f) const {
    At a;
    a.r = static_cast<uint32_t>((f * magic) >> 40);
    a.kz = f - a.r * K;
    a.ky = static_cast<int>(a.r & (n - 1));
    a.kx = static_cast<int>(a.r / static_cast<unsigned>(n));
    return a;
  }
  // whether the mode's conjugate partner is stored too (kz = 0 and n/2 planes)
  __device__ __forceinline__ bool edge(const At& a) const {
    return a.kz == 0 || a.kz == static_cast<uint32_t>(n / 2);
  }
  // row (kx n + ky) of the conjugate partner
  __device__ __forceinline__ uint32_t conj_row(const At& a) const {
    return static_cast<uint32_t>(((n - a.kx) & (n - 1)) * n + ((n - a.ky) & (n - 1)));
  }
  // k bin of an independent mode with |k| >= k_min, else 255
  __device__ __forceinline__ unsigned bin(const At& a) const {
    if (edge(a) && a.r >= conj_row(a)) return 255u;
    const int ix = a.kx < n / 2 ? a.kx : a.kx - n;
    const int iy = a.ky < n / 2 ? a.ky : a.ky - n;
    const int iz = static_cast<int>(a.kz);
    return tab[ix * ix + iy * iy + iz * iz];
  }
};
inline Modes make_modes(int n, const uint8_t* tab) {
  const int K = n / 2 + 1;
  return Modes{n, K, ((1ull << 40) + K - 1) / K, tab};
}

// The bin of the mode of element val (parts: element 2 f + c of mode f).
struct ByBin {
  static constexpr int kDrop = 255;
  Modes m;
  int parts;  // 1: elements are the real and imaginary parts
  template <typename K>
  __device__ __forceinline__ unsigned operator()(K, uint32_t e) const {
    return m.bin(m.at(parts ? e >> 1 : e));
  }
};

// Descending keys of every mode's amplitude |z| = |Z_f| scale (parts = 0) or
// of its real and imaginary parts times scale (elements 2 f and 2 f + 1).
template <typename T>
__global__ void k_mode_keys(const cx<T>* __restrict__ Z, Modes m, int kp, T scale, int parts,
                            sk::key_t<T>* __restrict__ keys, long long H) {
  for (long long f = blockIdx.x * (long long)blockDim.x + threadIdx.x; f < H;
       f += (long long)gridDim.x * blockDim.x) {
    const Modes::At a = m.at(static_cast<uint32_t>(f));
    const cx<T> z = Z[(long long)a.r * kp + a.kz];
    if (parts) {
      keys[2 * f] = sk::descending_key<T>(z.x * scale);
      keys[2 * f + 1] = sk::descending_key<T>(z.y * scale);
    } else {
      keys[f] = sk::descending_key<T>(sqrt(z.x * z.x + z.y * z.y) * scale);
    }
  }
}

// start[b] = first rank of bin b (exclusive scan of the bins' element counts).
static __global__ __launch_bounds__(sk::kDigits) void k_bin_starts(
    const uint32_t* __restrict__ count, uint32_t* __restrict__ start) {
  __shared__ uint32_t wsum[sk::kDigits / 64];
  const uint32_t c = count[threadIdx.x];
  start[threadIdx.x] = sk::scan_digits(c, wsum);
}

// Target of rank i: bin b (the last with start[b] <= i), index within the bin
// j = i - start[b], draw kind (1 = Rayleigh, 0 = normal) of the given stream
// times mult; its descending key, and the bin as payload.
template <typename T>
__global__ void k_fourier_targets(const uint32_t* __restrict__ start, int nbins, int kind,
                                  uint64_t stream, double mult, uint64_t event, uint64_t seed,
                                  sk::key_t<T>* __restrict__ keys, uint32_t* __restrict__ bins,
                                  long long n) {
  __shared__ uint32_t st[sk::kDigits];
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) st[b] = start[b];
  __syncthreads();
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    int lo = 0, hi = nbins;  // st[lo] <= i < st[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (st[mid] <= static_cast<uint32_t>(i))
        lo = mid;
      else
        hi = mid;
    }
    const uint64_t j = static_cast<uint64_t>(i) - st[lo];
    keys[i] = sk::descending_key<T>(
        static_cast<T>(fk::philox_draw(kind, j, lo, stream, event, seed) * mult));
    bins[i] = static_cast<uint32_t>(lo);
  }
}

// The matched values back into the spectrum, in one streaming pass (a scatter
// of whole modes through the ranks took 354 us at 256^3 in FP32; values go
// through ToElements, four bytes each): Z_f <- tau unscale Z_f / |Z_f| (tau
// unscale when Z_f = 0), or with parts its real and imaginary parts replaced;
// matched modes of the kz = 0 and kz = n/2 planes also set their conjugate
// partner, which is no matched mode itself.
template <typename T>
__global__ void k_modes_back(cx<T>* __restrict__ Z, Modes m, int kp, const T* __restrict__ tau,
                             T unscale, int parts, long long H) {
  for (long long f = blockIdx.x * (long long)blockDim.x + threadIdx.x; f < H;
       f += (long long)gridDim.x * blockDim.x) {
    const Modes::At a = m.at(static_cast<uint32_t>(f));
    if (m.bin(a) == 255u) continue;
    cx<T>* zp = Z + (long long)a.r * kp + a.kz;
    cx<T> v;
    if (parts) {
      v = mkc<T>(tau[2 * f] * unscale, tau[2 * f + 1] * unscale);
    } else {
      const cx<T> z = *zp;
      const T t = tau[f] * unscale;
      const T q = sqrt(z.x * z.x + z.y * z.y);
      v = q > T(0) ? mkc<T>(z.x * (t / q), z.y * (t / q)) : mkc<T>(t, T(0));
    }
    *zp = v;
    if (m.edge(a)) Z[(long long)m.conj_row(a) * kp + a.kz] = mkc<T>(v.x, -v.y);
  }
}

}  // namespace rk
}  // namespace ic
