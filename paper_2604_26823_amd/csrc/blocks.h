// Eulerian block ordering of the particles (gfx950).
//
// The grid is cut into 8^3-cell blocks.  Every particle belongs to the block
// of its CIC base cell (the wrapped floor cell of its position), so all eight
// corners of its stencil fall inside that block extended by one cell on the
// upper side: a fixed 9^3-cell window.  After each drift the particles are
// counting-sorted by block (per-block counts with wavefront- or workgroup-aggregated
// atomics, an exclusive scan, then a scatter of the ids alone, with the new
// order's map back to the old: the density paint reads the new positions
// through that map and stores them in the new order, the next step reads the
// momenta through it; states that must be complete in their order move
// positions and momenta too), and every paint and readout then runs over work
// items of at most 1024 particles of one block, with the block's window in
// LDS:
//   * paints accumulate in LDS windows (FP64 adds for FP64 grids, exact
//     64-bit fixed-point adds for FP32 grids, see WinAcc); a block's only
//     item stores its 8^3 own cells (the items of a block with several add
//     them atomically), its halo into fields of their own (halo.h) that
//     the consumer adds while reading: global float
//     atomics are served past the XCD's L2 and were the paints' largest
//     cost;
//   * gathers read their mesh fields from a window loaded with coalesced
//     loads.
// Unlike windows around Lagrangian patches, these windows cannot overflow,
// however far particles have moved or however strongly they cluster: a dense
// block simply yields more work items.
//
// The order inside a block follows the atomic ranks, so it can differ from
// run to run; the results then differ only by FP64 summation order in the
// LDS windows before the single rounding to the mesh type, and by the order
// of the global atomics, which is unordered anyway.
//
// Slot a of a sorted state holds the particle with Lagrangian index ids[a];
// dest[a] gives its slot in the next order.  The adjoint kernels of order n
// read the cotangents left in order n + 1 through dest and write them in
// order n, so no pass of its own moves them between orders (one gather takes
// order 0 back to the lattice order).
#pragma once

#include <type_traits>

#include "fixed.h"
#include "halo.h"
#include "particles.h"

namespace ic {
namespace bk {

using pk::Grid;
using pk::Stencil;

constexpr int kLB = 3;                 // log2 of the block side in cells
constexpr int kB = 1 << kLB;           // block side
constexpr int kW = kB + 1;             // window side
constexpr int kWin = kW * kW * kW;     // window cells (729)
constexpr int kThreads = 256;
constexpr int kPer = 4;                // particles per thread
constexpr int kChunk = kThreads * kPer;  // particles per work item

// Blocks of one grid of side 2^lm (lm >= 3), and how its fields lie in memory:
// [x][y][z], or in slabs [z / 8][x][y][z mod 8].  The force mesh is in
// slabs (its fields pass between the paints, the FFT's z passes and the
// readouts only): a block's window is then nine runs of 72 cells and one of
// nine cells 32 bytes apart per x, where [x][y][z] makes it 81 rows of nine
// cells, each in a 128-byte line of its own, and the planes x of a window lie
// 32 n bytes apart instead of 4 n^2 (FP32).  Loading those rows cost 120 us of the 345 us step and
// 150 us of the 389 us force adjoint at 256^3 in FP32, several times what the
// bytes take.
struct Layout {
  int lm;     // log2 of the grid side
  int lnb;    // log2 of the blocks per side
  int slabs;  // 1: fields in slabs
};

inline Layout layout_for(int lm, bool slabs) { return Layout{lm, lm - kLB, slabs ? 1 : 0}; }
// Index of cell (x, y, z).
__device__ __forceinline__ unsigned cell_at(unsigned x, unsigned y, unsigned z, const Layout& L) {
  return L.slabs ? ((((z >> kLB) << L.lm | x) << L.lm | y) << kLB) | (z & (kB - 1))
                 : (x << L.lm | y) << L.lm | z;
}
inline unsigned block_count(const Layout& L) { return 1u << (3 * L.lnb); }
// Upper bound of the work items of P particles: each non-empty block gives
// ceil(count / kChunk) <= count / kChunk + 1 items.
inline unsigned max_items(const Layout& L, long long P) {
  return static_cast<unsigned>((P + kChunk - 1) / kChunk) + block_count(L);
}
// Workgroups of an item kernel: the item bound plus the slack of the XCD
// dealing (item_of).
inline unsigned item_grid(const Layout& L, long long P) { return max_items(L, P) + 8; }

// Up to six field pointers of one state array set.
template <typename T>
struct Ptrs {
  const T* p[6];
};
template <typename T>
struct MPtrs {
  T* p[6];
};

// Block of the (wrapped) base cell of stencil s; wraps s.i0 in place.
template <typename T>
__device__ __forceinline__ unsigned block_of(Stencil<T>& s, const Layout& L) {
  const int mask = (1 << L.lm) - 1;
#pragma unroll
  for (int a = 0; a < 3; ++a) s.i0[a] &= mask;
  return (static_cast<unsigned>(s.i0[0] >> kLB) << (2 * L.lnb)) |
         (static_cast<unsigned>(s.i0[1] >> kLB) << L.lnb) |
         static_cast<unsigned>(s.i0[2] >> kLB);
}

// Origin (cell coordinates) of block b.
__device__ __forceinline__ void block_origin(unsigned b, const Layout& L, int o[3]) {
  const unsigned m = (1u << L.lnb) - 1;
  o[0] = static_cast<int>(b >> (2 * L.lnb)) << kLB;
  o[1] = static_cast<int>((b >> L.lnb) & m) << kLB;
  o[2] = static_cast<int>(b & m) << kLB;
}

// Window index of unwrapped cell c relative to origin o (c - o in [0, 8]).
__device__ __forceinline__ int win_index(const int o[3], int cx, int cy, int cz) {
  return ((cx - o[0]) * kW + (cy - o[1])) * kW + (cz - o[2]);
}

// Mesh index of window cell k of the window at origin o.
__device__ __forceinline__ unsigned win_cell(const int o[3], int k, const Layout& L) {
  const unsigned mask = (1u << L.lm) - 1;
  const int kx = k / (kW * kW), r = k - kx * kW * kW;
  const int ky = r / kW, kz = r - ky * kW;
  return cell_at(static_cast<unsigned>(o[0] + kx) & mask, static_cast<unsigned>(o[1] + ky) & mask,
                 static_cast<unsigned>(o[2] + kz) & mask, L);
}

// Lanes of the wavefront grouped by key with ballots: each active lane gets
// its group's first lane (leader) and its offset within the group, and the
// leader also gets the group size (0 elsewhere).  Every lane of the wavefront
// must call it; inactive lanes pass active = false.
struct RankTicket {
  unsigned base;  // the leader's reservation (atomic result), valid in leaders
  int leader;
  unsigned off;
};

__device__ __forceinline__ RankTicket group_by_key(unsigned key, bool active, unsigned& size) {
  const int lane = static_cast<int>(threadIdx.x & 63);
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  unsigned long long todo = __ballot(active);
  RankTicket t{0u, 0, 0u};
  size = 0;
  while (todo) {
    const int leader = __ffsll(static_cast<long long>(todo)) - 1;
    const unsigned k = static_cast<unsigned>(__shfl(static_cast<int>(key), leader, 64));
    const unsigned long long same = __ballot(active && key == k);
    if (lane == leader) size = static_cast<unsigned>(__popcll(same));
    if (active && key == k) {
      t.leader = leader;
      t.off = static_cast<unsigned>(__popcll(same & below));
    }
    todo &= ~same;
  }
  return t;
}

// Rank of this lane's particle within its block: each group's leader adds
// the group size to the block count, all groups in the same atomic
// instruction (one round trip whatever the number of distinct keys), and the
// lanes of a group take consecutive ranks from the leader's result.
// Inactive lanes get 0.
__device__ __forceinline__ unsigned rank_in_block(unsigned key, bool active,
                                                  unsigned* __restrict__ count) {
  unsigned size;
  RankTicket t = group_by_key(key, active, size);
  if (size) t.base = atomicAdd(count + key, size);
  const unsigned base = static_cast<unsigned>(__shfl(static_cast<int>(t.base), t.leader, 64));
  return active ? base + t.off : 0u;
}

// Ranks aggregated over a workgroup whose particles all start in block b0:
// after a drift nearly every particle is in b0 or one of its 26 neighbours,
// so particles reserve offsets on 27 LDS counters, and one thread per
// non-empty counter then reserves the workgroup's range in that block's
// global count with one atomic and leaves its first rank in the work item's
// row of a table (kNbrRow entries).  A particle keeps its neighbour slot and
// its offset within the workgroup, packed in one word (key and rank took
// two); the sort that follows adds the table's entry, so nothing in the
// counting kernel waits for the global atomics.  Keys farther away take a
// global atomic each and keep their key in an array of their own.
constexpr int kNbrRow = 32;   // table entries per work item
constexpr int kRankBits = 27;  // packed word: slot << kRankBits | rank (P <= 2^27)
constexpr int kNbr = 27;

// Neighbour slot (0..26) of block key relative to block b0, or kNbr if the
// blocks are not adjacent (periodic block grid of side 2^lnb).
__device__ __forceinline__ int neighbour_slot(unsigned b0, unsigned key, const Layout& L) {
  const unsigned m = (1u << L.lnb) - 1;
  int slot = 0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    const int sh = (2 - ax) * L.lnb;
    const unsigned d = ((key >> sh) - (b0 >> sh)) & m;
    int dd;
    if (d <= 1u) dd = static_cast<int>(d);
    else if (d == m) dd = -1;
    else return kNbr;
    slot = slot * 3 + dd + 1;
  }
  return slot;
}

// Block key of neighbour slot s of block b0.
__device__ __forceinline__ unsigned neighbour_key(unsigned b0, int s, const Layout& L) {
  const unsigned m = (1u << L.lnb) - 1;
  const int dd[3] = {s / 9 - 1, (s / 3) % 3 - 1, s % 3 - 1};
  unsigned key = 0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    const int sh = (2 - ax) * L.lnb;
    key |= ((((b0 >> sh) & m) + static_cast<unsigned>(dd[ax])) & m) << sh;
  }
  return key;
}

// First half.  Most particles of a wavefront stay in block b0 (a drift moves
// them by a fraction of the block's eight cells): their lanes take offsets
// from one ballot and one reservation by the first of them.  Every other lane
// reserves for itself, all lanes in the same instruction, on the workgroup
// counter of its neighbour slot or, farther away, on the global count.  All
// of a thread's reservations can be in flight at once.
constexpr int kStay = kNbr / 2;  // slot of b0 itself
__device__ __forceinline__ RankTicket rank_issue_wg(unsigned key, int slot, bool active,
                                                    unsigned* __restrict__ count,
                                                    unsigned* wcnt) {
  const int lane = static_cast<int>(threadIdx.x & 63);
  const unsigned long long stay = __ballot(active && slot == kStay);
  RankTicket t{0u, lane, 0u};
  unsigned size = 1u;
  bool reserve = active;
  if (slot == kStay) {
    t.leader = stay ? __ffsll(static_cast<long long>(stay)) - 1 : lane;
    t.off = __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(stay >> 32),
                                      __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(stay), 0u));
    size = static_cast<unsigned>(__popcll(stay));
    reserve = active && lane == t.leader;
  }
  if (reserve) {
    if (slot < kNbr)
      t.base = atomicAdd(wcnt + slot, size);
    else
      t.base = atomicAdd(count + key, size);
  }
  return t;
}

__device__ __forceinline__ unsigned rank_of(const RankTicket& t) {
  return static_cast<unsigned>(__shfl(static_cast<int>(t.base), t.leader, 64)) + t.off;
}

// Second half, after a barrier: the workgroup's ranges into the item's row.
__device__ __forceinline__ void rank_reserve_wg(unsigned b0, const Layout& L,
                                                unsigned* __restrict__ count, const unsigned* wcnt,
                                                unsigned* __restrict__ row) {
  const int t = static_cast<int>(threadIdx.x);
  if (t < kNbr && wcnt[t]) row[t] = atomicAdd(count + neighbour_key(b0, t, L), wcnt[t]);
}

// ---------------------------------------------------------------- sorting
// Particle of thread a when a kernel goes over the lattice to or from a block order:
// a wavefront takes 8 x 4 x 2 (z, y, x) neighbouring sites, and consecutive
// wavefronts follow along z.  Its particles are then in one block or a few, so
// they get their ranks with as many atomics and their slots are a few
// contiguous runs.  Wavefronts along z (64 sites: 8 blocks, or 16 when the mesh is twice
// the lattice) gave every block runs of eight or four.
__device__ __forceinline__ long long tile_site(long long a, int lp) {
  const unsigned lane = static_cast<unsigned>(a) & 63u, t = static_cast<unsigned>(a >> 6);
  const unsigned z = (t & ((1u << (lp - 3)) - 1)) << 3 | (lane & 7u);
  const unsigned y = ((t >> (lp - 3)) & ((1u << (lp - 2)) - 1)) << 2 | (lane >> 3 & 3u);
  const unsigned x = t >> (2 * lp - 5) << 1 | lane >> 5;
  return static_cast<long long>((x << lp | y) << lp | z);
}

// Key and rank of every slot: the block of the stencil of displacement d
// (particle ids[a] in slot a; when ids is null, thread a's is tile_site(a) and d
// is in lattice order) on grid g.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_keys(const T* __restrict__ d,
                                                   const unsigned* __restrict__ ids, long long P,
                                                   int lp, Grid<T> g, Layout L,
                                                   unsigned* __restrict__ count,
                                                   unsigned* __restrict__ key,
                                                   unsigned* __restrict__ rank) {
  const long long a = blockIdx.x * (long long)kThreads + threadIdx.x;
  const bool ok = a < P;
  unsigned b = 0;
  if (ok) {
    const long long j = ids ? static_cast<long long>(ids[a]) : tile_site(a, lp);
    int idx[3];
    pk::lattice(j, lp, idx);
    T dsp[3];
    pk::load3(d, P, ids ? a : j, dsp);
    Stencil<T> s = pk::stencil(idx, g.ratio, dsp, g.inv_cell, g.cell);
    b = block_of(s, L);
  }
  const unsigned r = rank_in_block(b, ok, count);
  if (ok) {
    key[a] = b;
    rank[a] = r;
  }
}

// Exclusive scan of the per-block counts and item counts
// (ceil(count / kChunk)) in three phases: chunk sums, a one-workgroup scan
// of the chunk sums, and the chunk-local scans with their offsets.  start and
// istart get nb + 1 entries (the last = the totals).
constexpr int kScanChunk = 2048;  // blocks per chunk (256 threads x 8)

static __global__ __launch_bounds__(256) void k_scan_sums(const unsigned* __restrict__ count,
                                                   unsigned nb, uint2* __restrict__ sums) {
  __shared__ unsigned sc[256], si[256];
  unsigned c = 0, it = 0;
  const unsigned base = blockIdx.x * kScanChunk;
  for (int j = 0; j < kScanChunk / 256; ++j) {
    const unsigned i = base + j * 256 + threadIdx.x;
    if (i < nb) {
      const unsigned v = count[i];
      c += v;
      it += (v + kChunk - 1) / kChunk;
    }
  }
  sc[threadIdx.x] = c;
  si[threadIdx.x] = it;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      sc[threadIdx.x] += sc[threadIdx.x + s];
      si[threadIdx.x] += si[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = make_uint2(sc[0], si[0]);
}

// In-place exclusive scan of n <= 1024 pairs by one workgroup of 1024 threads.
static __global__ __launch_bounds__(1024) void k_scan_top(uint2* __restrict__ sums, unsigned n) {
  __shared__ unsigned a[1024], b[1024];
  const unsigned t = threadIdx.x;
  const uint2 v = t < n ? sums[t] : make_uint2(0u, 0u);
  a[t] = v.x;
  b[t] = v.y;
  __syncthreads();
  for (unsigned off = 1; off < 1024; off <<= 1) {
    const unsigned xa = t >= off ? a[t - off] : 0u, xb = t >= off ? b[t - off] : 0u;
    __syncthreads();
    a[t] += xa;
    b[t] += xb;
    __syncthreads();
  }
  if (t < n) sums[t] = make_uint2(a[t] - v.x, b[t] - v.y);
}

static __global__ __launch_bounds__(256) void k_scan_out(const unsigned* __restrict__ count, unsigned nb,
                                                  const uint2* __restrict__ sums,
                                                  unsigned* __restrict__ start,
                                                  unsigned* __restrict__ istart) {
  __shared__ unsigned sc[256], si[256];
  constexpr int kPerT = kScanChunk / 256;
  const unsigned base = blockIdx.x * kScanChunk + threadIdx.x * kPerT;
  unsigned c[kPerT], it[kPerT], tc = 0, ti = 0;
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const unsigned i = base + j;
    const unsigned v = i < nb ? count[i] : 0u;
    c[j] = v;
    it[j] = (v + kChunk - 1) / kChunk;
    tc += c[j];
    ti += it[j];
  }
  sc[threadIdx.x] = tc;
  si[threadIdx.x] = ti;
  __syncthreads();
  for (unsigned off = 1; off < 256; off <<= 1) {
    const unsigned xa = threadIdx.x >= off ? sc[threadIdx.x - off] : 0u;
    const unsigned xb = threadIdx.x >= off ? si[threadIdx.x - off] : 0u;
    __syncthreads();
    sc[threadIdx.x] += xa;
    si[threadIdx.x] += xb;
    __syncthreads();
  }
  unsigned oc = sums[blockIdx.x].x + sc[threadIdx.x] - tc;
  unsigned oi = sums[blockIdx.x].y + si[threadIdx.x] - ti;
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const unsigned i = base + j;
    if (i < nb) {
      start[i] = oc;
      istart[i] = oi;
    }
    oc += c[j];
    oi += it[j];
    if (i + 1 == nb) {
      start[nb] = oc;
      istart[nb] = oi;
    }
  }
}

// One work item: block b, its slots [s0, s1) and its index i (kSingle set when
// it is the block's only item).  s0 = s1 marks the workgroups past the last.
constexpr unsigned kSingle = 1u << 31;
constexpr int kXcds = 8;

// Work items istart[b] + j, slots [start[b] + j kChunk, ...) of every block, in
// two orders of nwg = item_grid() records, one per workgroup: by_index in
// index order, by_xcd dealt so that each XCD gets a contiguous range (see
// item_of).  A workgroup then starts with one 16-byte load; looking up the
// item count, the item and the block's slots took three dependent ones.  The
// counts are left zeroed for the next order.
__device__ __forceinline__ void write_items(unsigned b, unsigned s0, unsigned s1, unsigned i,
                                            unsigned per, uint4* __restrict__ by_index,
                                            uint4* __restrict__ by_xcd) {
  const unsigned flag = s1 - s0 <= static_cast<unsigned>(kChunk) ? kSingle : 0u;
  for (unsigned s = s0; s < s1; s += kChunk, ++i) {
    const uint4 v = make_uint4(b, s, min(s + kChunk, s1), i | flag);
    by_index[i] = v;
    by_xcd[(i % per) * kXcds + i / per] = v;
  }
}
// The records of the workgroups past the n items.
__device__ __forceinline__ void write_ends(unsigned n, unsigned per, unsigned nwg, unsigned t0,
                                           unsigned step, uint4* __restrict__ by_index,
                                           uint4* __restrict__ by_xcd) {
  for (unsigned w = t0; w < nwg; w += step) {
    if (w >= n) by_index[w] = make_uint4(0u, 0u, 0u, 0u);
    if (w / kXcds >= per || (w % kXcds) * per + w / kXcds >= n)
      by_xcd[w] = make_uint4(0u, 0u, 0u, 0u);
  }
}
static __global__ __launch_bounds__(256) void k_fill_items(const unsigned* __restrict__ start,
                                                    const unsigned* __restrict__ istart,
                                                    unsigned nb, unsigned nwg,
                                                    uint4* __restrict__ by_index,
                                                    uint4* __restrict__ by_xcd,
                                                    unsigned* __restrict__ count) {
  const unsigned n = istart[nb];
  const unsigned per = (n + kXcds - 1) / kXcds;
  const unsigned t0 = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
  for (unsigned b = t0; b < nb; b += step) {
    write_items(b, start[b], start[b + 1], istart[b], per, by_index, by_xcd);
    count[b] = 0u;
  }
  write_ends(n, per, nwg, t0, step, by_index, by_xcd);
}

// The scan and the items of an order of at most kOneBlocks blocks (grids up to
// 128^3) by one workgroup: the four launches of the general path, three of them
// scans of a few thousand counts, took 12 us of every step at 32^3 and 64^3 (a
// paint of 32^3 particles 26.9 us instead of 34.5, of 128^3 89 instead of 94).  The
// 32768 blocks of a 256^3 grid are too many for one: that paint would go from 513 to 692 us.
constexpr unsigned kOneThreads = 1024;
constexpr unsigned kOnePer = 4;
constexpr unsigned kOneBlocks = kOneThreads * kOnePer;
static __global__ __launch_bounds__(kOneThreads) void k_order_one(
    unsigned* __restrict__ count, unsigned nb, unsigned nwg, unsigned* __restrict__ start,
    unsigned* __restrict__ istart, uint4* __restrict__ by_index, uint4* __restrict__ by_xcd) {
  __shared__ unsigned long long wsum[kOneThreads / 64];
  const unsigned t = threadIdx.x, lane = t & 63, w = t >> 6;
  unsigned c[kOnePer];
  unsigned long long sum = 0;  // items << 32 | particles
#pragma unroll
  for (unsigned j = 0; j < kOnePer; ++j) {
    const unsigned b = t * kOnePer + j;
    c[j] = b < nb ? count[b] : 0u;
    sum += static_cast<unsigned long long>((c[j] + kChunk - 1) / kChunk) << 32 | c[j];
  }
  unsigned long long s = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long o = __shfl_up(s, off, 64);
    if (lane >= static_cast<unsigned>(off)) s += o;
  }
  if (lane == 63) wsum[w] = s;
  __syncthreads();
  unsigned long long before = 0, total = 0;
  for (unsigned q = 0; q < kOneThreads / 64; ++q) {
    before += q < w ? wsum[q] : 0ull;
    total += wsum[q];
  }
  s += before - sum;
  const unsigned n = static_cast<unsigned>(total >> 32);
  const unsigned per = (n + kXcds - 1) / kXcds;
  unsigned p = static_cast<unsigned>(s), i = static_cast<unsigned>(s >> 32);
#pragma unroll
  for (unsigned j = 0; j < kOnePer; ++j) {
    const unsigned b = t * kOnePer + j;
    if (b >= nb) break;
    start[b] = p;
    istart[b] = i;
    count[b] = 0u;
    write_items(b, p, p + c[j], i, per, by_index, by_xcd);
    p += c[j];
    i += (c[j] + kChunk - 1) / kChunk;
  }
  if (t == 0) {
    start[nb] = static_cast<unsigned>(total);
    istart[nb] = n;
  }
  write_ends(n, per, nwg, t, kOneThreads, by_index, by_xcd);
}

// Moves nf fields (and the ids) of slot q to slot start[key[a]] + rank[a] of
// the new order; dest[q] receives that slot.  q is a, or tile_site(a) when ids_src
// is null (the lattice order, id = slot).
// (Keys and ranks of k_keys; the moves between block orders are k_scatter_b.)
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scatter(
    const unsigned* __restrict__ key, const unsigned* __restrict__ rank,
    const unsigned* __restrict__ start, Ptrs<T> src, MPtrs<T> dst, int nf,
    const unsigned* __restrict__ ids_src, unsigned* __restrict__ ids_dst,
    unsigned* __restrict__ dest, long long P, int lp) {
  const long long a = blockIdx.x * (long long)kThreads + threadIdx.x;
  if (a >= P) return;
  const long long q = ids_src ? a : tile_site(a, lp);
  const unsigned s = start[key[a]] + rank[a];
  for (int f = 0; f < nf; ++f) dst.p[f][s] = src.p[f][q];
  ids_dst[s] = ids_src ? ids_src[a] : static_cast<unsigned>(q);
  dest[q] = s;
}

// dst_f[q] = src_f[dest[q]] for nf fields, q = tile_site(a): values of order 0
// brought back to the lattice order.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_gather_back(const unsigned* __restrict__ dest,
                                                          Ptrs<T> src, MPtrs<T> dst, int nf,
                                                          long long P, int lp) {
  const long long a = blockIdx.x * (long long)kThreads + threadIdx.x;
  if (a >= P) return;
  const long long q = tile_site(a, lp);
  const unsigned s = dest[q];
  for (int f = 0; f < nf; ++f) dst.p[f][q] = src.p[f][s];
}

// dst_f[ids[a]] = src_f[a]: a sorted state back to lattice order.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_to_lattice(const unsigned* __restrict__ ids,
                                                         Ptrs<T> src, MPtrs<T> dst, int nf,
                                                         long long P) {
  const long long a = blockIdx.x * (long long)kThreads + threadIdx.x;
  if (a >= P) return;
  const unsigned j = ids[a];
  for (int f = 0; f < nf; ++f) dst.p[f][j] = src.p[f][a];
}

// ------------------------------------------------------------ work items
// Records of the order's work items (k_fill_items) and its particle ids.
struct Items {
  const uint4* by_index;
  const uint4* by_xcd;
  const unsigned* ids;
};

// Block, origin and slot range of this workgroup's item; false (for the
// whole workgroup) past the last item.  Workgroups are dealt to the eight
// XCDs round-robin (workgroup w runs on XCD w mod 8).  Gathers (CONTIG) take
// item (w mod 8) per + w / 8 with per = ceil(items / 8), so each XCD walks
// one contiguous range of neighbouring blocks whose windows share cache
// lines in that XCD's L2; paints take item w, so neighbouring blocks, whose
// flushes add into the same halo cells, run on different XCDs and their
// atomics do not queue behind each other.  The grid must hold item_grid()
// workgroups, as many as there are records.
struct Item {
  unsigned b;
  int o[3];
  unsigned s0, s1;
  unsigned i;       // item index
  bool single;      // the block's only item (it holds at most kChunk particles)
};

template <bool CONTIG>
__device__ __forceinline__ bool item_of(const Items& it, const Layout& L, Item& m) {
  const uint4 v = (CONTIG ? it.by_xcd : it.by_index)[blockIdx.x];
  if (v.y == v.z) return false;
  m.b = v.x;
  m.s0 = v.y;
  m.s1 = v.z;
  m.i = v.w & ~kSingle;
  m.single = (v.w & kSingle) != 0;
  block_origin(m.b, L, m.o);
  return true;
}

// Block of the grid of layout Ld (side 2^rs times smaller) that holds the
// item's block's origin: the centre of the neighbour slots.
__device__ __forceinline__ unsigned block_around(const Item& m, const Layout& Ld, int rs) {
  return ((static_cast<unsigned>(m.o[0] >> rs) >> kLB) << (2 * Ld.lnb)) |
         ((static_cast<unsigned>(m.o[1] >> rs) >> kLB) << Ld.lnb) |
         (static_cast<unsigned>(m.o[2] >> rs) >> kLB);
}

// f(R) with R = ceil(particles / kThreads) <= kPer as a compile-time constant.
// A block of the mean density holds two particles per thread, and rounds past
// its end would still issue their loads, so the kernels load by rounds (step
// and force adjoint 2 % faster in FP32, 2 and 3 % in FP64).  Only loads: arithmetic compiled once per R could round differently in each, and
// which particles of a dense block share an item differs from run to run.
template <class F>
__device__ __forceinline__ void with_rounds(const Item& m, F&& f) {
  switch ((m.s1 - m.s0 + kThreads - 1) / kThreads) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    default: f(std::integral_constant<int, kPer>{}); break;
  }
}

// Slots a[k] = s0 + threadIdx.x + k kThreads of this thread in the item and
// whether they hold a particle; slots past the item's end are clamped to its
// first slot (an item is never empty).  The kernels issue the loads of all
// R particles from these slots in one branch-free run and wait once:
// behind a branch per particle, the in-order memory counter made every
// particle's loads wait for all of the previous particle's.
template <int R>
__device__ __forceinline__ void item_slots(const Item& m, long long (&a)[R], bool (&ok)[R]) {
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const long long s = static_cast<long long>(m.s0) + threadIdx.x + k * kThreads;
    ok[k] = s < static_cast<long long>(m.s1);
    a[k] = ok[k] ? s : static_cast<long long>(m.s0);
  }
}

// u[k] = map[a[k]] for k < R (particle ids, slot maps).
template <int R, int N>
__device__ __forceinline__ void load_u32(const unsigned* __restrict__ map,
                                         const long long (&a)[N], unsigned (&u)[N]) {
#pragma unroll
  for (int k = 0; k < R; ++k) u[k] = map[a[k]];
}

// v[k] = the three fields of f (P apart) at slot s[k], k < R.
template <int R, typename T, typename S, int N>
__device__ __forceinline__ void load3_at(const T* __restrict__ f, long long P,
                                         const S (&s)[N], T (&v)[N][3]) {
#pragma unroll
  for (int k = 0; k < R; ++k) pk::load3(f, P, static_cast<long long>(s[k]), v[k]);
}

// Lagrangian lattice indices of the particle ids.
template <int R>
__device__ __forceinline__ void lattice_all(const unsigned (&id)[R], int lp, int (&idx)[R][3]) {
#pragma unroll
  for (int k = 0; k < R; ++k) pk::lattice(static_cast<long long>(id[k]), lp, idx[k]);
}

// Where the particles of one order go in the next, as a counting kernel over
// that order's items left it: packed neighbour slots and ranks, the keys of
// the far ones, the items' rows of first ranks, and the next order's block
// starts.
struct Moves {
  const unsigned* key;
  const unsigned* rank;
  const unsigned* nbr_base;
  const unsigned* start;
};

// Slots in the next order of the particles of item m: f(a, ok, id, s) with
// their slots a in this order, their ids and their slots s in the next; Ld is
// the next order's layout, rs = log2 of this grid's side over that one's;
// first: kNbr words of LDS.
template <class F>
__device__ __forceinline__ void for_moves(const Item& m, const unsigned* __restrict__ ids,
                                          const Moves& mv, const Layout& Ld, int rs,
                                          unsigned* first, F&& f) {
  const unsigned b0 = block_around(m, Ld, rs);
  if (threadIdx.x < kNbr)
    first[threadIdx.x] = mv.start[neighbour_key(b0, static_cast<int>(threadIdx.x), Ld)] +
                         mv.nbr_base[static_cast<size_t>(m.i) * kNbrRow + threadIdx.x];
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    long long a[R];
    bool ok[R];
    unsigned w[R], id[R];
    item_slots(m, a, ok);
    load_u32<R>(mv.rank, a, w);
    load_u32<R>(ids, a, id);
    __syncthreads();
    unsigned s[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const unsigned slot = w[k] >> kRankBits;
      s[k] = (slot < kNbr ? first[slot] : mv.start[mv.key[a[k]]]) + (w[k] & ((1u << kRankBits) - 1));
    }
    f(a, ok, id, s);
  });
}

// Moves nf fields (and the ids) of the order's particles to the next order's
// slots; dest[a] receives the slot of slot a.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scatter_b(Items it, Layout L, Layout Ld, int rs,
                                                        Moves mv, Ptrs<T> src, MPtrs<T> dst,
                                                        int nf, unsigned* __restrict__ ids_dst,
                                                        unsigned* __restrict__ dest) {
  __shared__ unsigned first[kNbr];
  Item m;
  if (!item_of<true>(it, L, m)) return;
  for_moves(m, it.ids, mv, Ld, rs, first, [&](const auto& a, const auto& ok, const auto& id,
                                              const auto& s) {
    constexpr int R = sizeof(s) / sizeof(s[0]);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (!ok[k]) continue;
      for (int f = 0; f < nf; ++f) dst.p[f][s[k]] = src.p[f][a[k]];
      ids_dst[s[k]] = id[k];
      dest[a[k]] = s[k];
    }
  });
}

template <typename T>
__device__ __forceinline__ Stencil<T> wrapped_stencil(const int idx[3], const T dsp[3],
                                                      const Grid<T>& g) {
  Stencil<T> s = pk::stencil(idx, g.ratio, dsp, g.inv_cell, g.cell);
  const int mask = (1 << g.lm) - 1;
#pragma unroll
  for (int a = 0; a < 3; ++a) s.i0[a] &= mask;
  return s;
}

// One cell of a gather window: its fields side by side, so a corner of a
// stencil is one 16-byte LDS read (two in FP64) instead of one read per field
// (force adjoint 344 -> 341 us at 256^3 in FP32; the others unchanged).
template <typename T>
struct alignas(4 * sizeof(T)) WinCell {
  T v[4];
};

// Loads the NF window fields (mesh fields src.p[f]) into lds[k].v[f].
template <int NF, typename T>
__device__ __forceinline__ void load_window(const int o[3], const Layout& L, const Ptrs<T>& src,
                                            WinCell<T>* lds) {
  constexpr int kIt = (kWin + kThreads - 1) / kThreads;
  WinCell<T> v[kIt];
#pragma unroll
  for (int j = 0; j < kIt; ++j) {
    const int k = min(static_cast<int>(threadIdx.x) + j * kThreads, kWin - 1);
    const unsigned c = win_cell(o, k, L);
#pragma unroll
    for (int f = 0; f < 4; ++f) v[j].v[f] = f < NF ? src.p[f][c] : T(0);
  }
#pragma unroll
  for (int j = 0; j < kIt; ++j) {
    const int k = static_cast<int>(threadIdx.x) + j * kThreads;
    if (k < kWin) lds[k] = v[j];
  }
}

// LDS accumulation of the paint windows.  FP64 grids: FP64 adds
// (ds_add_f64).  FP32 grids: 64-bit fixed point, value = integer x 2^-e
// (ds_add_u64 takes about half the time of ds_add_f64 on scattered cells
// of gfx950, and integer adds are exact, so the window sums do not depend
// on the order of the atomics).  e is chosen per work item so that nothing
// overflows (fx::scale_for; a window cell receives at most kChunk
// contributions).  The rounding of a contribution, at most 2^-52 amax, is far
// below the FP32 result's.
//
// A contribution w x becomes its integer with one fused multiply-add (fx::rounded):
// x 2^e is taken once per particle (exact).  gfx950 has no conversion
// from FP64 to 64-bit integers; the emulated one (a dozen FP64 and integer
// instructions) for 24 contributions per particle cost the cotangent paint
// 10 of 257 us at 256^3.
template <typename T>
struct WinAcc {
  using Cell = double;
  struct Scale {
    double s, inv;
  };
  __device__ static Scale scale_for(double) { return Scale{1.0, 1.0}; }
  // whether the particle contributes (one without a position makes its cells NaN)
  __device__ static bool takes(const Stencil<T>&) { return true; }
  // x ready for add: the contribution w x is added to the cell
  __device__ static double scaled(double x, const Scale&) { return x; }
  __device__ static void add(Cell* c, double w, double x) { atomicAdd(c, w * x); }
  __device__ static double get(Cell c, const Scale&) { return c; }
};
struct FixAcc {
  using Cell = unsigned long long;
  using Scale = fx::Scale;
  __device__ static Scale scale_for(double amax) { return fx::scale_for(amax); }
  // Whether the particle has a position.  The weights of one at NaN or infinity
  // are NaN, which has no integer: it adds nothing.
  template <typename T>
  __host__ __device__ static bool takes(const Stencil<T>& s) {
    const T t = s.t[0] + s.t[1] + s.t[2];
    return t == t;
  }
  // The scale of a deterministic paint, one for the whole paint: amax 2^e
  // 2^lpc < 2^62, so that a cell may receive one contribution from each of
  // the 2^lpc particles (a particle adds to a cell at most once) without
  // overflow; the rounding of a contribution is at most 2^(lpc - 62) amax.
  __device__ static Scale scale_det(double amax, int lpc) {
    if (!(amax > 0.0)) return Scale{1.0, 1.0};
    int k;
    frexp(amax, &k);
    return Scale{ldexp(1.0, 62 - lpc - k), ldexp(1.0, k + lpc - 62)};
  }
  // (a value that is not finite adds nothing either)
  __host__ __device__ static double scaled(double x, const Scale& sc) {
    return fabs(x) < HUGE_VAL ? x * sc.s : 0.0;
  }
  __device__ static void add(Cell* c, double w, double x) {
    atomicAdd(c, static_cast<unsigned long long>(fx::rounded(w, x)));
  }
  __device__ static double get(Cell c, const Scale& sc) {
    return static_cast<double>(static_cast<long long>(c)) * sc.inv;
  }
};
template <>
struct WinAcc<float> : FixAcc {};
// Deterministic paints: scale_det lets contributions grow past 2^52 on the
// smallest grid (8^3 particles), so they convert with the general rounding.
struct DetAcc : FixAcc {
  __device__ static void add(Cell* c, double w, double x) {
    atomicAdd(c, static_cast<unsigned long long>(__double2ll_rn(w * x)));
  }
};

// Window accumulator of a paint: WinAcc<T>, or fixed point in deterministic
// mode (DET) for both precisions.
template <typename T, bool DET>
using PaintAcc = typename std::conditional<DET, DetAcc, WinAcc<T>>::type;

// Largest |contribution| a deterministic paint's scale is chosen for: the
// CIC weights (at most 1) times coef times the largest |v| (vmax, device;
// null for a density paint).  Computed the same way by the paint and by
// k_det_to_field.
template <typename T>
__device__ __forceinline__ double det_amax(const double* vmax, T coef) {
  return vmax ? fabs(static_cast<double>(coef * static_cast<T>(*vmax))) : 1.0;
}

template <typename C>
__device__ __forceinline__ void zero_window(C* acc, int nf) {
  for (int k = threadIdx.x; k < nf * kWin; k += kThreads) acc[k] = C(0);
}

// Largest |x| over the workgroup's threads (red: kThreads / 64 doubles of
// LDS; every thread gets the result after the barrier the caller places
// between the two halves).
__device__ __forceinline__ void wg_max_issue(double x, double* red) {
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
}
__device__ __forceinline__ double wg_max_finish(const double* red) {
  double x = red[0];
  for (int w = 1; w < kThreads / 64; ++w) x = fmax(x, red[w]);
  return x;
}

// Flush of nf windows, value(f, k) being cell k of window f: the block's own 8^3
// cells into the fields dst, the 217 cells with a coordinate 8 into the halos hl
// (HaloMap, one after the other).  When this item is the block's only one (no
// other item of the launch writes its cells and entries) it stores them; else it
// adds the non-zero ones atomically to what zero_unowned cleared.
template <typename V, class Value, class Add>
__device__ __forceinline__ void flush(const Item& m, const Layout& L, int nf,
                                      const MPtrs<V>& dst, V* __restrict__ hl, Value&& value,
                                      Add&& add) {
  constexpr int kIt = (kWin + kThreads - 1) / kThreads;
  const HaloMap hm(L.lm);
  const unsigned bx = static_cast<unsigned>(m.o[0]) >> kLB,
                 by = static_cast<unsigned>(m.o[1]) >> kLB,
                 bz = static_cast<unsigned>(m.o[2]) >> kLB;
#pragma unroll
  for (int j = 0; j < kIt; ++j) {
    const int k = static_cast<int>(threadIdx.x) + j * kThreads;
    if (k >= kWin) continue;
    const unsigned kx = k / (kW * kW), r = k - kx * kW * kW;
    const unsigned ky = r / kW, kz = r - ky * kW;
    const bool own = kx < kB && ky < kB && kz < kB;
    const unsigned c = own ? win_cell(m.o, k, L) : hm.of_window(bx, by, bz, kx, ky, kz);
    for (int f = 0; f < nf; ++f) {
      V* out = (own ? dst.p[f] : hl + static_cast<size_t>(f) * hm.size()) + c;
      const V v = value(f, k);
      if (m.single)
        *out = v;
      else if (v != V(0))
        add(out, v);
    }
  }
}

template <typename T>
__device__ __forceinline__ void flush_owned(const Item& m, const Layout& L,
                                            const typename WinAcc<T>::Cell* acc,
                                            const typename WinAcc<T>::Scale& sc, int nf,
                                            const MPtrs<T>& dst, T* __restrict__ hl) {
  flush(m, L, nf, dst, hl,
        [&](int f, int k) { return static_cast<T>(WinAcc<T>::get(acc[f * kWin + k], sc)); },
        [](T* p, T v) { pk::atomic_add(p, v); });
}

// Before a paint of one order: zeroes the own cells (nf fields) and the
// halo entries of every block that no single work item owns, i.e. blocks
// with no particles or with several items (whose items add atomically); a
// block's only item stores all of them itself.  One wavefront per block:
// lane (i, j) clears the eight cells of its z row and its entries of the faces.
// istart: the order's item starts per block (nb + 1).
template <typename V>
__device__ __forceinline__ void zero_unowned(long long wg, const unsigned* __restrict__ istart,
                                             const Layout& L, int nf, const MPtrs<V>& dst,
                                             V* __restrict__ hl) {
  const long long t = wg * kThreads + threadIdx.x;
  const long long b = t >> 6;
  if (b >= (1ll << (3 * L.lnb))) return;
  if (istart[b + 1] - istart[b] == 1u) return;
  const unsigned lane = static_cast<unsigned>(t & 63), i = lane >> 3, j = lane & 7;
  int o[3];
  block_origin(static_cast<unsigned>(b), L, o);
  const unsigned ox = static_cast<unsigned>(o[0]), oy = static_cast<unsigned>(o[1]),
                 oz = static_cast<unsigned>(o[2]);
  const unsigned row = cell_at(ox + i, oy + j, oz, L);
  const HaloMap hm(L.lm);
  const unsigned bx = ox >> kLB, by = oy >> kLB, bz = oz >> kLB;
  for (int f = 0; f < nf; ++f) {
#pragma unroll
    for (int z = 0; z < kB; ++z) dst.p[f][row + z] = V(0);
    V* h = hl + static_cast<size_t>(f) * hm.size();
    h[hm.of_window(bx, by, bz, i, j, kB)] = V(0);
    h[hm.of_window(bx, by, bz, i, kB, j)] = V(0);
    h[hm.of_window(bx, by, bz, kB, i, j)] = V(0);
    if (i == 0) {
      h[hm.of_window(bx, by, bz, j, kB, kB)] = V(0);
      h[hm.of_window(bx, by, bz, kB, j, kB)] = V(0);
      h[hm.of_window(bx, by, bz, kB, kB, j)] = V(0);
      if (j == 0) h[hm.of_window(bx, by, bz, kB, kB, kB)] = V(0);
    }
  }
}
template <typename V>
__global__ __launch_bounds__(kThreads) void k_zero_unowned(const unsigned* __restrict__ istart,
                                                           Layout L, int nf, MPtrs<V> dst,
                                                           V* __restrict__ hl) {
  zero_unowned(blockIdx.x, istart, L, nf, dst, hl);
}
inline unsigned zero_grid(const Layout& L) {
  return static_cast<unsigned>(((1ll << (3 * L.lnb)) * 64 + kThreads - 1) / kThreads);
}

// What a density paint of the new order needs zeroed, done by extra workgroups of
// the kernel that moves the ids there (wg0: the first of them).
template <typename T>
struct ZeroFirst {
  unsigned wg0;
  const unsigned* istart;
  T* rho;
  T* hl;
};

// The ids of the lattice order's slots q = tile_site(a) to slots
// s = start[key[a]] + rank[a] of the new order, dest[q] = s.  The new order's map
// back, through which the next kernels read the state left in the lattice order,
// is its ids.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scatter_ids(
    const unsigned* __restrict__ key, const unsigned* __restrict__ rank,
    const unsigned* __restrict__ start, unsigned* __restrict__ ids_dst,
    unsigned* __restrict__ dest, long long P, int lp, Layout L, ZeroFirst<T> zf) {
  if (blockIdx.x >= zf.wg0) {
    zero_unowned(blockIdx.x - zf.wg0, zf.istart, L, 1, MPtrs<T>{{zf.rho}}, zf.hl);
    return;
  }
  const long long a = blockIdx.x * (long long)kThreads + threadIdx.x;
  if (a >= P) return;
  const long long q = tile_site(a, lp);
  const unsigned s = start[key[a]] + rank[a];
  ids_dst[s] = static_cast<unsigned>(q);
  dest[q] = s;
}

// The ids alone to the next order's slots, dest[a] = the slot of slot a, and
// inv[s] = a: the new order's map back to this one, through which the next
// kernels read the state left in this order.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scatter_ids_b(
    Items it, Layout L, Layout Ld, int rs, Moves mv, unsigned* __restrict__ ids_dst,
    unsigned* __restrict__ dest, unsigned* __restrict__ inv, ZeroFirst<T> zf) {
  if (blockIdx.x >= zf.wg0) {
    zero_unowned(blockIdx.x - zf.wg0, zf.istart, Ld, 1, MPtrs<T>{{zf.rho}}, zf.hl);
    return;
  }
  __shared__ unsigned first[kNbr];
  Item m;
  if (!item_of<true>(it, L, m)) return;
  for_moves(m, it.ids, mv, Ld, rs, first, [&](const auto& a, const auto& ok, const auto& id,
                                              const auto& s) {
    constexpr int R = sizeof(s) / sizeof(s[0]);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (!ok[k]) continue;
      ids_dst[s[k]] = id[k];
      inv[s[k]] = static_cast<unsigned>(a[k]);
      dest[a[k]] = s[k];
    }
  });
}

// Output of a paint in deterministic mode: the integer fields det (nf fields
// of ncells) and their halos hl, the device maximum |v| the scale is chosen for
// (null for a density paint) and lpc = log2 of the particle count.
struct DetOut {
  unsigned long long* det;
  unsigned long long* hl;
  const double* vmax;
  long long ncells;
  int lpc;
};

// Flush of a deterministic paint: the windows' integer sums themselves (one scale
// for the whole paint), with 64-bit integer atomics where a block has several
// items.  Integer adds commute, so the result depends neither on the order of the
// atomics nor on which particles share an item.
__device__ __forceinline__ void flush_det(const Item& m, const Layout& L, const FixAcc::Cell* acc,
                                          int nf, const DetOut& dt) {
  using V = unsigned long long;
  flush(m, L, nf, MPtrs<V>{{dt.det, dt.det + dt.ncells, dt.det + 2 * dt.ncells}}, dt.hl,
        [&](int f, int k) { return static_cast<V>(acc[f * kWin + k]); },
        [](V* p, V v) { atomicAdd(p, v); });
}

// Coordinates of cell i of a field.
__device__ __forceinline__ void cell_of(unsigned i, const Layout& L, unsigned c[3]) {
  const unsigned m = (1u << L.lm) - 1;
  if (L.slabs) {
    c[2] = i >> (2 * L.lm + kLB) << kLB | (i & (kB - 1));
    c[1] = i >> kLB & m;
    c[0] = i >> (L.lm + kLB) & m;
  } else {
    c[2] = i & m;
    c[1] = i >> L.lm & m;
    c[0] = i >> (2 * L.lm);
  }
}

// The fields of a deterministic paint: out_f[i] = (det_f[i] + what the halo holds
// for cell i) 2^-e with the paint's scale (vmax, coef, lpc as given to the paint).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_det_to_field(const unsigned long long* __restrict__ det,
                                                           const unsigned long long* __restrict__ hl,
                                                           int nf, long long ncells, Layout L,
                                                           const double* __restrict__ vmax,
                                                           T coef, int lpc, MPtrs<T> out) {
  const double inv = FixAcc::scale_det(det_amax<T>(vmax, coef), lpc).inv;
  const HaloMap hm(L.lm);
  for (long long i = blockIdx.x * (long long)kThreads + threadIdx.x; i < ncells;
       i += (long long)gridDim.x * kThreads) {
    unsigned c[3];
    cell_of(static_cast<unsigned>(i), L, c);
    for (int f = 0; f < nf; ++f) {
      const unsigned long long v =
          det[f * ncells + i] + hm.sum(hl + static_cast<size_t>(f) * hm.size(), c[0], c[1], c[2]);
      out.p[f][i] = static_cast<T>(static_cast<double>(static_cast<long long>(v)) * inv);
    }
  }
}

// The x part of the halos into the planes x = 0 mod 8 of the fields in slabs, one per
// blockIdx.y (fft_halo_x_apart).  Thread i: cell i of the fields' planes in turn.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_add_halo_x(MPtrs<T> dst, const T* __restrict__ hl,
                                                         Layout L) {
  const unsigned i = blockIdx.x * kThreads + threadIdx.x;
  if (i >> (3 * L.lm - kLB)) return;
  const HaloMap hm(L.lm);
  // i = [x / 8][z / 8][y][z mod 8]
  const unsigned m = (1u << L.lm) - 1;
  const unsigned z = (i >> (L.lm + kLB) & ((1u << L.lnb) - 1)) << kLB | (i & (kB - 1));
  const unsigned y = i >> kLB & m, x = i >> (2 * L.lm) << kLB;
  T* p = dst.p[blockIdx.y] + cell_at(x, y, z, L);
  const T v = *p;
  *p = v + hm.sum_x(hl + static_cast<size_t>(blockIdx.y) * hm.size(), x, y, z);
}

// rho += its halo, for one field of side 2^lm (the data grid, and the callers that
// want the painted field itself).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_add_halo(T* __restrict__ rho,
                                                       const T* __restrict__ hl, Layout L,
                                                       long long ncells) {
  const long long i = blockIdx.x * (long long)kThreads + threadIdx.x;
  if (i >= ncells) return;
  unsigned c[3];
  cell_of(static_cast<unsigned>(i), L, c);
  if (((c[0] & 7u) == 0) | ((c[1] & 7u) == 0) | ((c[2] & 7u) == 0))
    rho[i] += HaloMap(L.lm).sum(hl, c[0], c[1], c[2]);
}

// rho(c) += sum_n W(q_n + d_n - c) over the items of one order.  The
// displacement of slot a is d[a], or d[gsrc[a]] when it was left in the
// previous order (gsrc: this order's slots to that order's); then dcopy
// receives it in this order.  DET: the deterministic mode's output (dt)
// instead of rho and hl.
template <typename T, bool DET>
__global__ __launch_bounds__(kThreads) void k_paint_b(const T* __restrict__ d,
                                                      const unsigned* __restrict__ gsrc,
                                                      T* __restrict__ dcopy, long long P,
                                                      int lp, Grid<T> g, Layout L, Items it,
                                                      T* __restrict__ rho, T* __restrict__ hl,
                                                      DetOut dt) {
  using A = PaintAcc<T, DET>;
  __shared__ typename A::Cell acc[kWin];
  Item m;
  if (!item_of<false>(it, L, m)) return;
  typename A::Scale sc{};
  long long a[kPer];
  bool ok[kPer];
  unsigned id[kPer];
  int idx[kPer][3];
  T dsp[kPer][3];
  item_slots(m, a, ok);  // loads in flight while the window is cleared
  // all rounds at once: by rounds, whose loads through gsrc start later, this kernel
  // measured 158 us instead of 148 when it was split off, 164 instead of 168 with
  // the present flush (FP32, 256^3)
  load_u32<kPer>(it.ids, a, id);
  if (gsrc) {
    unsigned sa[kPer];
    load_u32<kPer>(gsrc, a, sa);
    load3_at<kPer>(d, P, sa, dsp);
  } else {
    load3_at<kPer>(d, P, a, dsp);
  }
  zero_window(acc, 1);
  if (dcopy) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (!ok[k]) continue;
      dcopy[a[k]] = dsp[k][0];
      dcopy[P + a[k]] = dsp[k][1];
      dcopy[2 * P + a[k]] = dsp[k][2];
    }
  }
  lattice_all(id, lp, idx);
  if constexpr (DET)
    sc = FixAcc::scale_det(1.0, dt.lpc);
  else
    sc = A::scale_for(1.0);
  const double one = A::scaled(1.0, sc);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (!ok[k]) continue;
    const Stencil<T> s = wrapped_stencil(idx[k], dsp[k], g);
    if (!A::takes(s)) continue;
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T w, T, T, T) {
      A::add(&acc[win_index(m.o, cx, cy, cz)], static_cast<double>(w), one);
    });
  }
  __syncthreads();
  if constexpr (DET)
    flush_det(m, L, acc, 1, dt);
  else
    flush_owned<T>(m, L, acc, sc, 1, MPtrs<T>{{rho}}, hl);
}

// g_bar_j(c) += coef * sum_n v_nj W(q_n + d_n - c), three meshes M apart; v
// of slot a is read at slot src[a] (the order the cotangents were left in).
// DET: the deterministic mode's output (dt, with dt.vmax = max |v|) instead
// of out and hl.
template <typename T, bool DET>
__global__ __launch_bounds__(kThreads) void k_paint_vec_b(const T* __restrict__ d,
                                                          const T* __restrict__ v, T coef,
                                                          long long P, int lp, Grid<T> g,
                                                          Layout L, Items it, T* __restrict__ out,
                                                          long long M,
                                                          const unsigned* __restrict__ src,
                                                          T* __restrict__ hl, DetOut dt) {
  using A = PaintAcc<T, DET>;
  __shared__ typename A::Cell acc[3 * kWin];
  __shared__ double red[kThreads / 64];
  Item m;
  if (!item_of<false>(it, L, m)) return;
  typename A::Scale sc{};
  long long a[kPer];
  bool ok[kPer];
  unsigned id[kPer], sa[kPer];
  int idx[kPer][3];
  T dsp[kPer][3], vv[kPer][3];
  item_slots(m, a, ok);  // loads in flight while the window is cleared
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    load_u32<R>(src, a, sa);
    load3_at<R>(d, P, a, dsp);
    load3_at<R>(v, P, sa, vv);
  });
  zero_window(acc, 3);
  lattice_all(id, lp, idx);
  double amax = 0.0;  // largest |coef v| of the item (the weights are at most 1)
  if constexpr (!DET) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (!ok[k]) continue;
#pragma unroll
      for (int q = 0; q < 3; ++q) amax = fmax(amax, fabs(static_cast<double>(coef * vv[k][q])));
    }
  }
  wg_max_issue(amax, red);
  __syncthreads();
  if constexpr (DET)
    sc = FixAcc::scale_det(det_amax<T>(dt.vmax, coef), dt.lpc);
  else
    sc = A::scale_for(wg_max_finish(red));
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (!ok[k]) continue;
    const double v0 = A::scaled(static_cast<double>(coef * vv[k][0]), sc),
                 v1 = A::scaled(static_cast<double>(coef * vv[k][1]), sc),
                 v2 = A::scaled(static_cast<double>(coef * vv[k][2]), sc);
    const Stencil<T> s = wrapped_stencil(idx[k], dsp[k], g);
    if (!A::takes(s)) continue;
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T w, T, T, T) {
      const int c = win_index(m.o, cx, cy, cz);
      const double wd = static_cast<double>(w);
      A::add(&acc[c], wd, v0);
      A::add(&acc[kWin + c], wd, v1);
      A::add(&acc[2 * kWin + c], wd, v2);
    });
  }
  __syncthreads();
  if constexpr (DET)
    flush_det(m, L, acc, 3, dt);
  else
    flush_owned<T>(m, L, acc, sc, 3, MPtrs<T>{{out, out + M, out + 2 * M}}, hl);
}

// Readout of g at d_n, kick p += kick F, drift d' = d_n + drift p; the new
// state goes to (dn, pn) in this order with its block key and rank on grid L
// (no keys when count is null: a replay into an order already recorded).
// The momentum of slot a is p[a], or p[pinv[a]] when the momenta were left
// in the previous order (pinv: this order's slots to that order's).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_step_b(
    const T* __restrict__ d, const T* __restrict__ p, const unsigned* __restrict__ pinv,
    const T* __restrict__ g, long long M, T kick, T drift, long long P, int lp, Grid<T> gr,
    Layout L, Items it, T* __restrict__ dn, T* __restrict__ pn, unsigned* __restrict__ count,
    unsigned* __restrict__ key, unsigned* __restrict__ rank,
    unsigned* __restrict__ nbr_base) {
  __shared__ WinCell<T> lds[kWin];
  __shared__ unsigned wcnt[kNbr];
  Item m;
  if (!item_of<true>(it, L, m)) return;
  long long a[kPer];
  bool ok[kPer];
  unsigned b[kPer], id[kPer];
  int idx[kPer][3];
  T dsp[kPer][3], mom[kPer][3];
  item_slots(m, a, ok);  // particle loads in flight while the window loads
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    if (pinv) {
      unsigned sa[kPer];
      load_u32<R>(pinv, a, sa);
      load3_at<R>(d, P, a, dsp);
      load3_at<R>(p, P, sa, mom);
    } else {
      load3_at<R>(d, P, a, dsp);
      load3_at<R>(p, P, a, mom);
    }
  });
  load_window<3>(m.o, L, Ptrs<T>{{g, g + M, g + 2 * M}}, lds);
  if (threadIdx.x < kNbr) wcnt[threadIdx.x] = 0;
  lattice_all(id, lp, idx);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    b[k] = 0;
    if (!ok[k]) continue;
    T F[3] = {0, 0, 0};
    const Stencil<T> s = wrapped_stencil(idx[k], dsp[k], gr);
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T w, T, T, T) {
      const WinCell<T> q = lds[win_index(m.o, cx, cy, cz)];
      F[0] += w * q.v[0];
      F[1] += w * q.v[1];
      F[2] += w * q.v[2];
    });
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      mom[k][q] += kick * F[q];
      pn[q * P + a[k]] = mom[k][q];
      dsp[k][q] += drift * mom[k][q];
      dn[q * P + a[k]] = dsp[k][q];
    }
    Stencil<T> s2 = pk::stencil(idx[k], gr.ratio, dsp[k], gr.inv_cell, gr.cell);
    b[k] = block_of(s2, L);
  }
  if (!count) return;
  // ranks aggregated over the workgroup (see rank_issue_wg)
  RankTicket t[kPer];
  int slot[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    slot[k] = neighbour_slot(m.b, b[k], L);
    t[k] = rank_issue_wg(b[k], slot[k], ok[k], count, wcnt);
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const unsigned r = rank_of(t[k]);
    if (!ok[k]) continue;
    rank[a[k]] = static_cast<unsigned>(slot[k]) << kRankBits | r;
    if (slot[k] == kNbr) key[a[k]] = b[k];
  }
  __syncthreads();
  rank_reserve_wg(m.b, L, count, wcnt, nbr_base + static_cast<size_t>(m.i) * kNbrRow);
}

// Position cotangent of one force evaluation with cotangent v = coef p_bar:
// d_bar += sum_c grad W(x - c) [sum_j v_j g_j(c) + rho_bar(c)], then the
// drift adjoint p_bar += drift d_bar; g (three meshes) and rho_bar are read
// from one four-field window.  p_bar and d_bar of slot a are read at slot
// src[a] of the order they were left in (the next order, or the data order)
// and the updates go to pbar_out[a] and dbar_out[a] in this order, so the
// move between orders costs no pass of its own.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_force_adjoint_b(
    const T* __restrict__ d, const T* __restrict__ pbar, const T* __restrict__ dbar, T coef,
    const T* __restrict__ g, const T* __restrict__ rho_bar, long long M, T drift, long long P,
    int lp, Grid<T> gm, Layout L, Items it, const unsigned* __restrict__ src,
    T* __restrict__ dbar_out, T* __restrict__ pbar_out) {
  __shared__ WinCell<T> lds[kWin];
  Item m;
  if (!item_of<true>(it, L, m)) return;
  long long a[kPer];
  int idx[kPer][3];
  bool ok[kPer];
  unsigned id[kPer], sa[kPer];
  T dsp[kPer][3], pb[kPer][3], db[kPer][3];
  item_slots(m, a, ok);  // particle loads in flight while the window loads
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    load_u32<R>(src, a, sa);
    load3_at<R>(d, P, a, dsp);
    load3_at<R>(pbar, P, sa, pb);
    load3_at<R>(dbar, P, sa, db);
  });
  load_window<4>(m.o, L, Ptrs<T>{{g, g + M, g + 2 * M, rho_bar}}, lds);
  lattice_all(id, lp, idx);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (!ok[k]) continue;
    const Stencil<T> s = wrapped_stencil(idx[k], dsp[k], gm);
    const T v0 = coef * pb[k][0], v1 = coef * pb[k][1], v2 = coef * pb[k][2];
    T xb[3] = {0, 0, 0};
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T, T d0, T d1, T d2) {
      const WinCell<T> q = lds[win_index(m.o, cx, cy, cz)];
      const T h = v0 * q.v[0] + v1 * q.v[1] + v2 * q.v[2] + q.v[3];
      xb[0] += d0 * h;
      xb[1] += d1 * h;
      xb[2] += d2 * h;
    });
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      db[k][q] += xb[q] * gm.inv_cell;
      dbar_out[q * P + a[k]] = db[k][q];
      pbar_out[q * P + a[k]] = pb[k][q] + drift * db[k][q];
    }
  }

}

// Kick-synchronised snapshot of a state in its own block order (lightcone,
// section 2.2.1 item 3): snap = (d, p + half_kick F(d)), six fields P apart,
// F read out of the three force meshes g through the item's window.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_snapshot_b(
    const T* __restrict__ d, const T* __restrict__ p, const T* __restrict__ g, long long M,
    T half_kick, long long P, int lp, Grid<T> gm, Layout L, Items it, T* __restrict__ snap) {
  __shared__ WinCell<T> lds[kWin];
  Item m;
  if (!item_of<true>(it, L, m)) return;
  long long a[kPer];
  bool ok[kPer];
  unsigned id[kPer];
  int idx[kPer][3];
  T dsp[kPer][3], mom[kPer][3];
  item_slots(m, a, ok);  // particle loads in flight while the window loads
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    load3_at<R>(d, P, a, dsp);
    load3_at<R>(p, P, a, mom);
  });
  load_window<3>(m.o, L, Ptrs<T>{{g, g + M, g + 2 * M}}, lds);
  lattice_all(id, lp, idx);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (!ok[k]) continue;
    T F[3] = {0, 0, 0};
    const Stencil<T> s = wrapped_stencil(idx[k], dsp[k], gm);
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T w, T, T, T) {
      const WinCell<T> q = lds[win_index(m.o, cx, cy, cz)];
      F[0] += w * q.v[0];
      F[1] += w * q.v[1];
      F[2] += w * q.v[2];
    });
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      snap[q * P + a[k]] = dsp[k][q];
      snap[(3 + q) * P + a[k]] = mom[k][q] + half_kick * F[q];
    }
  }

}

// Last kick (readout of g at d) of the momenta p into pout in this order,
// then the key and rank of the redshift-space position on the data grid
// (layout Ld).  The momentum of slot a is p[a] (pout may then be p: each
// slot is read and written by one thread), or p[pinv[a]] when the momenta
// were left in the previous order (pout apart from p).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_final_b(
    const T* __restrict__ d, const T* p, const unsigned* __restrict__ pinv, T* pout,
    const T* __restrict__ g, long long M, T kick, long long P, int lp, Grid<T> gm, Layout L,
    Items it, pk::Rsd<T> rsd, Grid<T> gd, Layout Ld, unsigned* __restrict__ count,
    unsigned* __restrict__ key, unsigned* __restrict__ rank,
    unsigned* __restrict__ nbr_base) {
  __shared__ WinCell<T> lds[kWin];
  __shared__ unsigned wcnt[kNbr];
  Item m;
  if (!item_of<true>(it, L, m)) return;
  // ranks aggregated over the workgroup around the data-grid block that
  // holds this mesh block's origin (see rank_issue_wg)
  const unsigned b0 = block_around(m, Ld, L.lm - Ld.lm);
  long long a[kPer];
  bool ok[kPer];
  unsigned b[kPer], id[kPer];
  int idx[kPer][3];
  T dsp[kPer][3], mom[kPer][3];
  item_slots(m, a, ok);  // particle loads in flight while the window loads
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    if (pinv) {
      unsigned sa[kPer];
      load_u32<R>(pinv, a, sa);
      load3_at<R>(d, P, a, dsp);
      load3_at<R>(p, P, sa, mom);
    } else {
      load3_at<R>(d, P, a, dsp);
      load3_at<R>(p, P, a, mom);
    }
  });
  load_window<3>(m.o, L, Ptrs<T>{{g, g + M, g + 2 * M}}, lds);
  if (threadIdx.x < kNbr) wcnt[threadIdx.x] = 0;
  lattice_all(id, lp, idx);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    b[k] = 0;
    if (!ok[k]) continue;
    T F[3] = {0, 0, 0}, ds[3];
    const Stencil<T> s = wrapped_stencil(idx[k], dsp[k], gm);
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T w, T, T, T) {
      const WinCell<T> q = lds[win_index(m.o, cx, cy, cz)];
      F[0] += w * q.v[0];
      F[1] += w * q.v[1];
      F[2] += w * q.v[2];
    });
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      mom[k][q] += kick * F[q];
      pout[q * P + a[k]] = mom[k][q];
    }
    pk::rsd_shift(rsd, idx[k], dsp[k], mom[k], ds);
    Stencil<T> s2 = pk::stencil(idx[k], gd.ratio, ds, gd.inv_cell, gd.cell);
    b[k] = block_of(s2, Ld);
  }
  RankTicket t[kPer];
  int slot[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    slot[k] = neighbour_slot(b0, b[k], Ld);
    t[k] = rank_issue_wg(b[k], slot[k], ok[k], count, wcnt);
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const unsigned r = rank_of(t[k]);
    if (!ok[k]) continue;
    rank[a[k]] = static_cast<unsigned>(slot[k]) << kRankBits | r;
    if (slot[k] == kNbr) key[a[k]] = b[k];
  }
  __syncthreads();
  rank_reserve_wg(b0, Ld, count, wcnt, nbr_base + static_cast<size_t>(m.i) * kNbrRow);
}

// Data-grid paint of the redshift-space positions (items of the data order).
// DET: the deterministic mode's output (dt) instead of rho and hl.
template <typename T, bool DET>
__global__ __launch_bounds__(kThreads) void k_data_paint_b(const T* __restrict__ d,
                                                           const T* __restrict__ p, long long P,
                                                           int lp, pk::Rsd<T> rsd, Grid<T> gd,
                                                           Layout Ld, Items it,
                                                           T* __restrict__ rho,
                                                           T* __restrict__ hl, DetOut dt) {
  using A = PaintAcc<T, DET>;
  __shared__ typename A::Cell acc[kWin];
  Item m;
  if (!item_of<false>(it, Ld, m)) return;
  typename A::Scale sc{};
  long long a[kPer];
  bool ok[kPer];
  unsigned id[kPer];
  int idx[kPer][3];
  T dsp[kPer][3], mom[kPer][3];
  item_slots(m, a, ok);  // loads in flight while the window is cleared
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    load3_at<R>(d, P, a, dsp);
    load3_at<R>(p, P, a, mom);
  });
  zero_window(acc, 1);
  lattice_all(id, lp, idx);
  if constexpr (DET)
    sc = FixAcc::scale_det(1.0, dt.lpc);
  else
    sc = A::scale_for(1.0);
  const double one = A::scaled(1.0, sc);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (!ok[k]) continue;
    T ds[3];
    pk::rsd_shift(rsd, idx[k], dsp[k], mom[k], ds);
    const Stencil<T> s = wrapped_stencil(idx[k], ds, gd);
    if (!A::takes(s)) continue;
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T w, T, T, T) {
      A::add(&acc[win_index(m.o, cx, cy, cz)], static_cast<double>(w), one);
    });
  }
  __syncthreads();
  if constexpr (DET)
    flush_det(m, Ld, acc, 1, dt);
  else
    flush_owned<T>(m, Ld, acc, sc, 1, MPtrs<T>{{rho}}, hl);
}

// Adjoint of the redshift-space distortion and the data paint over the data
// order: d_bar, p_bar in that order.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_data_adjoint_b(
    const T* __restrict__ d, const T* __restrict__ p, long long P, int lp, pk::Rsd<T> rsd,
    Grid<T> gd, Layout Ld, Items it, const T* __restrict__ rho_bar, T* __restrict__ dbar,
    T* __restrict__ pbar) {
  __shared__ T lds[kWin];
  Item m;
  if (!item_of<true>(it, Ld, m)) return;
  long long a[kPer];
  bool ok[kPer];
  unsigned id[kPer];
  int idx[kPer][3];
  T dsp[kPer][3], mom[kPer][3];
  item_slots(m, a, ok);  // particle loads in flight while the window loads
  with_rounds(m, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    load_u32<R>(it.ids, a, id);
    load3_at<R>(d, P, a, dsp);
    load3_at<R>(p, P, a, mom);
  });
  {
    constexpr int kIt = (kWin + kThreads - 1) / kThreads;
    T v[kIt];
#pragma unroll
    for (int j = 0; j < kIt; ++j)
      v[j] = rho_bar[win_cell(m.o, min(static_cast<int>(threadIdx.x) + j * kThreads, kWin - 1), Ld)];
#pragma unroll
    for (int j = 0; j < kIt; ++j) {
      const int k = static_cast<int>(threadIdx.x) + j * kThreads;
      if (k < kWin) lds[k] = v[j];
    }
  }
  lattice_all(id, lp, idx);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (!ok[k]) continue;
    T ds[3];
    pk::rsd_shift(rsd, idx[k], dsp[k], mom[k], ds);
    const Stencil<T> s = wrapped_stencil(idx[k], ds, gd);
    T xb[3] = {0, 0, 0};
    pk::for_corners_xyz(s, [&](int cx, int cy, int cz, T, T d0, T d1, T d2) {
      const T r = lds[win_index(m.o, cx, cy, cz)];
      xb[0] += d0 * r;
      xb[1] += d1 * r;
      xb[2] += d2 * r;
    });
#pragma unroll
    for (int q = 0; q < 3; ++q) xb[q] *= gd.inv_cell;
    T db[3] = {xb[0], xb[1], xb[2]}, pb[3] = {0, 0, 0};
    pk::rsd_transpose(rsd, idx[k], dsp[k], mom[k], xb, db, pb);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      dbar[q * P + a[k]] = db[q];
      pbar[q * P + a[k]] = pb[q];
    }
  }

}

}  // namespace bk
}  // namespace ic
