// sort.hpp -- counting sort of the particle slots by cell (c = i1 * n_th + i2).
//
// Not part of the paper's method: a layout device that keeps particles of one
// cell adjacent in memory, so that a wavefront streams contiguous SoA data,
// gathers from a few neighbouring field entries, and a deposit block's cells
// lie in the shared-memory tile around its middle one.  Empty and leaving slots get
// the key n_cells: they take no counter and no rank and are not moved; the
// destination's slots after the live particles get tag 0.
#pragma once

#include "particles.hpp"

namespace grpic {

constexpr int kScanBlock = 1024;  // elements scanned per block (4 per thread)

template <class T>
__device__ inline int sort_key(const Grid& g, const ParticleArraysT<T>& P, int64_t k) {
  const uint8_t t = P.tag[k];
  if (!is_live(t) || (t & kLeaving)) return g.n_r * g.n_th;
  return cell_key(g, t, P.i1[k], P.i2[k]);
}

// The rank pass takes kRankBlock consecutive slots per block of 256 threads
// (8 per thread) and counts them in a RankTable of kRankTable cells.
constexpr int kRankBits = 12;
constexpr int kRankBlock = 2048, kRankTable = 1 << kRankBits;
static_assert(kRankTable >= 2 * kRankBlock, "rank table too small for a block");

// Counts the live slots of each cell and gives every live slot its rank among
// the slots of its cell (block counting in an LDS hash table, one claim per
// cell and block: RankTable).  Ten steps after a sort, neighbouring slots
// mostly hold particles of different (nearby) cells, so runs of equal cells
// are short (about 2 slots at 16 particles per cell), while a block's slots
// fall in a few hundred distinct cells (measured: 262 of 2048 on a 4096^2
// grid at 16 particles per cell, 83 on 2048^2 at 90).  The rank is written to
// the source's i1p (the previous position is scratch between a push and its
// deposit, and the sort does not carry it), so the scatter needs no atomics.
// The fused push + deposit pass can do the same per block of its own
// (rank_fused), which makes this pass unnecessary.
template <class T>
__global__ void __launch_bounds__(256) sort_rank_kernel(Grid g, ParticleArraysT<T> P, int* __restrict__ counts) {
  RankTable<kRankBits>& rt = block_rank_table<kRankBits>();
  const int ncell = g.n_r * g.n_th;
  const int64_t k0 = (int64_t)blockIdx.x * kRankBlock;
  const int t = threadIdx.x;
  rank_clear(rt);
  __syncthreads();
  constexpr int kQ = kRankBlock / 256;
  int entry[kQ], local[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int64_t k = k0 + q * 256 + t;  // consecutive threads on consecutive slots
    const int key = k < P.n ? sort_key(g, P, k) : ncell;
    entry[q] = key < ncell ? rank_insert(rt, key, local[q]) : -1;
  }
  __syncthreads();
  rank_claim<kRankBits, 256>(rt, counts);
#pragma unroll
  for (int q = 0; q < kQ; ++q)
    if (entry[q] >= 0) P.i1p[k0 + q * 256 + t] = rt.n[entry[q]] + local[q];
}

// Exclusive scan of n ints in place, three phases: per-block scan (block sums
// out), scan of the block sums (one block), add the scanned block sums.
__device__ inline int block_exclusive_scan(int v, int* sh) {
  // Hillis-Steele over 256 threads in LDS
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const int add = t >= off ? sh[t - off] : 0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  const int incl = sh[t];
  __syncthreads();
  return incl - v;
}

__global__ void __launch_bounds__(256) scan_blocks_kernel(int* __restrict__ a, int64_t n,
                                                          int* __restrict__ sums) {
  __shared__ int sh[256];
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + 4 * threadIdx.x;
  int v[4];
  int tot = 0;
  for (int q = 0; q < 4; ++q) {
    v[q] = base + q < n ? a[base + q] : 0;
    tot += v[q];
  }
  const int ex = block_exclusive_scan(tot, sh);
  int run = ex;
  for (int q = 0; q < 4; ++q) {
    if (base + q < n) a[base + q] = run;
    run += v[q];
  }
  if (threadIdx.x == 255) sums[blockIdx.x] = ex + tot;
}

__global__ void __launch_bounds__(256) scan_sums_kernel(int* __restrict__ sums, int nb) {
  __shared__ int sh[256];
  // serial over chunks of 256 (nb is small: n / 1024)
  int carry = 0;
  for (int base = 0; base < nb; base += 256) {
    const int i = base + threadIdx.x;
    const int v = i < nb ? sums[i] : 0;
    const int ex = block_exclusive_scan(v, sh);
    if (i < nb) sums[i] = carry + ex;
    __syncthreads();
    if (threadIdx.x == 255) sh[0] = ex + v;
    __syncthreads();
    carry += sh[0];
    __syncthreads();
  }
}

__global__ void scan_add_kernel(int* __restrict__ a, int64_t n, const int* __restrict__ sums) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] += sums[i / kScanBlock];
}

// Source loads of the scatter: non-temporal in the single-precision form,
// which leaves the L2 to the destination lines that the wavefronts fill in
// pieces (measured at 4096^2, 16 particles per cell: -3 % for a sort after 10
// steps of motion, -18 % for a re-sort); plain in double precision, where the
// same loads gained nothing (4096^2 at 16 and 2048^2 at 90 particles per
// cell: the same or up to 5 % slower, against a spread of several per cent
// between single sorts).
template <class T, class V>
__device__ inline V scatter_load(const V* p) {
  if constexpr (sizeof(T) == 4) return __builtin_nontemporal_load(p);
  else return *p;
}

// Moves live slot k of S to slot off[key] + rank of D (rank from
// sort_rank_kernel, in S.i1p; off the exclusive scan of the cell counts).  No
// atomics: every load and store of a wavefront is independent.  Empty and leaving slots are not
// moved (sort_clear_tail_kernel empties the destination after the live
// slots).  The previous position (scratch between a push and its deposit) is
// not carried.
template <class T>
__global__ void __launch_bounds__(256) sort_scatter_kernel(Grid g, ParticleArraysT<T> S, ParticleArraysT<T> D,
                                                           const int* __restrict__ off) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= S.n) return;
  const uint8_t t = scatter_load<T>(S.tag + k);
  const int i1 = scatter_load<T>(S.i1 + k), i2 = scatter_load<T>(S.i2 + k);
  const int key = cell_key(g, t, i1, i2);
  if (key == g.n_r * g.n_th) return;
  const int64_t o = (int64_t)off[key] + scatter_load<T>(S.i1p + k);
  if (o < 0 || o >= D.n) return;  // ranks that do not belong to these counts (a caller's error)
  D.i1[o] = i1;
  D.i2[o] = i2;
  D.dx1[o] = scatter_load<T>(S.dx1 + k);
  D.dx2[o] = scatter_load<T>(S.dx2 + k);
  D.u1[o] = scatter_load<T>(S.u1 + k);
  D.u2[o] = scatter_load<T>(S.u2 + k);
  D.u3[o] = scatter_load<T>(S.u3 + k);
  D.w[o] = scatter_load<T>(S.w + k);
  D.phi[o] = scatter_load<T>(S.phi + k);
  D.tag[o] = t;
}

// The same scatter for many single-precision slots: each block of kScatBlock
// puts its particles in the order of their destinations in LDS first, so that
// a wavefront stores to a few runs of slots instead of one for every two lanes
// (what bounds the direct form: lines of the L2 that are filled in pieces,
// often from several XCDs).  The order is by bins of 8 destinations modulo
// 8 kScatBins, which the few rows that a block's particles go to share without
// mixing them finely; within a bin it is arbitrary.  Two LDS buffers take
// turns, one barrier per array.  Measured, a whole sort in single precision on
// (r, theta) grids whose particles moved by 0.2 to 2.5 cells, direct and this,
// ms: 512^2 16 per cell 0.219, 0.201; 1024^2 16 0.819, 0.754; 700^2 64 1.89,
// 1.38; 1024^2 64 3.90, 2.67; 1500 x 1100 24 2.37, 2.20; 2048^2 24 5.53, 4.48.
// Blocks of 2048 to 8192 slots gain more on some of these (1024^2 64: 2.45,
// 2.27) and lose on others (2048^2 8: direct 1.68, this 1.62, 8192 slots 1.99;
// 1500 x 1100 24: 2048 slots 2.55).
constexpr int kScatBlock = 1024, kScatBins = 1024;
static_assert(kScatBins == kScatBlock, "one thread per slot and per bin");

// Where a sort takes it: n^2 / cells >= 2^26.  The gain grows with the slots and
// with the slots per cell; whole sorts of sets ten steps old, us, direct and
// this: 2^20 slots 256^2 16 per cell 83, 86; 2^21 256^2 32 118, 106, 512^2 8 122, 133,
// 1024^2 2 152, 163; 2^22 512^2 16 207, 177, 1024^2 4 235, 250, 2048^2 1 308, 328;
// 2^23 512^2 32 361, 325, 1024^2 8 380, 369, 2048^2 2 493, 519; 2^24 1024^2 16 691, 628,
// 2048^2 4 806, 768; 2^26 2048^2 16 2751, 2372.  Sets in order already lose 3 %,
// and sets in no order 0 to 7 % at 2^22 (beyond that 0 to 60 % less).  In double
// precision, where twice the bytes pass LDS, it gains 15 % at 512^2 with 16 per
// cell and loses 20 % at 1400^2 with 24 (3.64, 4.37 ms): the direct form stays.
inline bool scatter_ordered(int64_t n, int64_t cells) { return (double)n * (double)n >= 0x1p26 * (double)cells; }

template <class V>
__device__ inline void scatter_array(V* sh, V v, int pos, bool store, uint32_t o, V* D) {
  if (pos >= 0) sh[pos] = v;
  lds_barrier();
  if (store) D[o] = sh[threadIdx.x];
}

__global__ void __launch_bounds__(kScatBlock)
sort_scatter_ordered_kernel(Grid g, ParticleArraysT<float> S, ParticleArraysT<float> D, const int* __restrict__ off) {
  __shared__ int bin[kScatBins];
  __shared__ int part[kScatBlock / 64];
  __shared__ float buf[2][kScatBlock];
  const int t = threadIdx.x;
  const ParticleArraysT<float> P = from_slot(S, (int64_t)blockIdx.x * kScatBlock);
  const bool in = t < P.n;
  const auto load = [&](const auto* a) {
    return in ? __builtin_nontemporal_load(a + t) : std::remove_cv_t<std::remove_reference_t<decltype(*a)>>(0);
  };
  bin[t] = 0;
  const uint8_t tag = load(P.tag);
  const int i1 = load(P.i1), i2 = load(P.i2), rank = load(P.i1p);
  const float dx1 = load(P.dx1);
  lds_barrier();
  const int key = cell_key(g, tag, i1, i2);
  const int64_t to = key == g.n_r * g.n_th ? -1 : (int64_t)off[key] + rank;
  const bool moves = to >= 0 && to < D.n;  // (as above)
  uint32_t o = moves ? (uint32_t)to : 0;
  const int mine = (int)(o >> 3) & (kScatBins - 1);
  int pos = moves ? atomicAdd(&bin[mine], 1) : -1;
  lds_barrier();
  // exclusive scan of the bins: within the wavefronts, then over them
  const int cnt = bin[t];
  int incl = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int up = __shfl_up(incl, d);
    if ((t & 63) >= d) incl += up;
  }
  if ((t & 63) == 63) part[t >> 6] = incl;
  lds_barrier();
  int base = incl - cnt, n = 0;
#pragma unroll
  for (int q = 0; q < kScatBlock / 64; ++q) {
    base += q < (t >> 6) ? part[q] : 0;
    n += part[q];
  }
  bin[t] = base;
  lds_barrier();
  if (moves) {
    pos += bin[mine];
    ((uint32_t*)buf[0])[pos] = o;
  }
  lds_barrier();
  const bool store = t < n;
  if (store) o = ((uint32_t*)buf[0])[t];
  // each array is loaded while the one before it is stored (all loads at the
  // start: 1500 x 1100 with 24 per cell 2.50 ms instead of 2.20)
  const float dx2 = load(P.dx2);
  scatter_array(buf[1], dx1, pos, store, o, D.dx1);
  const float u1 = load(P.u1);
  scatter_array(buf[0], dx2, pos, store, o, D.dx2);
  const float u2 = load(P.u2);
  scatter_array(buf[1], u1, pos, store, o, D.u1);
  const float u3 = load(P.u3);
  scatter_array(buf[0], u2, pos, store, o, D.u2);
  const float w = load(P.w);
  scatter_array(buf[1], u3, pos, store, o, D.u3);
  const float phi = load(P.phi);
  scatter_array(buf[0], w, pos, store, o, D.w);
  scatter_array(buf[1], phi, pos, store, o, D.phi);
  scatter_array((int*)buf[0], i1, pos, store, o, D.i1);
  scatter_array((int*)buf[1], i2, pos, store, o, D.i2);
  scatter_array((uint8_t*)buf[0], tag, pos, store, o, D.tag);
}

// Tag 0 on the destination slots from the live count (*live, the scan's
// total) to n: a grid-stride loop, so the launch can be small.
__global__ void __launch_bounds__(256) sort_clear_tail_kernel(uint8_t* __restrict__ tag, int64_t n,
                                                              const int* __restrict__ live) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = (int64_t)*live + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) tag[k] = 0;
}

}  // namespace grpic
