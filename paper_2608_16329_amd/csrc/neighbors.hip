// Cell-list neighbour builder for gfx950 (the binning step the paper takes
// from LAMMPS, Section 4.1; neighbour sets of Section 3.1).
//
// Atoms are binned into cells of edge >= cutoff + skin and counting-sorted by
// key = species * ncell + cell, so every (species, cell) bucket is a
// contiguous run of "sorted slots".  Rows are then found by scanning the
// 27 surrounding cells (deduplicated when a dimension has fewer than 3
// cells), species by species, which groups a row's entries by neighbour
// species.  The distance test is the exact one of the library's contract:
// wrapped coordinates, one minimum-image fold, (dx*dx + dy*dy) + dz*dz with
// round-to-nearest products and sums (no contraction), strict comparison.
#include <algorithm>

#include "kernel_math.h"
#include "mlip_internal.h"

namespace mlip {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanSeg = kScanThreads * kScanItems;

__device__ inline double wrap1(double x, double L) {
  double w = fmod(x, L);
  if (w < 0.0) w = w + L;
  if (w >= L) w = w - L;
  return w;
}

__device__ inline int cell_of(double w, double scale, int nc) {
  int c = int(w * scale);
  return c < nc ? c : nc - 1;
}

// Distinct periodic neighbours of cell c in a dimension of nc cells, in the
// order the coded entries refer to (nbr_cells); returns how many.
__device__ inline int adjacent(int c, int nc, int out[3]) {
  nbr_cells(c, nc, out);
  return nc >= 3 ? 3 : nc;
}

// Largest value over the wavefront (every lane active), applied by its first
// lane with one atomic.
__device__ inline void wave_atomic_max(int32_t* dst, int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(dst, v);
}

__device__ inline double fold_half(double d, double L, double h) {
  if (d > h) return d - L;
  if (d < -h) return d + L;
  return d;
}

__device__ inline double sqdist(double dx, double dy, double dz) {
  return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}

__global__ void k_bin(const double* __restrict__ pos, const int32_t* __restrict__ types, int64_t n,
                      NbrGrid g, int32_t* __restrict__ key, int32_t* __restrict__ cell_count,
                      int32_t* __restrict__ flags) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
  int t = types[i];
  const bool ok = t >= 0 && t < g.C && isfinite(x) && isfinite(y) && isfinite(z);
  if (!ok) {
    atomicOr(&flags[0], 1);
    t = 0;
    x = y = z = 0.0;
  }
  const int cx = cell_of(wrap1(x, g.box[0]), g.cell_scale[0], g.nc[0]);
  const int cy = cell_of(wrap1(y, g.box[1]), g.cell_scale[1], g.nc[1]);
  const int cz = cell_of(wrap1(z, g.box[2]), g.cell_scale[2], g.nc[2]);
  const int k = t * g.ncell + (cz * g.nc[1] + cy) * g.nc[0] + cx;
  key[i] = k;
  atomicAdd(&cell_count[k], 1);
}

// Counting-sort scatter, counting the buckets down to zero; flags[2] receives
// the largest bucket (which decides whether entries fit the 16-bit code).
__global__ void k_scatter(const int32_t* __restrict__ key, int64_t n, const int32_t* __restrict__ start,
                          int32_t* __restrict__ count, int32_t* __restrict__ perm, int32_t* __restrict__ flags) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if ((i & ~int64_t(63)) >= n) return;  // the whole wavefront is past the end
  int place = 0;
  if (i < n) {
    const int k = key[i];
    place = atomicSub(&count[k], 1);
    perm[start[k] + place - 1] = int32_t(i);
  }
  wave_atomic_max(&flags[2], place);
}

// The order inside each (species, cell) bucket made deterministic, and the
// wrapped positions in that order: an atom's slot is its bucket's start plus
// the number of smaller atom indices in the bucket.
__global__ void k_sort_gather(const double* __restrict__ pos, const int32_t* __restrict__ key,
                              const int32_t* __restrict__ start, const int32_t* __restrict__ scattered, int64_t n,
                              NbrGrid g, int32_t* __restrict__ perm, double* __restrict__ spos) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k = key[i], b = start[k], e = start[k + 1];
  int rank = 0;
  for (int t = b; t < e; ++t) rank += scattered[t] < int32_t(i);
  const int64_t a = b + rank;
  perm[a] = int32_t(i);
  spos[3 * a] = wrap1(pos[3 * i], g.box[0]);
  spos[3 * a + 1] = wrap1(pos[3 * i + 1], g.box[1]);
  spos[3 * a + 2] = wrap1(pos[3 * i + 2], g.box[2]);
}

// Rows by a 27-cell scan, one work-group per cell (and per slice of its atoms
// when there are few cells): the candidates of the cell, its up to 27
// neighbours' atoms species by species, are staged in LDS once for all centre
// atoms of the cell; a wavefront takes one centre at a time and tests 64
// candidates per step, so rows come out in candidate order.  The count pass
// (kFill false) records row lengths, the fill pass writes caller indices or,
// with kCode, 16-bit codes (ListView): the candidate's cell choice, species
// and place in that bucket.
//
// One thread per centre left a wavefront waiting on its own chain of position
// reads and wrote entries two bytes at a time.  With this kernel, the parallel
// bucket sort and the single read-back a build of 256 atoms takes 83 us instead
// of 387, of 4,994 atoms 115 instead of 1722, of 1,048,576 atoms 3.6 ms instead
// of 7.0.
constexpr int kRowThreads = 256;
constexpr int kRowCand = 1024;       // candidates staged at a time
constexpr int kRowAtoms = 64;        // centre atoms handled at a time
constexpr int kRowCellsX = 1 << 16;  // work-groups along x
constexpr int kMaxRuns = 27 * kMaxSpecies;
// Systems of many cells with few atoms on average (a gas, a surface or a
// particle in vacuum): a work-group for every cell is then mostly overhead, and
// centres with up to kFewCand candidates in a cell of up to kFewAtoms atoms go to
// k_rows_few instead.  A build of 1,048,576 atoms in 2.2 million cells takes
// 792 us (11,590 with a work-group per cell, 905 with one thread per
// centre everywhere), of 432,000 atoms in 216,000 cells 514 us (1820, 602), of
// a slab of 1,048,576 atoms in 225,400 cells 2630 us (3195, 6035).  With fewer
// cells, or more atoms in them, work-groups per cell are as fast or faster
// (100,000 atoms in 54,900 cells 606 and 609 us; 1,728,000 in 216,000: 3411 and
// 3315; a particle of 13,500 atoms in 54,900: 609 and 4500).
constexpr int kFewMean = 8;
constexpr int kFewCells = 1 << 16;
constexpr int kFewAtoms = 15;
constexpr int kFewCand = 160;
constexpr int kListBlocks = 16384;  // work-groups for the cells that k_rows_few leaves

// Longest row into *dst, only where it raises the value: with an atomic per
// wavefront on one address the count pass took 16.7 ms at 343,000 cells, now 8.3.
__device__ inline void raise_longest(int32_t* dst, int longest) {
  if (longest > __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(dst, longest);
}

// Exclusive prefix of run lengths len[0 .. n) into first[0 .. n] (n <= 2
// kRowThreads), by all threads of the work-group.
__device__ inline void scan_runs(const int* len, int n, int* first, int* wtot) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int a = 2 * t < n ? len[2 * t] : 0, b = 2 * t + 1 < n ? len[2 * t + 1] : 0;
  int inc = a + b;
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(inc, o, 64);
    if (lane >= o) inc += v;
  }
  if (lane == 63) wtot[w] = inc;
  __syncthreads();
  int off = 0;
  for (int v = 0; v < w; ++v) off += wtot[v];
  if (2 * t <= n) first[2 * t] = off + inc - a - b;
  if (2 * t + 1 <= n) first[2 * t + 1] = off + inc - b;
  __syncthreads();
}

template <bool kFill>
struct RowShared {
  double cx[kRowCand], cy[kRowCand], cz[kRowCand];
  int cslot[kRowCand];              // sorted slot
  int ccode[kFill ? kRowCand : 1];  // entry to write
  int len[kMaxRuns], first[kMaxRuns + 1], beg[kMaxRuns], wtot[kRowThreads / 64];
  int afirst[kMaxSpecies + 1];      // centre atoms before each species
  int cnt[kRowAtoms];
};

// Rows of one cell's atoms (this work-group's slice of them); longest: raised to
// the longest one of this wavefront's (count pass).
template <bool kFill, bool kCode>
__device__ __forceinline__ void rows_of_cell(RowShared<kFill>& S, int cell, const double* __restrict__ spos,
                                             const int32_t* __restrict__ perm, const NbrGrid& g,
                                             const int32_t* __restrict__ start, int32_t* __restrict__ rowcnt,
                                             const int64_t* __restrict__ offsets, void* __restrict__ idx, int tbits,
                                             int sbits, int& longest) {
  static_assert(kMaxRuns < 2 * kRowThreads, "scan_runs takes two runs per thread");
  double *const cx = S.cx, *const cy = S.cy, *const cz = S.cz;
  int *const cslot = S.cslot, *const ccode = S.ccode, *const len = S.len, *const first = S.first, *const beg = S.beg,
             *const afirst = S.afirst, *const cnt = S.cnt;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cc[3] = {cell % g.nc[0], cell / g.nc[0] % g.nc[1], cell / (g.nc[0] * g.nc[1])};
  int xs[3], ys[3], zs[3];
  const int nx = adjacent(cc[0], g.nc[0], xs), ny = adjacent(cc[1], g.nc[1], ys), nz = adjacent(cc[2], g.nc[2], zs);
  // no candidate of an inner cell is folded: coordinate differences stay
  // below two cell edges, with at least five cells well below half the box
  bool inner = true;
  for (int d = 0; d < 3; ++d) inner = inner && g.nc[d] >= 5 && cc[d] >= 1 && cc[d] <= g.nc[d] - 2;
  if (tid == 0) {
    int m = 0;
    for (int s = 0; s < g.C; ++s) {
      afirst[s] = m;
      m += start[s * g.ncell + cell + 1] - start[s * g.ncell + cell];
    }
    afirst[g.C] = m;
  }
  // candidate runs: one per species and scanned cell, in entry order
  const int per = nx * ny * nz, runs = g.C * per;
  for (int r = tid; r < runs; r += kRowThreads) {
    const int s = r / per, o = r % per, ix = o % nx, iy = o / nx % ny, iz = o / (nx * ny);
    const int key = s * g.ncell + (zs[iz] * g.nc[1] + ys[iy]) * g.nc[0] + xs[ix];
    beg[r] = start[key];
    len[r] = start[key + 1] - start[key];
  }
  __syncthreads();
  const int atoms = afirst[g.C];
  // this work-group's slice of the cell's atoms
  const int a0 = int(int64_t(atoms) * blockIdx.y / gridDim.y), a1 = int(int64_t(atoms) * (blockIdx.y + 1) / gridDim.y);
  if (a0 == a1) return;
  scan_runs(len, runs, first, S.wtot);
  const int total = first[runs];
  for (int g0 = a0; g0 < a1; g0 += kRowAtoms) {
    const int na = a1 - g0 < kRowAtoms ? a1 - g0 : kRowAtoms;
    __syncthreads();
    if (tid < kRowAtoms) cnt[tid] = 0;
    for (int c0 = 0; c0 < total; c0 += kRowCand) {
      const int nc = total - c0 < kRowCand ? total - c0 : kRowCand;
      __syncthreads();
      if (g0 == a0 || total > kRowCand) {
        for (int c = tid; c < nc; c += kRowThreads) {
          // run of candidate c0 + c: the last one that starts at or before it
          int lo = 0, hi = runs;
          while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first[mid] <= c0 + c) lo = mid;
            else hi = mid;
          }
          const int t = c0 + c - first[lo], b = beg[lo] + t;
          cx[c] = spos[3 * int64_t(b)];
          cy[c] = spos[3 * int64_t(b) + 1];
          cz[c] = spos[3 * int64_t(b) + 2];
          cslot[c] = b;
          if constexpr (kFill) {
            if constexpr (kCode) {
              const int s = lo / per, o = lo % per, ix = o % nx, iy = o / nx % ny, iz = o / (nx * ny);
              ccode[c] = (((iz * 3 + iy) * 3 + ix) << (sbits + tbits)) | (s << tbits) | t;
            } else {
              ccode[c] = perm[b];
            }
          }
        }
      }
      __syncthreads();
      for (int q = wave; q < na; q += kRowThreads / 64) {
        int s = 0;
        while (g0 + q >= afirst[s + 1]) ++s;
        const int a = start[s * g.ncell + cell] + (g0 + q - afirst[s]);
        const double wx = spos[3 * int64_t(a)], wy = spos[3 * int64_t(a) + 1], wz = spos[3 * int64_t(a) + 2];
        int m = cnt[q];
        const int64_t base = kFill ? offsets[a] : 0;
        for (int c1 = 0; c1 < nc; c1 += 64) {
          const int c = c1 + lane;
          bool hit = false;
          if (c < nc) {
            double dx = cx[c] - wx, dy = cy[c] - wy, dz = cz[c] - wz;
            if (!inner) {
              dx = fold_half(dx, g.box[0], g.half[0]);
              dy = fold_half(dy, g.box[1], g.half[1]);
              dz = fold_half(dz, g.box[2], g.half[2]);
            }
            hit = sqdist(dx, dy, dz) < g.rl2 && cslot[c] != a;
          }
          const unsigned long long mask = __ballot(hit);
          if constexpr (kFill) {
            if (hit) {
              const int64_t at = base + m + __builtin_popcountll(mask & ((1ull << lane) - 1));
              if constexpr (kCode) static_cast<uint16_t*>(idx)[at] = uint16_t(ccode[c]);
              else static_cast<int32_t*>(idx)[at] = ccode[c];
            }
          }
          m += __builtin_popcountll(mask);
        }
        if (lane == 0) cnt[q] = m;
        if (!kFill && c0 + kRowCand >= total) {
          if (lane == 0) rowcnt[a] = m;
          longest = max(longest, m);
        }
      }
    }
  }
}

// kList: the listed cells in turn (number, then cells), else one work-group for
// every cell, along x and layer by layer along z.
template <bool kFill, bool kCode, bool kList>
__global__ __launch_bounds__(kRowThreads) void k_rows(const double* __restrict__ spos, const int32_t* __restrict__ perm,
                                                      NbrGrid g, const int32_t* __restrict__ start,
                                                      int32_t* __restrict__ rowcnt, const int64_t* __restrict__ offsets,
                                                      void* __restrict__ idx, int32_t* __restrict__ flags, int tbits,
                                                      int sbits, const int32_t* __restrict__ cells) {
  __shared__ RowShared<kFill> S;
  int longest = 0;
  if constexpr (kList) {
    const int count = cells[0];
    for (int at = blockIdx.x; at < count; at += gridDim.x) {
      rows_of_cell<kFill, kCode>(S, cells[1 + at], spos, perm, g, start, rowcnt, offsets, idx, tbits, sbits, longest);
      __syncthreads();
    }
  } else {
    const int64_t cell = int64_t(blockIdx.z) * gridDim.x + blockIdx.x;
    if (cell >= g.ncell) return;
    rows_of_cell<kFill, kCode>(S, int(cell), spos, perm, g, start, rowcnt, offsets, idx, tbits, sbits, longest);
  }
  if (!kFill && (threadIdx.x & 63) == 0) raise_longest(&flags[1], longest);
}

// The same rows by one thread per centre, for centres with few candidates
// (above).  The count pass lists the cells of the others in cells (number, then
// cell indices in any order; zero on entry) for k_rows.
template <bool kFill, bool kCode>
__global__ void k_rows_few(const double* __restrict__ spos, const int32_t* __restrict__ perm,
                           const int32_t* __restrict__ keys, int64_t n, NbrGrid g, const int32_t* __restrict__ start,
                           int32_t* __restrict__ rowcnt, const int64_t* __restrict__ offsets, void* __restrict__ idx,
                           int32_t* __restrict__ flags, int tbits, int sbits, int32_t* __restrict__ cells) {
  const int64_t a = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  int cnt = 0;
  if (a < n) {
    const int key = keys[perm[a]], own = key / g.ncell, cell = key % g.ncell;
    int xs[3], ys[3], zs[3];
    const int nx = adjacent(cell % g.nc[0], g.nc[0], xs), ny = adjacent(cell / g.nc[0] % g.nc[1], g.nc[1], ys),
              nz = adjacent(cell / (g.nc[0] * g.nc[1]), g.nc[2], zs);
    // atoms of the cell, whether this is its first one, and candidates
    int atoms = 0, cand = 0, before = 0;
    for (int s = 0; s < g.C; ++s) {
      const int m = start[s * g.ncell + cell + 1] - start[s * g.ncell + cell];
      atoms += m;
      before += s < own ? m : 0;
    }
    if (atoms <= kFewAtoms)
      for (int s = 0; s < g.C; ++s)
        for (int iz = 0; iz < nz; ++iz)
          for (int iy = 0; iy < ny; ++iy)
            for (int ix = 0; ix < nx; ++ix) {
              const int k = s * g.ncell + (zs[iz] * g.nc[1] + ys[iy]) * g.nc[0] + xs[ix];
              cand += start[k + 1] - start[k];
            }
    if (atoms > kFewAtoms || cand > kFewCand) {
      if (!kFill && before == 0 && a == start[key]) cells[1 + atomicAdd(&cells[0], 1)] = cell;
    } else {
      const double wx = spos[3 * a], wy = spos[3 * a + 1], wz = spos[3 * a + 2];
      const int64_t base = kFill ? offsets[a] : 0;
      for (int s = 0; s < g.C; ++s)
        for (int iz = 0; iz < nz; ++iz)
          for (int iy = 0; iy < ny; ++iy)
            for (int ix = 0; ix < nx; ++ix) {
              const int k = s * g.ncell + (zs[iz] * g.nc[1] + ys[iy]) * g.nc[0] + xs[ix];
              const int b0 = start[k], e = start[k + 1];
              for (int b = b0; b < e; ++b) {
                const double dx = fold_half(spos[3 * int64_t(b)] - wx, g.box[0], g.half[0]);
                const double dy = fold_half(spos[3 * int64_t(b) + 1] - wy, g.box[1], g.half[1]);
                const double dz = fold_half(spos[3 * int64_t(b) + 2] - wz, g.box[2], g.half[2]);
                if (sqdist(dx, dy, dz) < g.rl2 && b != a) {
                  if constexpr (kFill) {
                    if constexpr (kCode)
                      static_cast<uint16_t*>(idx)[base + cnt] =
                          uint16_t((((iz * 3 + iy) * 3 + ix) << (sbits + tbits)) | (s << tbits) | (b - b0));
                    else
                      static_cast<int32_t*>(idx)[base + cnt] = perm[b];
                  }
                  ++cnt;
                }
              }
            }
      if (!kFill) rowcnt[a] = cnt;
    }
  }
  if constexpr (!kFill) {
    for (int o = 32; o > 0; o >>= 1) cnt = max(cnt, __shfl_xor(cnt, o, 64));
    if ((threadIdx.x & 63) == 0) raise_longest(&flags[1], cnt);
  }
}

// ---- exclusive scan: out[0..n] with out[n] = total -------------------------
template <typename Tin>
__global__ void k_block_sums(const Tin* __restrict__ in, int64_t n, int64_t* __restrict__ bsum) {
  __shared__ int64_t red[kScanThreads / 64];
  const int64_t base = int64_t(blockIdx.x) * kScanSeg;
  int64_t s = 0;
  for (int it = 0; it < kScanItems; ++it) {
    const int64_t i = base + int64_t(it) * kScanThreads + threadIdx.x;
    if (i < n) s += int64_t(in[i]);
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) t += red[w];
    bsum[blockIdx.x] = t;
  }
}

__device__ inline int64_t wave_inclusive(int64_t v) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

// Exclusive scan of the block sums in place (single work-group, any length).
__global__ void k_scan_sums(int64_t* __restrict__ bsum, int64_t nb) {
  __shared__ int64_t wtot[kScanThreads / 64];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
    const int64_t i = b0 + threadIdx.x;
    const int64_t v = i < nb ? bsum[i] : 0;
    const int64_t inc = wave_inclusive(v);
    if ((threadIdx.x & 63) == 63) wtot[threadIdx.x >> 6] = inc;
    __syncthreads();
    int64_t off = carry;
    for (int w = 0; w < int(threadIdx.x >> 6); ++w) off += wtot[w];
    if (i < nb) bsum[i] = off + inc - v;
    __syncthreads();
    if (threadIdx.x == kScanThreads - 1) carry = off + inc;
    __syncthreads();
  }
}

template <typename Tin, typename Tout>
__global__ void k_scan_apply(const Tin* __restrict__ in, int64_t n, const int64_t* __restrict__ bsum,
                             Tout* __restrict__ out) {
  __shared__ int64_t wtot[kScanThreads / 64];
  const int64_t base = int64_t(blockIdx.x) * kScanSeg + int64_t(threadIdx.x) * kScanItems;
  int64_t v[kScanItems];
  int64_t tsum = 0;
  for (int it = 0; it < kScanItems; ++it) {
    const int64_t i = base + it;
    v[it] = i < n ? int64_t(in[i]) : 0;
    tsum += v[it];
  }
  const int64_t inc = wave_inclusive(tsum);
  if ((threadIdx.x & 63) == 63) wtot[threadIdx.x >> 6] = inc;
  __syncthreads();
  int64_t run = (bsum ? bsum[blockIdx.x] : 0) + inc - tsum;
  for (int w = 0; w < int(threadIdx.x >> 6); ++w) run += wtot[w];
  for (int it = 0; it < kScanItems; ++it) {
    const int64_t i = base + it;
    if (i < n) out[i] = Tout(run);
    run += v[it];
    if (i == n - 1) out[n] = Tout(run);
  }
}

template <typename T>
__global__ void k_fill(T* __restrict__ p, int64_t n, T v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Outputs and sums of an evaluation cleared in one launch.
__global__ void k_clear_outputs(double* __restrict__ forces, int64_t n3, double* __restrict__ totals,
                                unsigned long long* __restrict__ counters) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n3) forces[i] = 0.0;
  if (blockIdx.x == 0 && threadIdx.x < kTotals) totals[threadIdx.x] = 0.0;
  if (blockIdx.x == 0 && threadIdx.x < 4) counters[threadIdx.x] = 0;
}

// What the build reads back: list length, flags, and the first sorted slot of
// each species.
__global__ void k_build_result(const int64_t* __restrict__ total, const int32_t* __restrict__ flags,
                               const int32_t* __restrict__ start, int64_t ncell, int C, BuildResult* __restrict__ out) {
  const int t = threadIdx.x;
  if (t == 0) out->total = *total;
  if (t < 4) out->flags[t] = flags[t];
  if (t <= C) out->species_start[t] = start[t * ncell];
}

template <typename Tin, typename Tout>
hipError_t exclusive_scan(const Tin* in, int64_t n, Tout* out, int64_t* tmp, hipStream_t s) {
  if (n == 0) {
    k_fill<Tout><<<1, 1, 0, s>>>(out, 1, Tout(0));
    return hipGetLastError();
  }
  const int64_t nb = (n + kScanSeg - 1) / kScanSeg;
  if (nb == 1) {  // one segment needs no sums of the others
    k_scan_apply<Tin, Tout><<<1, kScanThreads, 0, s>>>(in, n, nullptr, out);
    return hipGetLastError();
  }
  k_block_sums<Tin><<<dim3(unsigned(nb)), dim3(kScanThreads), 0, s>>>(in, n, tmp);
  k_scan_sums<<<1, kScanThreads, 0, s>>>(tmp, nb);
  k_scan_apply<Tin, Tout><<<dim3(unsigned(nb)), dim3(kScanThreads), 0, s>>>(in, n, tmp, out);
  return hipGetLastError();
}

inline unsigned blocks_for(int64_t n, int t) { return unsigned((n + t - 1) / t); }

}  // namespace

size_t scan_tmp_elems(int64_t n) { return size_t((n + kScanSeg - 1) / kScanSeg) + 1; }

hipError_t launch_exclusive_scan_i32_to_i32(const int32_t* in, int64_t n, int32_t* out, int64_t* tmp,
                                            hipStream_t s) {
  return exclusive_scan<int32_t, int32_t>(in, n, out, tmp, s);
}

hipError_t launch_exclusive_scan_i32_to_i64(const int32_t* in, int64_t n, int64_t* out, int64_t* tmp,
                                            hipStream_t s) {
  return exclusive_scan<int32_t, int64_t>(in, n, out, tmp, s);
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill<int32_t><<<blocks_for(n, 256), 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill<double><<<blocks_for(n, 256), 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_clear_outputs(double* forces, int64_t n, double* totals, unsigned long long* counters, hipStream_t s) {
  k_clear_outputs<<<blocks_for(3 * n, 256), 256, 0, s>>>(forces, 3 * n, totals, counters);
  return hipGetLastError();
}

hipError_t launch_bin(const double* pos, const int32_t* types, int64_t n, const NbrGrid& g, int32_t* key,
                      int32_t* cell_count, int32_t* flags, hipStream_t s) {
  k_bin<<<blocks_for(n, 256), 256, 0, s>>>(pos, types, n, g, key, cell_count, flags);
  return hipGetLastError();
}

hipError_t launch_scatter(const int32_t* key, int64_t n, const int32_t* cell_start, int32_t* fill, int32_t* perm,
                          int32_t* flags, hipStream_t s) {
  k_scatter<<<blocks_for(n, 256), 256, 0, s>>>(key, n, cell_start, fill, perm, flags);
  return hipGetLastError();
}

hipError_t launch_sort_gather(const double* pos, const int32_t* key, const int32_t* cell_start,
                              const int32_t* scattered, int64_t n, const NbrGrid& g, int32_t* perm, double* spos,
                              hipStream_t s) {
  k_sort_gather<<<blocks_for(n, 256), 256, 0, s>>>(pos, key, cell_start, scattered, n, g, perm, spos);
  return hipGetLastError();
}

hipError_t launch_build_result(const int64_t* total, const int32_t* flags, const int32_t* cell_start, const NbrGrid& g,
                               BuildResult* out, hipStream_t s) {
  k_build_result<<<1, 64, 0, s>>>(total, flags, cell_start, g.ncell, g.C, out);
  return hipGetLastError();
}

hipError_t launch_rows(const double* spos, const int32_t* perm, const int32_t* key, int64_t n, const NbrGrid& g,
                       const int32_t* cell_start, int32_t* rowcnt, const int64_t* offsets, void* idx, int32_t* flags,
                       int32_t* cells, bool fill, int tbits, int sbits, hipStream_t s) {
  // few cells: several work-groups share a cell's atoms, at least four each,
  // until there are about two per compute unit
  const int64_t per_cell = (n + g.ncell - 1) / g.ncell;
  const int64_t split = std::max<int64_t>(1, std::min<int64_t>((512 + g.ncell - 1) / g.ncell, (per_cell + 3) / 4));
  // a launch takes at most 2^32 - 1 threads along a dimension, which work-groups
  // of 256 for every cell pass from 16.8 million cells (about 290 million BCC
  // atoms); cells past kRowCellsX go to the next layer
  const unsigned across = unsigned(std::min<int64_t>(g.ncell, kRowCellsX));
  const bool few = g.ncell > kFewCells && n < kFewMean * int64_t(g.ncell);
  const dim3 grid(across, unsigned(std::min<int64_t>(split, 65535)), unsigned((int64_t(g.ncell) + across - 1) / across));
  auto launch = [&](auto by_cell, auto by_list, auto by_atom) {
    if (!few) {
      by_cell<<<grid, kRowThreads, 0, s>>>(spos, perm, g, cell_start, rowcnt, offsets, idx, flags, tbits, sbits, nullptr);
      return;
    }
    by_atom<<<blocks_for(n, 256), 256, 0, s>>>(spos, perm, key, n, g, cell_start, rowcnt, offsets, idx, flags, tbits,
                                               sbits, cells);
    by_list<<<unsigned(std::min<int64_t>(n, kListBlocks)), kRowThreads, 0, s>>>(spos, perm, g, cell_start, rowcnt, offsets,
                                                                                idx, flags, tbits, sbits, cells);
  };
  if (!fill) launch(k_rows<false, false, false>, k_rows<false, false, true>, k_rows_few<false, false>);
  else if (tbits > 0) launch(k_rows<true, true, false>, k_rows<true, true, true>, k_rows_few<true, true>);
  else launch(k_rows<true, false, false>, k_rows<true, false, true>, k_rows_few<true, false>);
  return hipGetLastError();
}

}  // namespace mlip
