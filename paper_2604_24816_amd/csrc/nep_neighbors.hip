// Cell binning, stable sort of atoms by cell, and neighbour-list construction.
//
// Atoms are kept sorted by (cell, original id) so that the atoms one wavefront
// handles, and their neighbours, are contiguous in HBM. Lists are stored
// slot-major ([slot][N]) so that lane i of a wavefront reads the list entry of
// atom i: consecutive lanes touch consecutive words.
//
// Pair membership is decided by r^2 < (cutoff + skin)^2 with FP64 minimum-image
// differences and r^2 = (dx*dx + dy*dy) + dz*dz, evaluated without fused
// multiply-add so that the set is reproducible bit for bit (Section VI.A
// neighbour-list buffer; Fig. 1 radial and angular cutoffs).
#include "nep_common.h"

namespace nep {
namespace {

__global__ void k_clear(int32_t* flags, int32_t* cells, int ncell, int32_t* nbr, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) nbr[i] = 0;
  if (i < FLAG_COUNT) flags[i] = 0;
  for (int64_t c = i; c < ncell; c += (int64_t)gridDim.x * blockDim.x) cells[c] = 0;
}

// Workgroups of the rebuild kernels. Every rebuild kernel is enqueued each step and
// returns at once when no rebuild is due, so there are few of them (a dispatch that does
// nothing still takes about 2 us of the step) and the per-atom and per-cell ones stride
// over a capped grid (a multiple of the 8 dies, so that a workgroup stays on its die): a
// step without a rebuild then dispatches a few thousand workgroups, not one per cell or per
// 256 atoms.
constexpr int kRebuildGrid = 8192;
constexpr int kCopyGrid = 2048;  // workgroups that copy the sorted state back (a multiple of the dies)
inline int rebuild_grid(int64_t nblocks) { return (int)(nblocks < kRebuildGrid ? nblocks : kRebuildGrid); }

__device__ __forceinline__ int cell_coord(double xv, double L, int n) {
  int c = (int)(xv * ((double)n / L));
  if (c < 0) c = 0;
  if (c > n - 1) c = n - 1;
  return c;
}

__device__ __forceinline__ int cell_of(const CellGrid& g, const double* __restrict__ x, int64_t N, int64_t p) {
  return cell_lin(g, cell_coord(x[p], g.box[0], g.nc[0]), cell_coord(x[N + p], g.box[1], g.nc[1]),
                  cell_coord(x[2 * N + p], g.box[2], g.nc[2]));
}

// Inclusive prefix sum over the lanes of a wavefront.
__device__ __forceinline__ int wave_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    v += lane >= o ? t : 0;
  }
  return v;
}

// Exclusive prefix sum over a workgroup of WAVES wavefronts, the total in tot; sh holds
// WAVES ints. Two barriers; sh may be reused after a further one.
template <int WAVES>
__device__ __forceinline__ int block_scan(int v, int* sh, int& tot) {
  const int incl = wave_scan(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 63) sh[w] = incl;
  __syncthreads();
  int before = 0;
  tot = 0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const int t = sh[k];
    before += k < w ? t : 0;
    tot += t;
  }
  return before + incl - v;
}

// The step's rebuild decision and the distance bins its evaluations visit: from d2, the
// largest squared displacement since the build. REBUILD is set on a scheduled step and when
// an atom has moved more than skin / 2. k = first bin fraction with bin_frac(k) * skin >=
// 2 sqrt(d2); the evaluation visits the bins up to the edges rc_radial + f_k skin and
// rc_angular + f_k skin; after a build the displacements are 0, so k = 0. One thread.
__device__ void select_bins(const RebuildRule& rule, double d2, int32_t* flags) {
  if (rule.reset)
    for (int k = 0; k < FLAG_COUNT; ++k) flags[k] = 0;
  const int build = rule.scheduled || d2 > rule.half_skin2;
  flags[FLAG_REBUILD] = build;
  const double d = build ? 0.0 : sqrt(d2);
  int k = kFracs - 1;
  for (int j = kFracs - 1; j >= 0; --j)
    if ((double)bin_frac(j) * rule.skin >= 2.0 * d * (1.0 + 1e-12)) k = j;
  int br0 = 0, ba0 = 0, br1 = 0, ba1 = 0;
  for (int j = 0; j < kFracs; ++j)
    if (j == k) {
      br0 = rule.be.idxR[0][j];
      ba0 = rule.be.idxA[0][j];
      br1 = rule.be.idxR[1][j];
      ba1 = rule.be.idxA[1][j];
    }
  flags[FLAG_BIN_R] = br0;
  flags[FLAG_BIN_A] = ba0;
  flags[FLAG_BIN_R1] = br1;
  flags[FLAG_BIN_A1] = ba1;
  if (build) flags[FLAG_NBUILD] += 1;
}

// Whether the step rebuilds: from the largest of the n partial maxima (the same in every
// workgroup that asks), with the flag words set when `write`. sh holds BLOCK / 64 doubles.
constexpr int kSelBlock = 1024;
template <int BLOCK>
__device__ __forceinline__ bool decide(const RebuildRule& rule, const double* __restrict__ d2, int n, bool write,
                                       int32_t* __restrict__ flags, double* sh) {
  double m = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < n; b += BLOCK) m = fmax(m, d2[b]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  m = sh[0];
#pragma unroll
  for (int k = 1; k < BLOCK / 64; ++k) m = fmax(m, sh[k]);
  if (write && threadIdx.x == 0) select_bins(rule, m, flags);
  return rule.scheduled || m > rule.half_skin2;
}

__global__ void __launch_bounds__(kSelBlock)
k_select(RebuildRule rule, const double* __restrict__ d2, int nd2, int32_t* __restrict__ flags) {
  __shared__ double sh[kSelBlock / 64];
  decide<kSelBlock>(rule, d2, nd2, true, flags, sh);
}

// Systems of up to kSortAtoms atoms in kSortCells cells: the decision, the binning, the
// scan and the scatter in one workgroup, with the cell counts in LDS. One launch instead of
// four; beyond these sizes one workgroup is slower than the launches it saves.
constexpr int kSortAtoms = 16384, kSortCells = 2048;

__global__ void __launch_bounds__(kSelBlock)
k_select_sort(RebuildRule rule, const double* __restrict__ d2, int nd2, int64_t N, CellGrid g,
              const double* __restrict__ x, const int32_t* __restrict__ perm, int32_t* __restrict__ start,
              int32_t* __restrict__ src, int32_t* __restrict__ key, int32_t* __restrict__ flags) {
  __shared__ double shd[kSelBlock / 64];
  __shared__ int count[kSortCells], sh[kSelBlock / 64];
  const int t = threadIdx.x;
  if (!decide<kSelBlock>(rule, d2, nd2, true, flags, shd)) return;
  for (int c = t; c < kSortCells; c += kSelBlock) count[c] = 0;
  __syncthreads();
  constexpr int PER = kSortAtoms / kSelBlock;
  int cr[PER];  // cell | rank in the cell << 16
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t p = t + (int64_t)u * kSelBlock;
    cr[u] = 0;
    if (p < N) {
      const int c = cell_of(g, x, N, p);
      cr[u] = c | atomicAdd(&count[c], 1) << 16;
    }
  }
  __syncthreads();
  constexpr int CPER = kSortCells / kSelBlock;
  int v[CPER], sum = 0, tot;
#pragma unroll
  for (int k = 0; k < CPER; ++k) {
    v[k] = count[CPER * t + k];
    sum += v[k];
  }
  int run = block_scan<kSelBlock / 64>(sum, sh, tot);
#pragma unroll
  for (int k = 0; k < CPER; ++k) {
    const int c = CPER * t + k;
    count[c] = run;
    if (c <= g.ncell) start[c] = run;  // start[ncell] = N: the cells past the grid are empty
    run += v[k];
  }
  if (t == 0 && g.ncell == kSortCells) start[g.ncell] = tot;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t p = t + (int64_t)u * kSelBlock;
    if (p < N) {
      const int pos = count[cr[u] & 0xffff] + (cr[u] >> 16);
      src[pos] = (int32_t)p;
      key[pos] = perm[p];
    }
  }
}

// Cell of every atom and its rank among the cell's atoms in arrival order. count is zero
// on entry (k_sort_halo clears it for the next build). DECIDE: the rebuild decision is taken
// here, by every workgroup for itself from at most kDecideMax partial maxima, which saves
// the launch of k_select; with more of them their re-reading would cost more.
constexpr int kDecideMax = 1024;
template <bool DECIDE>
__global__ void __launch_bounds__(kBlock)
k_bin(RebuildRule rule, const double* __restrict__ d2, int nd2, int64_t N, CellGrid g, const double* __restrict__ x,
      int32_t* __restrict__ cellid, int32_t* __restrict__ rank, int32_t* __restrict__ count,
      int32_t* __restrict__ flags) {
  __shared__ double sh[kBlock / 64];
  if constexpr (DECIDE) {
    if (!decide<kBlock>(rule, d2, nd2, blockIdx.x == 0, flags, sh)) return;
  } else if (flags[FLAG_REBUILD] == 0) {
    return;
  }
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
    const int c = cell_of(g, x, N, p);
    cellid[p] = c;
    rank[p] = atomicAdd(&count[c], 1);
  }
}

// Exclusive scan of the cell counts: each workgroup scans 1024 cells and leaves its total;
// k_scan_add then adds the totals of the workgroups before.
constexpr int kScanPer = 4;
constexpr int kScanTile = kBlock * kScanPer;

__global__ void k_scan_tiles(const int32_t* __restrict__ in, int32_t* __restrict__ out, int n,
                             int32_t* __restrict__ tile_sums, const int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  __shared__ int sh[kBlock / 64];
  const int base = blockIdx.x * kScanTile + threadIdx.x * kScanPer;
  int32_t v[kScanPer];
  int sum = 0, tot;
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0;
    sum += v[k];
  }
  int run = block_scan<kBlock / 64>(sum, sh, tot);
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kScanTile)
k_scan_add(int32_t* __restrict__ out, int n, int64_t N, const int32_t* __restrict__ sums,
           const int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  __shared__ int sh[kScanTile / 64];
  int s = 0, before;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += kScanTile) s += sums[b];
  block_scan<kScanTile / 64>(s, sh, before);
  const int i = blockIdx.x * kScanTile + threadIdx.x;
  if (i < n) out[i] += before;
  if (i == n - 1) out[n] = (int32_t)N;
}

__global__ void k_scatter(int64_t N, const int32_t* __restrict__ cellid, const int32_t* __restrict__ rank,
                          const int32_t* __restrict__ start, const int32_t* __restrict__ perm,
                          int32_t* __restrict__ src, int32_t* __restrict__ key,
                          const int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
    const int pos = start[cellid[p]] + rank[p];
    src[pos] = (int32_t)p;
    key[pos] = perm[p];
  }
}

// Up to kScanCells cells: every workgroup scans all the counts itself, in LDS, and scatters
// its atoms (the first also stores the starts): one launch instead of three.
constexpr int kScanCells = 8192;
__global__ void __launch_bounds__(kBlock)
k_scan_scatter(int64_t N, int ncell, const int32_t* __restrict__ count, const int32_t* __restrict__ cellid,
               const int32_t* __restrict__ rank, const int32_t* __restrict__ perm, int32_t* __restrict__ start,
               int32_t* __restrict__ src, int32_t* __restrict__ key, const int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  __shared__ int st[kScanCells];
  __shared__ int sh[kBlock / 64];
  for (int c = threadIdx.x; c < ncell; c += kBlock) st[c] = count[c];
  __syncthreads();
  const int per = (ncell + kBlock - 1) / kBlock;
  const int c0 = threadIdx.x * per, c1 = c0 + per < ncell ? c0 + per : ncell;
  int sum = 0, tot;
  for (int c = c0; c < c1; ++c) sum += st[c];
  int run = block_scan<kBlock / 64>(sum, sh, tot);
  for (int c = c0; c < c1; ++c) {
    const int v = st[c];
    st[c] = run;
    run += v;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int c = threadIdx.x; c < ncell; c += kBlock) start[c] = st[c];
    if (threadIdx.x == 0) start[ncell] = (int32_t)N;
  }
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
    const int pos = st[cellid[p]] + rank[p];
    src[pos] = (int32_t)p;
    key[pos] = perm[p];
  }
}

// Within each cell, order atoms by original id and move their state there. One wavefront
// per cell: each lane holds atoms of the cell, counts the cell's smaller keys (the keys are
// distinct original ids) and moves its atom to that rank, so the result is the stable order
// whatever order the scatter's atomics left. The keys are read through LDS kSortMax at a
// time: once for a cell of up to that many atoms (all cells at metallic densities), once for
// each 64 atoms of a larger one. By one lane, with an insertion sort, those cost n^2
// dependent accesses: the list build of 4,000 atoms in one cell took 53 ms (30 so), of 1,200
// in a 10 A cube 5.3 (1.5).
constexpr int kSortMax = 256;
constexpr int kSortWaves = kBlock / 64;

// The sorted state of a build, in the alternate buffers until the positions that the build
// still reads in the old order are free (k_build_cells copies it back); xb stays, as the
// positions at the build.
struct SortedState {
  double *x2, *v2, *xb;
  int32_t *type2, *perm2;
};

__device__ void sort_cells(int64_t N, int ncell, const int32_t* __restrict__ start, int32_t* __restrict__ count,
                           int32_t* __restrict__ key, int32_t* __restrict__ src, const double* __restrict__ x,
                           const double* __restrict__ v, const int32_t* __restrict__ type, const SortedState& o,
                           int block, int nblocks, int32_t (*kk)[kSortMax]) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  constexpr int U = kSortMax / 64;
  for (int c = block * kSortWaves + w; c < ncell; c += nblocks * kSortWaves) {  // wave-uniform
    const int a = start[c], n = start[c + 1] - a;
    if (lane == 0) count[c] = 0;
    if (n <= 0) continue;
    // sorted atom p of the cell from atom s, original id k
    auto move = [&](int64_t p, int64_t s, int32_t k) {
      for (int d = 0; d < 3; ++d) {
        const double xv = x[d * N + s];
        o.x2[d * N + p] = xv;
        o.xb[d * N + p] = xv;
        o.v2[d * N + p] = v[d * N + s];
      }
      o.type2[p] = type[s];
      o.perm2[p] = k;
    };
    if (__builtin_expect(n > kSortMax, 0)) {
      for (int l0 = 0; l0 < n; l0 += 64) {  // 64 atoms, one to a lane
        const bool on = l0 + lane < n;
        const int32_t k = on ? key[a + l0 + lane] : 0;
        int rank = 0;
        for (int c0 = 0; c0 < n; c0 += kSortMax) {
          const int nk = n - c0 < kSortMax ? n - c0 : kSortMax;
          for (int l = lane; l < nk; l += 64) kk[w][l] = key[a + c0 + l];
          wave_lds_sync();
          for (int m = 0; m < nk; ++m) rank += kk[w][m] < k ? 1 : 0;
          wave_lds_sync();
        }
        if (on) move(a + rank, src[a + l0 + lane], k);
      }
      continue;
    }
    int32_t mk[U], ms[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int l = lane + 64 * u;
      mk[u] = l < n ? key[a + l] : 0;
      ms[u] = l < n ? src[a + l] : 0;
      if (l < n) kk[w][l] = mk[u];
    }
    wave_lds_sync();
    int rank[U];
#pragma unroll
    for (int u = 0; u < U; ++u) rank[u] = 0;
    for (int m = 0; m < n; ++m) {
      const int32_t km = kk[w][m];
#pragma unroll
      for (int u = 0; u < U; ++u) rank[u] += km < mk[u] ? 1 : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (lane + 64 * u < n) move(a + rank[u], ms[u], mk[u]);
    wave_lds_sync();
  }
}

// One workgroup per 256-atom tile: the tile's force halo (every non-empty cell within
// one cell, periodic, of a cell holding tile atoms), sorted by cell id, with local
// offsets. ok = 0 when the tile or its halo exceeds the LDS tables of the force kernel.
// The halo's cells are marked in a bitmap of the grid, which is then read in id order: no
// duplicates and no sort. Grids of more than kMapCells cells (above eight million atoms at
// metallic density), whose bitmap would not fit in LDS, sort the candidates instead (a
// bitonic sort of up to 2,048 ids, whose 66 barriers made this kernel 30 us even for a
// system of a few tiles).
constexpr int kMapCells = 262144;

__device__ void halo_none(int32_t* info) {
  if (threadIdx.x < 4) info[threadIdx.x] = 0;
}

// Stencil cell o (0..26) of cell c_lo + t / 27, or -1 when that cell or the stencil cell is
// empty.
__device__ __forceinline__ int halo_cand(const CellGrid& g, const int32_t* __restrict__ cell_start, int c_lo, int t) {
  const int c = c_lo + t / 27, o = t % 27;
  int cx, cy, cz;
  if (!(cell_start[c + 1] > cell_start[c] && cell_coords(g, c, cx, cy, cz))) return -1;
  const int nx = (cx + o % 3 - 1 + g.nc[0]) % g.nc[0];
  const int ny = (cy + (o / 3) % 3 - 1 + g.nc[1]) % g.nc[1];
  const int nz = (cz + o / 9 - 1 + g.nc[2]) % g.nc[2];
  const int v = cell_lin(g, nx, ny, nz);
  return cell_start[v + 1] > cell_start[v] ? v : -1;
}

template <bool MAP>
struct HaloWork {
  static constexpr int kWords = MAP ? kMapCells / 32 : kCandMax;
  uint32_t buf[kWords];  // bitmap, or candidate ids to sort
  int scan[kBlock / 64];
  int cnt[kHaloCellsMax];
};

template <bool MAP>
__device__ void halo_tile(int64_t N, const CellGrid& g, const double* __restrict__ x, const int32_t* __restrict__ src,
                          const int32_t* __restrict__ cell_start, const HaloTables& ht, int tile, HaloWork<MAP>& hw) {
  uint32_t* buf = hw.buf;
  int* scan = hw.scan;
  int* cnt = hw.cnt;
  const int64_t t0 = (int64_t)tile * kBlock;
  const int64_t t1 = t0 + kBlock < N ? t0 + kBlock : N;
  int32_t* info = ht.info + 4 * tile;
  // the cells of the tile's first and last atoms (src is ordered by cell; the order inside a
  // cell does not matter)
  const int c_lo = cell_of(g, x, N, src[t0]), c_hi = cell_of(g, x, N, src[t1 - 1]);
  const int ncr = c_hi - c_lo + 1;
  if (ncr > kTileCellsMax) return halo_none(info);
  int n_list = 64;  // words of buf in use
  if constexpr (MAP) {
    n_list = (g.ncell + 31) / 32;
    for (int t = threadIdx.x; t < n_list; t += kBlock) buf[t] = 0;
    __syncthreads();
    for (int t = threadIdx.x; t < 27 * ncr; t += kBlock) {
      const int v = halo_cand(g, cell_start, c_lo, t);
      if (v >= 0) atomicOr(&buf[v >> 5], 1u << (v & 31));
    }
    __syncthreads();
  } else {
    while (n_list < 27 * ncr) n_list <<= 1;
    for (int t = threadIdx.x; t < n_list; t += kBlock)
      buf[t] = t < 27 * ncr ? (uint32_t)halo_cand(g, cell_start, c_lo, t) : ~0u;
    __syncthreads();
    for (int k = 2; k <= n_list; k <<= 1)
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int t = threadIdx.x; t < n_list; t += kBlock) {
          const int u = t ^ j;
          if (u > t) {
            const uint32_t a = buf[t], c = buf[u];
            if ((a > c) == ((t & k) == 0)) {
              buf[t] = c;
              buf[u] = a;
            }
          }
        }
        __syncthreads();
      }
  }
  // the thread's words, in id order: every halo cell once
  const int per = (n_list + kBlock - 1) / kBlock;
  const int e0 = threadIdx.x * per, e1 = e0 + per < n_list ? e0 + per : n_list;
  auto each = [&](auto&& f) {
    for (int e = e0; e < e1; ++e) {
      if constexpr (MAP) {
        for (uint32_t m = buf[e]; m; m &= m - 1) f(32 * e + __ffs(m) - 1);
      } else {
        const uint32_t c = buf[e];
        if (c != ~0u && (e == 0 || buf[e - 1] != c)) f((int)c);
      }
    }
  };
  int mine = 0;
  each([&](int) { ++mine; });
  int ncells;
  int pos = block_scan<kBlock / 64>(mine, scan, ncells);
  if (ncells > kHaloCellsMax) return halo_none(info);
  int32_t* hs = ht.start + (int64_t)tile * kHaloCellsMax;
  int32_t* ho = ht.off + (int64_t)tile * (kHaloCellsMax + 1);
  each([&](int c) {
    hs[pos] = cell_start[c];
    cnt[pos] = cell_start[c + 1] - cell_start[c];
    ++pos;
  });
  __syncthreads();
  const int per2 = (ncells + kBlock - 1) / kBlock;
  const int k0 = threadIdx.x * per2;
  int sum = 0;
  for (int k = k0; k < k0 + per2 && k < ncells; ++k) sum += cnt[k];
  int natoms;
  int run = block_scan<kBlock / 64>(sum, scan, natoms);
  for (int k = k0; k < k0 + per2 && k < ncells; ++k) {
    ho[k] = run;
    run += cnt[k];
  }
  if (threadIdx.x == 0) {
    ho[ncells] = natoms;
    info[0] = ncells;
    info[1] = natoms;
    info[2] = natoms <= kHaloMax ? 1 : 0;
    info[3] = 0;
  }
}

// The cell sort and the tiles' halo tables, which need each other's results no more than the
// scatter's: workgroups [0, nsort) sort, the others build tables.
template <bool MAP>
__global__ void __launch_bounds__(kBlock)
k_sort_halo(int64_t N, CellGrid g, int nsort, const int32_t* __restrict__ start, int32_t* __restrict__ count,
            int32_t* __restrict__ key, int32_t* __restrict__ src, const double* __restrict__ x,
            const double* __restrict__ v, const int32_t* __restrict__ type, SortedState o, HaloTables ht,
            const int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  __shared__ union {
    int32_t kk[kSortWaves][kSortMax];
    HaloWork<MAP> halo;
  } sh;
  if ((int)blockIdx.x < nsort) {
    sort_cells(N, g.ncell, start, count, key, src, x, v, type, o, blockIdx.x, nsort, sh.kk);
    return;
  }
  const int ntiles = (int)((N + kBlock - 1) / kBlock);
  for (int tile = blockIdx.x - nsort; tile < ntiles; tile += gridDim.x - nsort) {
    halo_tile<MAP>(N, g, x, src, start, ht, tile, sh.halo);
    __syncthreads();  // the LDS tables are reused by the next tile
  }
}

// Halo-local index of sorted atom q, which must lie in the halo of ncells cells with first
// atoms hs and offsets ho.
__device__ __forceinline__ int halo_search(const int32_t* hs, const int32_t* ho, int ncells, int q) {
  int lo = 0, hi = ncells - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (hs[mid] <= q) lo = mid;
    else hi = mid - 1;
  }
  return ho[lo] + (q - hs[lo]);
}
// The same in tile `tile`.
__device__ __forceinline__ int halo_index(const HaloTables& ht, int tile, int ncells, int q) {
  return halo_search(ht.start + (int64_t)tile * kHaloCellsMax, ht.off + (int64_t)tile * (kHaloCellsMax + 1), ncells, q);
}

// Distance bin of a pair inside the list cutoff: the number of interior edges <= r^2,
// testing the first NE edges (the outer edge and the unused ones, set to infinity, are
// never reached; NE >= nbins - 1).
template <int NE>
__device__ __forceinline__ int bin_of(double r2, const BinEdges& be) {
  int k = 0;
#pragma unroll
  for (int m = 0; m < NE; ++m) k += r2 >= be.e2[m] ? 1 : 0;
  return k;
}
// Edge tests of the list build: one model's nine interior edges, or the union of two
// models' edges.
constexpr int kEdgesOne = 2 * kFracs - 1;
constexpr int kEdgesTwo = kMaxBins - 1;

// kMaxBins 16-bit counters packed in 64-bit registers: a counter update is a shift
// and a few selects and adds instead of a select chain over kMaxBins registers.
struct BinCounts {
  static constexpr int kWords = (kMaxBins + 3) / 4;
  uint64_t w[kWords] = {};
  __device__ __forceinline__ void add(int b) {
    const uint64_t inc = (uint64_t)1 << (16 * (b & 3));
#pragma unroll
    for (int k = 0; k < kWords; ++k) w[k] += (b >> 2) == k ? inc : 0;
  }
  __device__ __forceinline__ int get(int b) const {
    uint64_t v = w[0];
#pragma unroll
    for (int k = 1; k < kWords; ++k) v = (b >> 2) == k ? w[k] : v;
    return (int)((v >> (16 * (b & 3))) & 0xffffu);
  }
};

constexpr int kStage = 16;  // entries of a scratch segment

// The list entries of a cell's atoms: PARTS workgroups to a cell (one in large systems, more
// where one per cell would leave the chip idle). The positions of the stencil cells' atoms
// (27 cells; along a dimension of one or two cells, each cell once) are staged in LDS once,
// in stencil order and by sorted index inside a cell, and each wavefront takes the
// workgroup's atoms in turn, its 64 lanes testing two chunks of 64 candidates at a time
// (read together and without a branch, for the latency; cells away from the periodic
// boundary have a loop without the shifts). The accepted candidates are
// compacted (ballot and prefix count) into a per-wavefront LDS queue in candidate
// order; only those are binned and written, 64 entries per pass, to the atom's
// scratch column as q | bin << 28 with its halo-local index. Stencils larger than the staging
// (compressed boxes and dense clusters) are staged and tested part by part, in the same
// order, the length of each atom's column kept in cnt between the parts. Candidate vectors
// are x_q - x_p in FP64 plus the periodic shift of the stencil cell (-L, 0 or +L: what the
// minimum-image rule gives every pair that can lie within the cutoff when the dimension
// holds at least three cells), or the minimum-image rule itself in a dimension of fewer
// cells; r^2 = (dx*dx + dy*dy) + dz*dz without FMA.
//
// The staging holds kCellCand atoms, or as many as the stencil of a uniform box of this size
// with a margin of 15%, up to kCellCandMax: a cell edge is 7.0 to 7.6 A in large boxes, 750 to
// 1,000 stencil atoms at metallic densities, but up to 9.3 A where a side holds three cells.
// us for the kernel with that stencil staged / read from global memory: 1,372 atoms (8.4 A)
// 19 / 37, 5,324 (8.0 A) 30 / 72, 13,500 (7.7 A) 67 / 127, 27,436 (7.6 A) 93 / 215. With 2,048
// atoms staged whatever the box, two workgroups instead of four fit a compute unit (4,000
// atoms 34 us, 24 with 1,024). Past that, whole list builds in parts / with the stencil read
// from global memory: 30,000 random atoms at 0.24 A^-3 482 / 738, 122,880 1,654 / 2,663,
// 204,800 at 0.4 A^-3 4,923 / 7,676.
constexpr int kCellCand = 1024, kCellCandMax = 2048;
inline int cell_cand(int64_t N, const CellGrid& g) {
  double part = 1.0;  // of the box that a stencil covers
  for (int d = 0; d < 3; ++d) part *= g.nc[d] < 3 ? 1.0 : 3.0 / g.nc[d];
  const double want = 1.15 * part * (double)N;
  return want <= kCellCand ? kCellCand : (want >= kCellCandMax ? kCellCandMax : ((int)want + 63) & ~63);
}
// The staged candidates, one array after the other in the launch's LDS.
struct Cands {
  double *X, *Y, *Z;
  uint8_t* C;  // stencil cells
};
inline int cand_bytes(int cand) { return cand * (int)(3 * sizeof(double) + 1); }
constexpr int kCellQueue = 192;  // accepted candidates queued per wavefront (two chunks past a drain)

struct CellStage {
  int cq0[27], cum[28];
  double shift[3][27];
  union {
    struct {
      uint32_t qk[kBlock / 64][kCellQueue];
      double qr[kBlock / 64][kCellQueue];
    };
    int32_t halo[2][2][kHaloCellsMax];  // first atoms and offsets of two tiles' halo cells, before the queues are used
  };
  int loc0s[2][27];  // halo offset of each stencil cell for the cell's first two tiles
};

// Atoms s0 + first, s0 + first + step, ... of the cell [s0, s1), whose own stencil cell is
// `home`, against the staged candidates c0 .. c0 + nc - 1: all of the stencil, or (PART) a part
// of it, the last one or not.
template <int NE, bool PART, bool SHIFT, bool MINIMG>
__device__ void build_atoms(int64_t N, const CellGrid& g, const double* __restrict__ x, const BinEdges& be, int capR,
                            const ListOut& lo_, const HaloTables& ht, const ListScratch& sc,
                            int32_t* __restrict__ flags, CellStage& S, const Cands& P, int s0, int s1, int first, int step, int ns,
                            int home, int nc, int c0 = 0, bool last = true) {
#pragma clang fp contract(off)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile0 = s0 / kBlock;
  const double cut2 = be.e2[be.nbins - 1];
  uint32_t* scq = reinterpret_cast<uint32_t*>(sc.q);
  uint16_t* scl = reinterpret_cast<uint16_t*>(sc.l);
  int cached_tile = -1, hok = 0, hcells = 0, loc0 = 0;  // loc0: of stencil cell `lane`, for the atom's tile
  for (int p = s0 + first; p < s1; p += step) {  // wave-uniform
    const int tile = p / kBlock;
    if (tile != cached_tile) {
      cached_tile = tile;
      hcells = ht.info[4 * tile + 0];
      hok = ht.info[4 * tile + 2] != 0;
      loc0 = 0;
      if (tile - tile0 < 2) {
        if (lane < ns) loc0 = S.loc0s[tile - tile0][lane];
      } else if (hok && lane < ns && S.cum[lane + 1] > S.cum[lane]) {
        loc0 = halo_index(ht, tile, hcells, S.cq0[lane]) - S.cq0[lane];
      }
    }
    const int self_off = __shfl(loc0, home);
    if (lane == 0) lo_.selfl[p] = hok ? (uint16_t)(self_off + p) : kNoLocal;
    const int ks = S.cum[home] + (p - s0) - c0;  // the atom's own slot
    double xi, yi, zi;
    if constexpr (PART) {
      xi = x[p];
      yi = x[N + p];
      zi = x[2 * N + p];
    } else {
      xi = P.X[ks];
      yi = P.Y[ks];
      zi = P.Z[ks];
    }
    int nw = PART && c0 > 0 ? lo_.cnt[p] : 0, nq = 0;  // entries written, entries queued (wave-uniform)
    auto drain = [&]() {
      wave_lds_sync();
      for (int j0 = 0; j0 < nq; j0 += 64) {
        const int j = j0 + lane;
        const bool v = j < nq;
        const int k = v ? (int)S.qk[w][j] : 0;
        const int sidx = P.C[k];
        const int lc = __shfl(loc0, sidx);
        const int e = nw + j;
        if (v && e < capR) {
          const int q = S.cq0[sidx] + (c0 + k - S.cum[sidx]);
          const int64_t o = ((int64_t)(e / kStage) * N + p) * kStage + e % kStage;
          scq[o] = (uint32_t)q | ((uint32_t)bin_of<NE>(S.qr[w][j], be) << 28);
          scl[o] = hok ? (uint16_t)(lc + q) : kNoLocal;
        }
      }
      nw += nq;
      nq = 0;
      wave_lds_sync();
    };
    auto dist2 = [&](int k) {
      double dx = P.X[k] - xi, dy = P.Y[k] - yi, dz = P.Z[k] - zi;
      if constexpr (SHIFT) {
        const int sidx = P.C[k];
        if constexpr (MINIMG) {
          dx = g.nc[0] < 3 ? min_image(dx, g.box[0]) : dx + S.shift[0][sidx];
          dy = g.nc[1] < 3 ? min_image(dy, g.box[1]) : dy + S.shift[1][sidx];
          dz = g.nc[2] < 3 ? min_image(dz, g.box[2]) : dz + S.shift[2][sidx];
        } else {
          dx = dx + S.shift[0][sidx];
          dy = dy + S.shift[1][sidx];
          dz = dz + S.shift[2][sidx];
        }
      }
      const double sxx = dx * dx;
      const double syy = dy * dy;
      const double szz = dz * dz;
      const double sxy = sxx + syy;
      return sxy + szz;
    };
    // appends the accepted candidates of one 64-candidate chunk, in candidate order
    auto enqueue = [&](int k, bool acc, double r2) {
      const uint64_t m = __ballot(acc);
      const int pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
      if (acc) {
        S.qk[w][nq + pre] = (uint32_t)k;
        S.qr[w][nq + pre] = r2;
      }
      nq += __popcll(m);
    };
    // two chunks per pass, their staged positions read together
    for (int k0 = 0; k0 < nc; k0 += 128) {
      const int ka = k0 + lane, kb = k0 + 64 + lane;
      const int kn = PART ? 0 : ks;  // a slot for the lanes past the last one
      const double ra = dist2(ka < nc ? ka : kn), rb = dist2(kb < nc ? kb : kn);
      enqueue(ka, ra < cut2 && ka < nc && ka != ks, ra);
      enqueue(kb, rb < cut2 && kb < nc && kb != ks, rb);
      if (nq > kCellQueue - 128) drain();
    }
    drain();
    if (lane == 0) {
      lo_.cnt[p] = !last || nw < capR ? nw : capR;
      if (last && nw > capR) {
        atomicMax(&flags[FLAG_OVF_R], nw);
        if (lo_.alarm) lo_.alarm[FLAG_OVF_R] = 1;
      }
    }
  }
}

template <int NE, bool MINIMG>
__device__ void build_cell(int64_t N, const CellGrid& g, const double* __restrict__ x,
                           const int32_t* __restrict__ start, const BinEdges& be, int capR, const ListOut& lo_,
                           const HaloTables& ht, const ListScratch& sc, int32_t* __restrict__ flags, int c, int part,
                           int parts, CellStage& S, const Cands& P, int cand) {
  const int s0 = start[c], s1 = start[c + 1];
  constexpr int W = kBlock / 64;
  if (s0 + part * W >= s1) return;  // empty cell, brick slot outside the grid, or no atom left for this part
  int cx, cy, cz;
  cell_coords(g, c, cx, cy, cz);
  const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tile0 = s0 / kBlock;
  // stencil cells t = (a n1 + b) n0 + e: along a dimension of at least three cells the
  // offsets -1, 0, 1, otherwise every cell once, starting with the cell's own
  const int n0 = !MINIMG || g.nc[0] >= 3 ? 3 : g.nc[0], n1 = !MINIMG || g.nc[1] >= 3 ? 3 : g.nc[1],
            n2 = !MINIMG || g.nc[2] >= 3 ? 3 : g.nc[2];
  const int o0 = n0 == 3 ? 1 : 0, o1 = n1 == 3 ? 1 : 0, o2 = n2 == 3 ? 1 : 0;
  const int ns = n0 * n1 * n2;
  const int home = (o2 * n1 + o1) * n0 + o0;
  int n_s = 0;
  if (t < ns) {
    const int r3[3] = {cx + t % n0 - o0, cy + (t / n0) % n1 - o1, cz + t / (n0 * n1) - o2};
    int w3[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      w3[d] = (r3[d] + g.nc[d]) % g.nc[d];
      S.shift[d][t] = r3[d] < 0 ? -g.box[d] : (r3[d] >= g.nc[d] ? g.box[d] : 0.0);
    }
    const int cc = cell_lin(g, w3[0], w3[1], w3[2]);
    const int q0 = start[cc];
    n_s = start[cc + 1] - q0;
    S.cq0[t] = q0;
  }
  // the halo tables of the tile of the cell's first atom and of the next tile if it holds
  // atoms of the cell (other tiles, for cells of more than 256 atoms, are searched in global
  // memory when reached)
  int hn[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int tl = tile0 + u;
    hn[u] = tl * kBlock < s1 && ht.info[4 * tl + 2] != 0 ? ht.info[4 * tl] : 0;
    for (int k = t; k < hn[u]; k += kBlock) {
      S.halo[u][0][k] = ht.start[(int64_t)tl * kHaloCellsMax + k];
      S.halo[u][1][k] = ht.off[(int64_t)tl * (kHaloCellsMax + 1) + k];
    }
  }
  if (w == 0) {  // exclusive prefix of the stencil cells' counts
    const int incl = wave_scan(n_s);
    if (t < ns) S.cum[t] = incl - n_s;
    if (t == ns - 1) S.cum[ns] = incl;
  }
  __syncthreads();
  const int nc = S.cum[ns];
  // halo-local offset of each stencil cell in the two tiles
  if (t >= 64 && t < 64 + 2 * ns) {
    const int u = (t - 64) / ns, sc0 = (t - 64) % ns;
    int v = 0;
    if (hn[u] > 0 && S.cum[sc0 + 1] > S.cum[sc0])
      v = halo_search(S.halo[u][0], S.halo[u][1], hn[u], S.cq0[sc0]) - S.cq0[sc0];
    S.loc0s[u][sc0] = v;
  }
  // a cell away from the periodic boundary has no image shifts
  const bool shifted = cx == 0 || cy == 0 || cz == 0 || cx == g.nc[0] - 1 || cy == g.nc[1] - 1 ||
                       cz == g.nc[2] - 1;
  const int first = part * W + w, step = parts * W;
  auto stage = [&](int c0, int n) {
    for (int k = t; k < n; k += kBlock) {
      int sidx = 0;
#pragma unroll
      for (int m = 1; m < 27; ++m) sidx += m < ns && c0 + k >= S.cum[m] ? 1 : 0;
      const int q = S.cq0[sidx] + (c0 + k - S.cum[sidx]);
      P.X[k] = x[q];
      P.Y[k] = x[N + q];
      P.Z[k] = x[2 * N + q];
      P.C[k] = (uint8_t)sidx;
    }
    __syncthreads();
  };
  if (nc <= cand) {
    stage(0, nc);
    if (MINIMG || shifted)
      build_atoms<NE, false, true, MINIMG>(N, g, x, be, capR, lo_, ht, sc, flags, S, P, s0, s1, first, step, ns, home, nc);
    else
      build_atoms<NE, false, false, MINIMG>(N, g, x, be, capR, lo_, ht, sc, flags, S, P, s0, s1, first, step, ns, home, nc);
    return;
  }
  for (int c0 = 0; c0 < nc; c0 += cand) {
    const int n = nc - c0 < cand ? nc - c0 : cand;
    if (c0 > 0) __syncthreads();  // the part before is read no more
    stage(c0, n);
    build_atoms<NE, true, true, MINIMG>(N, g, x, be, capR, lo_, ht, sc, flags, S, P, s0, s1, first, step, ns, home, n, c0,
                                        c0 + n == nc);
  }
}

// Primary state from the sorted one (workgroups [0, ncopy)), and the cells' lists from the
// positions at the build, which the copy does not touch (the others).
struct PrimaryState {
  double *x, *v;
  int32_t *type, *perm;
  uint4* pos;
};
__device__ void copy_back(int64_t N, const CellGrid& g, const SortedState& o, const PrimaryState& s, int block,
                          int nblocks) {
  for (int64_t p = (int64_t)block * kBlock + threadIdx.x; p < N; p += (int64_t)nblocks * kBlock) {
    double xn[3];
    for (int c = 0; c < 3; ++c) {
      xn[c] = o.x2[c * N + p];
      s.x[c * N + p] = xn[c];
      s.v[c * N + p] = o.v2[c * N + p];
    }
    const int32_t tp = o.type2[p];
    pos_put(s.pos, p, xn[0], xn[1], xn[2], tp, g.box);
    s.type[p] = tp;
    s.perm[p] = o.perm2[p];
  }
}

template <int NE, bool MINIMG>
__global__ void __launch_bounds__(kBlock)
k_build_cells(int64_t N, CellGrid g, SortedState o, PrimaryState prim, int ncopy, const int32_t* __restrict__ start,
              BinEdges be, int capR, ListOut lo_, HaloTables ht, ListScratch sc, int parts, int cand,
              int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  __shared__ CellStage S;
  extern __shared__ double cands[];
  const Cands P{cands, cands + cand, cands + 2 * cand, reinterpret_cast<uint8_t*>(cands + 3 * cand)};
  if ((int)blockIdx.x < ncopy) return copy_back(N, g, o, prim, blockIdx.x, ncopy);
  const double* __restrict__ x = o.xb;
  const int n = g.ncell * parts;
  for (int cb = blockIdx.x - ncopy; cb < n; cb += gridDim.x - ncopy) {
    const int u = xcd_tile(cb, n);
    build_cell<NE, MINIMG>(N, g, x, start, be, capR, lo_, ht, sc, flags, u / parts, u % parts, parts, S, P, cand);
    __syncthreads();  // the LDS staging is reused by the next cell
  }
}

// Workgroups to a cell: as many as fill the chip's 256 compute units once, four to a unit
// (what the staging's LDS allows), up to one atom per wavefront of a 32-atom cell; every
// workgroup of a cell stages the whole stencil. us with 1 / 2 / 4 / 8 of them:
//   8 cells (256 atoms)     28 19 14 12      512 (16,384)   48 38 45 55
//   216 (4,000)             43 27 23 26    1,000 (32,000)   62 65 76 95
inline int build_parts(int ncell) {
  const int p = 1024 / ncell;
  return p < 1 ? 1 : (p > 8 ? 8 : p);
}

// One wavefront per 64 / PARTS atoms, PARTS lanes per atom: counts each atom's scratch
// entries per bin, writes the bin breakpoints, and orders the entries by bin (stable
// inside a bin), writing the list and its halo-local indices row by row, 64 / PARTS
// consecutive atoms (64 or 16 bytes) per store, through LDS tiles of kPlaceRows rows;
// longer lists take further rounds. Lane h counts and places entries [PLEN h, PLEN (h + 1))
// (the last lane the rest), starting each bin after the entries of earlier parts.
// Entries outside the current round go to a spare row. Four lanes with 32 entries each write
// whole 64-byte rows; where the chip is not full (place_parts) 16 lanes with 16 entries each
// shorten the serial chain of counts and positions.
constexpr int kPlaceRows = 159;  // one round for lists up to 159 entries (FCC metals at 7 A: ~135-150)
constexpr int kPlaceGrid = 16384;  // workgroups of the placement (grid-stride over atom groups)

template <int PARTS>
__global__ void __launch_bounds__(64)
k_place_lists(int64_t N, int nbins, int binA, int capR, int capA, ListOut lo_, ListScratch sc,
              int32_t* __restrict__ flags) {
  if (flags[FLAG_REBUILD] == 0) return;
  constexpr int kPlaceAtoms = 64 / PARTS, PLEN = PARTS == 4 ? 32 : 16;
  __shared__ uint32_t tile[(kPlaceRows + 1) * kPlaceAtoms];
  __shared__ uint16_t ltile[(kPlaceRows + 1) * kPlaceAtoms];
  __shared__ uint16_t off[kMaxBins * 64];  // next position of each bin, per lane
  __shared__ uint64_t parts[PARTS][BinCounts::kWords][kPlaceAtoms];  // per-bin counts of each part
  const int lane = threadIdx.x;
  const int a = lane % kPlaceAtoms;  // atom of the wavefront
  const int h = lane / kPlaceAtoms;  // which part of its column
  // groups of kPlaceAtoms atoms, strided over a capped grid: a step without a rebuild
  // then dispatches few workgroups
  const int64_t ngroups = (N + kPlaceAtoms - 1) / kPlaceAtoms;
  // the list length of the lane's atom in the next group is loaded one group ahead
  int cnt_next = (int64_t)blockIdx.x * kPlaceAtoms + a < N ? lo_.cnt[(int64_t)blockIdx.x * kPlaceAtoms + a] : 0;
  for (int64_t grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const int64_t p = grp * kPlaceAtoms + a;
    const bool valid = p < N;
    const int cnt = valid ? cnt_next : 0;
    {
      const int64_t pn = (grp + gridDim.x) * kPlaceAtoms + a;
      cnt_next = grp + gridDim.x < ngroups && pn < N ? lo_.cnt[pn] : 0;
    }
    const int g_lo = h * PLEN;
    const int g_hi = h == PARTS - 1 ? cnt : (g_lo + PLEN < cnt ? g_lo + PLEN : cnt);
    const bool work = valid && g_lo < cnt;
    // longest list of the wavefront (uniform loop bounds for the row writes)
    int rows_max = cnt;
  #pragma unroll
    for (int o = 32; o > 0; o >>= 1) rows_max = max(rows_max, __shfl_xor(rows_max, o, 64));
    // per-bin counts of this lane's part (16-bit fields), then of the parts before it
    // and of the whole list
    // this lane's part of the scratch column: the first two 16-entry chunks stay in
    // registers from the counting pass to the placement (parts hold 32 entries, the last
    // part the rest), later chunks are read again
    auto load_q = [&](int g, uint32_t* v) {
      const uint4* src = sc.q + ((int64_t)(g / kStage) * N + p) * (kStage / 4);
  #pragma unroll
      for (int j = 0; j < kStage / 4; ++j) {
        const uint4 w = src[j];
        v[4 * j] = w.x;
        v[4 * j + 1] = w.y;
        v[4 * j + 2] = w.z;
        v[4 * j + 3] = w.w;
      }
    };
    // the halo indices of a chunk, 16-bit, as two 16-byte words
    auto load_l = [&](int g, uint4* lw) {
      const uint4* ls = sc.l + ((int64_t)(g / kStage) * N + p) * (kStage / 8);
  #pragma unroll
      for (int j = 0; j < kStage / 8; ++j) lw[j] = ls[j];
    };
    BinCounts mine;
    auto count_chunk = [&](int g, const uint32_t* v) {
  #pragma unroll
      for (int u = 0; u < kStage; ++u)
        if (g + u < g_hi) mine.add((int)(v[u] >> 28));
    };
    uint32_t c0[kStage], c1[kStage];
    uint4 l0[kStage / 8], l1[kStage / 8];  // their halo indices, loaded with them
    const bool two = PLEN > kStage && work && g_lo + kStage < g_hi;
    if (work) {
      load_q(g_lo, c0);
      load_l(g_lo, l0);
      if (two) {
        load_q(g_lo + kStage, c1);
        load_l(g_lo + kStage, l1);
      }
      count_chunk(g_lo, c0);
      if (two) count_chunk(g_lo + kStage, c1);
      for (int g = g_lo + PLEN; g < g_hi; g += kStage) {
        uint32_t t[kStage];
        load_q(g, t);
        count_chunk(g, t);
      }
    }
  #pragma unroll
    for (int k = 0; k < BinCounts::kWords; ++k) parts[h][k][a] = mine.w[k];
    __syncthreads();
    BinCounts before, total;
  #pragma unroll
    for (int q = 0; q < PARTS; ++q)
  #pragma unroll
      for (int k = 0; k < BinCounts::kWords; ++k) {
        const uint64_t c = parts[q][k][a];
        total.w[k] += c;
        before.w[k] += q < h ? c : 0;
      }
    // bin breakpoints (cumulative counts); angular candidates are the bins up to binA
    int bstart[kMaxBins];
    {
      int t = 0;
  #pragma unroll
      for (int k = 0; k < kMaxBins; ++k) {
        bstart[k] = t;
        t += k < nbins ? total.get(k) : 0;
        if (valid && h == 0 && k < nbins) lo_.bp[(int64_t)k * N + p] = t < capR ? t : capR;
        if (valid && h == 0 && k == binA && t > capA) {
          atomicMax(&flags[FLAG_OVF_A], t);
          if (lo_.alarm) lo_.alarm[FLAG_OVF_A] = 1;
        }
      }
    }
    constexpr int rows = kPlaceRows;  // row `rows` of the tiles is the spare row
    for (int r0 = 0; r0 < rows_max; r0 += rows) {
      if (work) {
  #pragma unroll
        for (int k = 0; k < kMaxBins; ++k) off[k * 64 + lane] = (uint16_t)(bstart[k] + before.get(k));
        auto place_chunk = [&](int g, const uint32_t* v, const uint4* lw) {
          uint32_t hl[kStage];
  #pragma unroll
          for (int j = 0; j < kStage / 8; ++j) {
            const uint4 w = lw[j];
            const uint32_t t[4] = {w.x, w.y, w.z, w.w};
  #pragma unroll
            for (int u = 0; u < 4; ++u) {
              hl[8 * j + 2 * u] = t[u] & 0xffffu;
              hl[8 * j + 2 * u + 1] = t[u] >> 16;
            }
          }
  #pragma unroll
          for (int u = 0; u < kStage; ++u) {
            const bool live = g + u < g_hi;
            const int oi = (int)(v[u] >> 28) * 64 + lane;
            int pos = -1;
            if (live) {
              pos = off[oi];
              off[oi] = (uint16_t)(pos + 1);
            }
            pos -= r0;
            const int slot = (live && pos >= 0 && pos < rows ? pos : rows) * kPlaceAtoms + a;
            tile[slot] = v[u] & 0x0fffffffu;
            ltile[slot] = (uint16_t)hl[u];
          }
        };
        place_chunk(g_lo, c0, l0);
        if (two) place_chunk(g_lo + kStage, c1, l1);
        for (int g = g_lo + PLEN; g < g_hi; g += kStage) {
          uint32_t t[kStage];
          uint4 lt[kStage / 8];
          load_q(g, t);
          load_l(g, lt);
          place_chunk(g, t, lt);
        }
      }
      __syncthreads();
      // the PARTS lane groups write interleaved rows
      const int nrow = rows_max - r0 < rows ? rows_max - r0 : rows;
      for (int r = h; r < nrow; r += PARTS) {
        if (valid && r0 + r < cnt) {
          lo_.nbr[(int64_t)(r0 + r) * N + p] = (int32_t)tile[r * kPlaceAtoms + a];
          lo_.nbrl[(int64_t)(r0 + r) * N + p] = ltile[r * kPlaceAtoms + a];
        }
      }
      __syncthreads();
    }
    __syncthreads();  // the LDS tiles are reused by the next group
  }
}

// Lists in original ids, one row per original atom, ascending.
__global__ void k_export(int64_t N, const int32_t* __restrict__ perm, const int32_t* __restrict__ nbr,
                         const int32_t* __restrict__ cnt, int cap, int32_t* __restrict__ rows,
                         int32_t* __restrict__ row_cnt) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const int64_t o = perm[p];
  const int n = cnt[p] < cap ? cnt[p] : cap;
  int32_t* row = rows + o * cap;
  for (int k = 0; k < n; ++k) {
    const int32_t val = perm[nbr[(int64_t)k * N + p]];
    int j = k - 1;
    while (j >= 0 && row[j] > val) {
      row[j + 1] = row[j];
      --j;
    }
    row[j + 1] = val;
  }
  row_cnt[o] = n;
}

}  // namespace

hipError_t launch_clear(int32_t* flags, int32_t* cells, int ncell, int32_t* nbr, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_clear, dim3(grid_blocks(n > 0 ? n : 1)), dim3(kBlock), 0, st, flags, cells, ncell, nbr, n);
  return hipGetLastError();
}

// Lanes per atom in the placement; us with 4 / 16: 256 atoms 15 / 9, 4,000 16 / 13,
// 16,384 21 / 27, 32,000 23 / 47.
inline int place_parts(int64_t N) { return N <= 8192 ? 16 : 4; }

// The rebuild decision (see RebuildRule) from nd2 partial displacement maxima, then the
// rebuild: every kernel after the decision returns at once when flags[FLAG_REBUILD] == 0,
// so the whole rebuild can be enqueued each step and skipped on the device without a host
// sync.
hipError_t launch_rebuild(const RebuildRule& rule, const double* d2, int nd2, int64_t N, const CellGrid& g, int capR,
                          int capA, double* x, double* v, int32_t* type, int32_t* perm, double* x_alt, double* v_alt,
                          int32_t* type_alt, int32_t* perm_alt, double* x_build, int32_t* cellid,
                          int32_t* src, int32_t* key, int32_t* rank, int32_t* cell_count,
                          int32_t* cell_start, int32_t* scan_tmp, uint4* pos, const ListOut& lout, HaloTables ht,
                          ListScratch sc, int32_t* flags, hipStream_t st) {
  const int nb = grid_blocks(N);
  const int ncell = g.ncell;
  const BinEdges& be = rule.be;
  const dim3 gb(rebuild_grid(nb)), kb(kBlock);
  if (N <= kSortAtoms && ncell <= kSortCells) {
    hipLaunchKernelGGL(k_select_sort, dim3(1), dim3(kSelBlock), 0, st, rule, d2, nd2, N, g, x, perm, cell_start, src,
                       key, flags);
  } else {
    if (nd2 <= kDecideMax) {
      hipLaunchKernelGGL(k_bin<true>, gb, kb, 0, st, rule, d2, nd2, N, g, x, cellid, rank, cell_count, flags);
    } else {
      hipLaunchKernelGGL(k_select, dim3(1), dim3(kSelBlock), 0, st, rule, d2, nd2, flags);
      hipLaunchKernelGGL(k_bin<false>, gb, kb, 0, st, rule, d2, nd2, N, g, x, cellid, rank, cell_count, flags);
    }
    if (ncell <= kScanCells) {
      hipLaunchKernelGGL(k_scan_scatter, gb, kb, 0, st, N, ncell, cell_count, cellid, rank, perm, cell_start, src,
                         key, flags);
    } else {
      const int ntiles = (ncell + kScanTile - 1) / kScanTile;
      hipLaunchKernelGGL(k_scan_tiles, dim3(ntiles), kb, 0, st, cell_count, cell_start, ncell, scan_tmp, flags);
      hipLaunchKernelGGL(k_scan_add, dim3(ntiles), dim3(kScanTile), 0, st, cell_start, ncell, N, scan_tmp, flags);
      hipLaunchKernelGGL(k_scatter, gb, kb, 0, st, N, cellid, rank, cell_start, perm, src, key, flags);
    }
  }
  const SortedState sorted{x_alt, v_alt, x_build, type_alt, perm_alt};
  const PrimaryState prim{x, v, type, perm, pos};
  const int nsort = rebuild_grid(grid_blocks(ncell, kSortWaves));
  auto sort_halo = ncell <= kMapCells ? k_sort_halo<true> : k_sort_halo<false>;
  hipLaunchKernelGGL(sort_halo, dim3(nsort + rebuild_grid(nb)), kb, 0, st, N, g, nsort, cell_start, cell_count, key,
                     src, x, v, type, sorted, ht, flags);
  // the minimum-image rule inside the candidate loop only for boxes with fewer than
  // three cells along some dimension
  const bool small = g.nc[0] < 3 || g.nc[1] < 3 || g.nc[2] < 3;
  const bool one = be.nbins - 1 <= kEdgesOne;
  const int parts = build_parts(ncell);
  const int ncopy = nb < kCopyGrid ? nb : kCopyGrid;
  auto cells = small ? (one ? k_build_cells<kEdgesOne, true> : k_build_cells<kEdgesTwo, true>)
                     : (one ? k_build_cells<kEdgesOne, false> : k_build_cells<kEdgesTwo, false>);
  const int cand = cell_cand(N, g);
  hipLaunchKernelGGL(cells, dim3(ncopy + rebuild_grid((int64_t)ncell * parts)), kb, cand_bytes(cand), st, N, g, sorted,
                     prim, ncopy, cell_start, be, capR, lout, ht, sc, parts, cand, flags);
  const int pp = place_parts(N);
  const int place_groups = grid_blocks(N, 64 / pp);
  hipLaunchKernelGGL(pp == 16 ? k_place_lists<16> : k_place_lists<4>,
                     dim3(place_groups < kPlaceGrid ? place_groups : kPlaceGrid), dim3(64), 0, st, N, be.nbins,
                     be.idxA[0][kFracs - 1], capR, capA, lout, sc, flags);
  return hipGetLastError();
}

hipError_t launch_export(int64_t N, const int32_t* perm, const int32_t* nbr, const int32_t* cnt,
                         int cap, int32_t* rows, int32_t* row_cnt, hipStream_t st) {
  hipLaunchKernelGGL(k_export, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, perm, nbr, cnt, cap, rows, row_cnt);
  return hipGetLastError();
}

}  // namespace nep
