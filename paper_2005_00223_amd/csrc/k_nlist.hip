// Neighbour-list kernels: periodic wrap, per-type row ordering, cell list,
// skin candidate list and the formatted list of Section V-B (type-sorted,
// distance-sorted with index tie-break, nearest sel per type kept, -1
// padded).  The distance of every pair is the IEEE result of
//   d = x_j - x_i (one minimum-image correction), r = sqrt((dx dx + dy dy) + dz dz)
// in exactly this order; this file is compiled with -ffp-contract=off so no
// multiply-add is fused and the list is reproducible bit for bit.
//
// The paper packs (type, floor(|r| 1e8), j) into one 64-bit decimal key
// before sorting.  Here the same lexicographic order is bit-packed:
// type in bits 58..63, floor(r 1e8) in bits 26..57, j in bits 0..25, which
// bounds rc < 42.9 A and n < 2^26 (checked by the host).
#include <cmath>

#include "dp_internal.h"

namespace dpk {

__device__ inline double wrap1(double x, double L) {
  double y = x - L * floor(x / L);
  if (y >= L) y = 0.0;
  return y;
}

__device__ inline double min_image(double v, double L) {
  // v - L, v or v + L: selects, not branches, and the sign from v's own
  return fabs(v) > 0.5 * L ? v - copysign(L, v) : v;
}
__device__ inline float min_image(float v, float L) { return fabsf(v) > 0.5f * L ? v - copysignf(L, v) : v; }

__global__ void k_wrap(int64_t n, const double *__restrict__ x, const int32_t *__restrict__ types, int ntypes,
                       double L0, double L1, double L2, double4 *__restrict__ xw, uint32_t *flags) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int t = types[i];
  if (t < 0 || t >= ntypes) {
    atomicOr(flags, FLAG_BAD_TYPE);
    t = 0;
  }
  double4 o;
  o.x = wrap1(x[3 * i + 0], L0);
  o.y = wrap1(x[3 * i + 1], L1);
  o.z = wrap1(x[3 * i + 2], L2);
  o.w = (double)t;
  xw[i] = o;
}

void launch_wrap(hipStream_t s, int64_t n, const double *coords, const int32_t *types, int ntypes, const double *L,
                 double4 *xw, uint32_t *flags) {
  if (n <= 0) return;
  int bs = 256;
  hipLaunchKernelGGL(k_wrap, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, s, n, coords, types, ntypes, L[0],
                     L[1], L[2], xw, flags);
}

// ---------------------------------------------------------------------------
// per-type row order: atoms of type t occupy rows type_start[t] + rank, with
// rank the index order inside the type and each type's block padded to
// ROW_TILE rows (padding rows have atom_of_pos = -1).
// ---------------------------------------------------------------------------
constexpr int TS_BLOCK = 256;

// mask (may be NULL): only atoms with mask[i] != 0 get rows
__global__ void k_type_count(int64_t n, const double4 *__restrict__ xw, int ntypes, int32_t *blk_counts,
                             const int32_t *mask) {
  __shared__ int32_t c[MAXT];
  if (threadIdx.x < MAXT) c[threadIdx.x] = 0;
  __syncthreads();
  int64_t i = (int64_t)blockIdx.x * TS_BLOCK + threadIdx.x;
  if (i < n && (!mask || mask[i])) atomicAdd(&c[(int)xw[i].w], 1);
  __syncthreads();
  if (threadIdx.x < ntypes) blk_counts[(int64_t)blockIdx.x * MAXT + threadIdx.x] = c[threadIdx.x];
}

// single block, one wave per type: exclusive scan of block counts per type, 64
// blocks at a time (one lane walking them: 19 us at 32,000 atoms, 254 at
// 500,000), padded type starts
__global__ void __launch_bounds__(64 * MAXT) k_type_scan(int nblk, int ntypes, int32_t *blk_counts,
                                                         int32_t *type_count, int32_t *type_start) {
  __shared__ int32_t tot[MAXT];
  const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (t < ntypes) {
    int32_t run = 0;
    int32_t next = lane < nblk ? blk_counts[(int64_t)lane * MAXT + t] : 0;
    for (int b = lane; b - lane < nblk; b += 64) {
      const int32_t v = next;
      next = b + 64 < nblk ? blk_counts[(int64_t)(b + 64) * MAXT + t] : 0;
      int32_t x = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
      }
      if (b < nblk) blk_counts[(int64_t)b * MAXT + t] = run + x - v;
      run += __shfl(x, 63);
    }
    if (lane == 0) {
      tot[t] = run;
      type_count[t] = run;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t s = 0;
    for (int u = 0; u < ntypes; ++u) {
      type_start[u] = s;
      s += (tot[u] + ROW_TILE - 1) / ROW_TILE * ROW_TILE;
    }
    type_start[ntypes] = s;
  }
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_type_place(int64_t n, const double4 *__restrict__ xw, int ntypes, const int32_t *blk_off,
                             const int32_t *type_start, int32_t *pos_of_atom, int32_t *atom_of_pos,
                             const int32_t *mask) {
  __shared__ int32_t wtot[TS_BLOCK / 64][MAXT];
  int64_t i = (int64_t)blockIdx.x * TS_BLOCK + threadIdx.x;
  int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int t = (i < n && (!mask || mask[i])) ? (int)xw[i].w : -1;
  int myrank = 0;
  for (int u = 0; u < ntypes; ++u) {
    unsigned long long m = __ballot(t == u);
    if (lane == 0) wtot[wv][u] = __popcll(m);
    if (t == u) myrank = __popcll(m & ((1ull << lane) - 1ull));
  }
  __syncthreads();
  if (t >= 0) {
    for (int w = 0; w < wv; ++w) myrank += wtot[w][t];
    int32_t pos = type_start[t] + blk_off[(int64_t)blockIdx.x * MAXT + t] + myrank;
    if (pos_of_atom) pos_of_atom[i] = pos;
    atom_of_pos[pos] = (int32_t)i;
  }
}

void launch_type_sort(hipStream_t s, int64_t n, const double4 *xw, int ntypes, int32_t *blk_counts,
                      int32_t *type_count, int32_t *type_start, int32_t *pos_of_atom, int32_t *atom_of_pos,
                      int64_t rows_cap, const int32_t *mask) {
  int nblk = (int)((n + TS_BLOCK - 1) / TS_BLOCK);
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((rows_cap + 255) / 256)), dim3(256), 0, s, atom_of_pos, rows_cap,
                     -1);
  if (n <= 0) {
    hipLaunchKernelGGL(k_type_scan, dim3(1), dim3(64 * ntypes), 0, s, 0, ntypes, blk_counts, type_count, type_start);
    return;
  }
  hipLaunchKernelGGL(k_type_count, dim3(nblk), dim3(TS_BLOCK), 0, s, n, xw, ntypes, blk_counts, mask);
  hipLaunchKernelGGL(k_type_scan, dim3(1), dim3(64 * ntypes), 0, s, nblk, ntypes, blk_counts, type_count, type_start);
  hipLaunchKernelGGL(k_type_place, dim3(nblk), dim3(TS_BLOCK), 0, s, n, xw, ntypes, blk_counts, type_start,
                     pos_of_atom, atom_of_pos, mask);
}

// ---------------------------------------------------------------------------
// cell list: side >= rlist, counting sort by cell (order inside a cell is
// irrelevant: the formatted list is sorted by key afterwards)
// ---------------------------------------------------------------------------
__device__ inline int cell_coord(double x, double side, int nc) {
  int c = (int)floor(x / side);
  if (c >= nc) c = nc - 1;
  if (c < 0) c = 0;
  return c;
}

__device__ inline bool skip_build(const uint32_t *cond) { return cond && !(*cond & FLAG_REBUILD); }

__global__ void k_fill_cond(int32_t *p, int64_t n, int32_t v, const uint32_t *cond) {
  if (skip_build(cond)) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_cell_assign(int64_t n, const double4 *__restrict__ xw, CellGrid g, int32_t *cell_of,
                              int32_t *cell_count, const uint32_t *cond) {
  if (skip_build(cond)) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double4 p = xw[i];
  int cx = cell_coord(p.x, g.side[0], g.nc[0]);
  int cy = cell_coord(p.y, g.side[1], g.nc[1]);
  int cz = cell_coord(p.z, g.side[2], g.nc[2]);
  int c = (cx * g.nc[1] + cy) * g.nc[2] + cz;
  cell_of[i] = c;
  atomicAdd(&cell_count[c], 1);
}

// single-block exclusive scan of m int32 values: out[0..m] (out[m] = total)
__global__ void __launch_bounds__(1024) k_scan_single(const int32_t *in, int64_t m, int32_t *out,
                                                      const uint32_t *cond) {
  if (skip_build(cond)) return;
  __shared__ int32_t wsum[16];
  __shared__ int32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int64_t base = 0; base < m; base += 1024) {
    int64_t i = base + threadIdx.x;
    int32_t v = (i < m) ? in[i] : 0;
    int32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
      int32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    int32_t woff = 0;
    for (int w = 0; w < wv; ++w) woff += wsum[w];
    int32_t c0 = carry;
    if (i < m) out[i] = c0 + woff + x - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry = c0 + woff + x;
    __syncthreads();
  }
  if (threadIdx.x == 0) out[m] = carry;
}

// code[i] = cx << 24 | cy << 16 | cz << 8 | min(index inside the cell, 255)
// (cell coordinates modulo 256; used only with at most 255 cells per axis)
// xs: position in FP32 and index of the atoms in cell order
__global__ void k_cell_fill(int64_t n, const double4 *__restrict__ xw, CellGrid g, const int32_t *cell_of,
                            const int32_t *cell_start, int32_t *cell_fill, int32_t *cell_atoms, uint32_t *code,
                            CellPos *__restrict__ xs, const uint32_t *cond) {
  if (skip_build(cond)) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int c = cell_of[i];
  int p = atomicAdd(&cell_fill[c], 1);
  const int q = cell_start[c] + p;
  cell_atoms[q] = (int32_t)i;
  const double4 x = xw[i];
  xs[q] = CellPos{(float)x.x, (float)x.y, (float)x.z, (int32_t)i};
  if (code) {
    const int cz = c % g.nc[2], cy = (c / g.nc[2]) % g.nc[1], cx = c / (g.nc[1] * g.nc[2]);
    code[i] = ((uint32_t)(cx & 255) << 24) | ((uint32_t)(cy & 255) << 16) | ((uint32_t)(cz & 255) << 8) |
              (uint32_t)(p < 255 ? p : 255);
  }
}

void launch_cells(hipStream_t s, int64_t n, const double4 *xw, const CellGrid &g, int32_t *cell_of,
                  int32_t *cell_start, int32_t *cell_fill, int32_t *cell_atoms, uint32_t *cell_code,
                  CellPos *xs, int32_t *scan_tmp, const uint32_t *cond) {
  int64_t ncell = (int64_t)g.nc[0] * g.nc[1] * g.nc[2];
  unsigned gc = (unsigned)((ncell + 255) / 256);
  hipLaunchKernelGGL(k_fill_cond, dim3(gc), dim3(256), 0, s, scan_tmp, ncell, 0, cond);
  hipLaunchKernelGGL(k_fill_cond, dim3(gc), dim3(256), 0, s, cell_fill, ncell, 0, cond);
  if (n > 0)
    hipLaunchKernelGGL(k_cell_assign, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, xw, g, cell_of,
                       scan_tmp, cond);
  hipLaunchKernelGGL(k_scan_single, dim3(1), dim3(1024), 0, s, scan_tmp, ncell, cell_start, cond);
  if (n > 0)
    hipLaunchKernelGGL(k_cell_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, xw, g,
                       cell_of, cell_start, cell_fill, cell_atoms, cell_code, xs, cond);
}

// ---------------------------------------------------------------------------
// small systems: the wrap, the row order and the cell list above in one
// workgroup (they are ten launches, 29 us and the gaps between them, at 500
// atoms; this 4.8 us, 6.9 at 1,367).  The rows' order and the cells' contents
// are the same; the order inside a cell is irrelevant there too.  Two atoms and
// four cells a thread: what its registers and LDS hold without a loop.
// ---------------------------------------------------------------------------
constexpr int PREP_THREADS = 1024, PREP_WAVES = PREP_THREADS / 64;
constexpr int PREP_ATOMS = 2 * PREP_THREADS;  // two atoms a thread
constexpr int PREP_CELLS = 4 * PREP_THREADS;  // four cells a thread

struct PrepArgs {
  int n, n_rows, ntypes, rows;  // atoms, centres, their rows with the padding
  const double *x;
  const int32_t *types;
  CellGrid g;
  double4 *xw;
  int32_t *type_count, *type_start, *pos_of_atom, *atom_of_pos;
  int32_t *cell_of, *cell_start, *cell_atoms;
  uint32_t *code;
  CellPos *xs;
  uint32_t *flags;
};

__global__ void __launch_bounds__(PREP_THREADS) k_prep_small(PrepArgs a) {
  __shared__ int32_t cells[PREP_CELLS];             // counts, then next free places
  __shared__ int32_t first[2][PREP_WAVES][MAXT];    // a wave's atoms of a type: counts, then first ranks
  __shared__ int32_t tstart[MAXT + 1], wsum[PREP_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int ncell = a.g.nc[0] * a.g.nc[1] * a.g.nc[2];
  for (int o = tid; o < ncell; o += PREP_THREADS) cells[o] = 0;
  for (int o = tid; o < a.rows; o += PREP_THREADS) a.atom_of_pos[o] = -1;
  __syncthreads();
  double4 p[2];
  int t[2], c[2], rank[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = h * PREP_THREADS + tid;
    const bool in = i < a.n;
    t[h] = -1;
    rank[h] = 0;
    if (in) {
      int u = a.types[i];
      if (u < 0 || u >= a.ntypes) {
        atomicOr(a.flags, FLAG_BAD_TYPE);
        u = 0;
      }
      p[h].x = wrap1(a.x[3 * i + 0], a.g.L[0]);
      p[h].y = wrap1(a.x[3 * i + 1], a.g.L[1]);
      p[h].z = wrap1(a.x[3 * i + 2], a.g.L[2]);
      p[h].w = (double)u;
      a.xw[i] = p[h];
      c[h] = (cell_coord(p[h].x, a.g.side[0], a.g.nc[0]) * a.g.nc[1] + cell_coord(p[h].y, a.g.side[1], a.g.nc[1])) *
                 a.g.nc[2] + cell_coord(p[h].z, a.g.side[2], a.g.nc[2]);
      a.cell_of[i] = c[h];
      atomicAdd(&cells[c[h]], 1);
      if (i < a.n_rows) t[h] = u;
    }
    for (int u = 0; u < a.ntypes; ++u) {
      const unsigned long long m = __ballot(t[h] == u);
      if (lane == 0) first[h][wv][u] = __popcll(m);
      if (t[h] == u) rank[h] = __popcll(m & ((1ull << lane) - 1ull));
    }
  }
  __syncthreads();
  if (tid < a.ntypes) {  // ranks run over the atoms in order: half by half, wave by wave
    int run = 0;
    for (int h = 0; h < 2; ++h)
      for (int w = 0; w < PREP_WAVES; ++w) {
        const int v = first[h][w][tid];
        first[h][w][tid] = run;
        run += v;
      }
    a.type_count[tid] = run;
    tstart[tid + 1] = (run + ROW_TILE - 1) / ROW_TILE * ROW_TILE;
  }
  // the cells' first atoms: four cells a thread, then the waves
  int v[4], sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = 4 * tid + k < ncell ? cells[4 * tid + k] : 0;
    sum += v[k];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  if (tid == 0) {
    tstart[0] = 0;
    for (int u = 0; u < a.ntypes; ++u) tstart[u + 1] += tstart[u];
    for (int u = 0; u <= a.ntypes; ++u) a.type_start[u] = tstart[u];
  }
  int at = incl - sum;
  for (int w = 0; w < wv; ++w) at += wsum[w];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (4 * tid + k < ncell) a.cell_start[4 * tid + k] = cells[4 * tid + k] = at;
    at += v[k];
  }
  if (tid == PREP_THREADS - 1) a.cell_start[ncell] = at;  // every cell lies before
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = h * PREP_THREADS + tid;
    if (i >= a.n) continue;
    if (t[h] >= 0) {
      const int pos = tstart[t[h]] + first[h][wv][t[h]] + rank[h];
      a.pos_of_atom[i] = pos;
      a.atom_of_pos[pos] = i;
    }
    const int cc = c[h], b = a.cell_start[cc], q = atomicAdd(&cells[cc], 1);
    a.cell_atoms[q] = i;
    a.xs[q] = CellPos{(float)p[h].x, (float)p[h].y, (float)p[h].z, i};
    const int cz = cc % a.g.nc[2], cy = (cc / a.g.nc[2]) % a.g.nc[1], cx = cc / (a.g.nc[1] * a.g.nc[2]);
    a.code[i] = ((uint32_t)(cx & 255) << 24) | ((uint32_t)(cy & 255) << 16) | ((uint32_t)(cz & 255) << 8) |
                (uint32_t)(q - b < 255 ? q - b : 255);
  }
}

bool launch_prep_small(hipStream_t s, int64_t n, int64_t n_rows, const double *coords, const int32_t *types, int ntypes,
                       const CellGrid &g, double4 *xw, uint32_t *flags, int32_t *type_count, int32_t *type_start,
                       int32_t *pos_of_atom, int32_t *atom_of_pos, int64_t rows, int32_t *cell_of,
                       int32_t *cell_start, int32_t *cell_atoms, uint32_t *cell_code, CellPos *xs) {
  if (n > PREP_ATOMS || (int64_t)g.nc[0] * g.nc[1] * g.nc[2] > PREP_CELLS) return false;
  const PrepArgs a{(int)n, (int)n_rows, ntypes, (int)rows, coords, types, g, xw, type_count, type_start,
                   pos_of_atom, atom_of_pos, cell_of, cell_start, cell_atoms, cell_code, xs, flags};
  hipLaunchKernelGGL(k_prep_small, dim3(1), dim3(PREP_THREADS), 0, s, a);
  return true;
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

void launch_fill_u32(hipStream_t s, uint32_t *p, int64_t n, uint32_t v) {
  if (n > 0) hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
}

// ---------------------------------------------------------------------------
// candidates within rlist (= rc + skin, inflated by the rounding of this
// kernel's FP32 distances, so that the exact r <= rc test of the formatting
// kernel only ever removes pairs): one wave per atom.  Its neighbour cells'
// atoms are runs of the cell order, cells adjacent there joined to one run
// (nine runs of three cells inside the box).  A run lies in one periodic image
// of each axis with at least three cells, so there its image shift stands in
// for the minimum image.  Bound by instruction issue, 27 cells' atoms a wave:
// three blocks of 64 are loaded together, so one latency is paid per run, and
// nothing but the test and the append is left per block.  32,000 copper
// atoms: cell by cell through the index list to FP64 positions, 150 us;
// positions in cell order loaded one block ahead by a cursor over the runs
// 117 (FP32 112), this 59.  62,565-centre brick 282 -> 101, 12,165 water atoms
// 71 -> 25, 500,000 atoms with 2 A skin 3.47 -> 1.05 ms.
// ---------------------------------------------------------------------------
constexpr int CAND_BATCH = 3;  // blocks of 64 atoms loaded together
__global__ void __launch_bounds__(256) k_candidates(int64_t n, const double4 *__restrict__ xw, CellGrid g,
                                                    const int32_t *__restrict__ cell_start,
                                                    const CellPos *__restrict__ xs, float rl2, int cap,
                                                    int32_t *__restrict__ cand, int32_t *__restrict__ cand_n,
                                                    uint32_t *flags, const uint32_t *cond) {
  if (skip_build(cond)) return;
  const int lane = threadIdx.x & 63;
  // uniform over the wave: the atom's data come by scalar loads
  const int64_t i = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= n) return;
  const double4 p = xw[i];
  // lane r < 27: the cell at offset (r / 9, r / 3 % 3, r % 3) - 1, each cell
  // once, and its image
  const int c0[3] = {cell_coord(p.x, g.side[0], g.nc[0]), cell_coord(p.y, g.side[1], g.nc[1]),
                     cell_coord(p.z, g.side[2], g.nc[2])};
  const int off[3] = {lane / 9 - 1, lane / 3 % 3 - 1, lane % 3 - 1};
  bool use = lane < 27;
  int v[3], img[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    v[a] = c0[a] + off[a];
    img[a] = 0;
    // one cell: itself only; two: itself and the one after it
    if (g.nc[a] < 3) use = use && (off[a] == 0 || (g.nc[a] == 2 && off[a] == 1));
    if (v[a] < 0) {
      v[a] += g.nc[a];
      img[a] = -1;
    } else if (v[a] >= g.nc[a]) {
      v[a] -= g.nc[a];
      img[a] = 1;
    }
    if (g.nc[a] < 3) img[a] = 0;  // by the minimum image
  }
  const int c = use ? (v[0] * g.nc[1] + v[1]) * g.nc[2] + v[2] : 0;
  const int cb = use ? cell_start[c] : 0;
  int ce = use ? cell_start[c + 1] : 0;
  const int ic = (img[0] + 1) * 9 + (img[1] + 1) * 3 + img[2] + 1;
  // join a cell to the one before it where both the order and the image go on
  const int pe = __shfl_up(ce, 1), pi = __shfl_up(ic, 1), pu = __shfl_up((int)use, 1);
  const bool joined = use && lane > 0 && pu && pe == cb && pi == ic;
  unsigned long long heads = __ballot(use && !joined);
  const unsigned long long tails = __ballot(joined);
  const bool mi = g.nc[0] < 3 || g.nc[1] < 3 || g.nc[2] < 3;
  int32_t count = 0;
  int32_t *out = cand + i * (int64_t)cap;
  while (heads) {
    const int r = __ffsll(heads) - 1;
    heads &= heads - 1;
    const int last = r + __ffsll(~(tails >> (r + 1))) - 1;  // lane 27 and on hold no cell
    const int b = __builtin_amdgcn_readlane(cb, r), e = __builtin_amdgcn_readlane(ce, last);
    const int im = __builtin_amdgcn_readlane(ic, r);
    const float px = (float)(p.x - (double)(im / 9 - 1) * g.L[0]), py = (float)(p.y - (double)(im / 3 % 3 - 1) * g.L[1]),
                pz = (float)(p.z - (double)(im % 3 - 1) * g.L[2]);
    for (int q0 = b; q0 < e; q0 += 64 * CAND_BATCH) {
      CellPos x[CAND_BATCH];
#pragma unroll
      for (int u = 0; u < CAND_BATCH; ++u) {
        const int q = q0 + 64 * u + lane;
        if (q0 + 64 * u < e) x[u] = xs[q < e ? q : e - 1];
      }
#pragma unroll
      for (int u = 0; u < CAND_BATCH; ++u) {
        if (q0 + 64 * u >= e) break;
        float dx = x[u].x - px, dy = x[u].y - py, dz = x[u].z - pz;
        if (mi) {
          if (g.nc[0] < 3) dx = min_image(dx, (float)g.L[0]);
          if (g.nc[1] < 3) dy = min_image(dy, (float)g.L[1]);
          if (g.nc[2] < 3) dz = min_image(dz, (float)g.L[2]);
        }
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        const bool keep = r2 <= rl2 && q0 + 64 * u + lane < e && x[u].j != (int)i;
        const unsigned long long m = __ballot(keep);
        const int at = count + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
        if (keep && at < cap) out[at] = x[u].j;
        count += __popcll(m);
      }
    }
  }
  if (lane == 0) {
    cand_n[i] = count < cap ? count : cap;
    if (count > cap) atomicOr(flags, FLAG_CAND_CAP);
  }
}

void launch_candidates(hipStream_t s, int64_t n, const double4 *xw, const CellGrid &g, const int32_t *cell_start,
                       const CellPos *xs, double rlist, int cand_cap, int32_t *cand, int32_t *cand_n,
                       uint32_t *flags, const uint32_t *cond) {
  if (n <= 0) return;
  // positions, the image's shift and their difference are each rounded to
  // 24 bits: at most 9 L 2^-24 in the distance
  const double far = rlist + 16.0 * std::max(g.L[0], std::max(g.L[1], g.L[2])) / 16777216.0;
  const float rl2 = (float)(far * far * (1.0 + 1e-6));
  hipLaunchKernelGGL(k_candidates, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, n, xw, g, cell_start, xs, rl2,
                     cand_cap, cand, cand_n, flags, cond);
}

// ---------------------------------------------------------------------------
// formatting (Section V-B): one wave per atom, keys in LDS.  The keys are
// ranked exactly by a bucketed counting sort: bucket = type * nb +
// floor(nb (quantised distance / (quantised rc + 1))^3), monotone in the key
// and holding equal expected counts (neighbours grow like r^3).  The keys are
// laid out by bucket, and rank = the bucket's start + the smaller keys in it.
// Bound by instruction issue (70 % of cycles on the VALU): 256 buckets hold
// less than one key on average, so few compare with another, and the keys'
// layout makes the writes of the list and the environment rows nearly
// contiguous.  Against 64 buckets with linked lists, keys left in candidate
// order: 500,000 atoms (2 A skin, environment rows) 1.66 -> 1.38 ms, 24,576
// water atoms 58 -> 49 us, 32,000 copper atoms (no skin) 80 -> 67 us.
// ---------------------------------------------------------------------------
constexpr int FMT_WAVES = 4;
constexpr int FMT_CAP = KEY_CAP;
constexpr int FMT_NB = 256;  // distance buckets, divided among the types
constexpr int FMT_KPL = FMT_CAP / 64;
static_assert(FMT_CAP % 64 == 0 && FMT_NB == 4 * 64, "keys and buckets per lane");

// bucket of a key with type t and quantised distance qd < qlim (inv_qlim =
// 1 / qlim in FP32); monotone non-decreasing in (t, qd) (every step is)
__device__ inline int fmt_bucket(int t, int nb, uint32_t qd, float inv_qlim) {
  const float x = (float)qd * inv_qlim;
  const int b = (int)(x * x * x * (float)nb);
  return t * nb + (b < nb - 1 ? b : nb - 1);
}
constexpr int FMT_BATCH = 4; // candidate gathers in flight per lane

// per-wave LDS of the format kernel: keys (staged r^2 first) [FMT_CAP] u64,
// neighbour and type, later the bucket [FMT_CAP] i32, bucket counts, later
// starts [FMT_NB + 1] i32
struct FmtLds {
  unsigned long long keys[FMT_CAP];
  int32_t jt[FMT_CAP];
  int32_t start[FMT_NB + 4];
};

__global__ void __launch_bounds__(256) k_format(int64_t n, const double4 *__restrict__ xw, Dims d, double L0,
                                                double L1, double L2, double rc2max,
                                                const int32_t *__restrict__ cand,
                                                const int32_t *__restrict__ cand_n, int cap,
                                                int32_t *__restrict__ nlist, int32_t *__restrict__ nreal,
                                                unsigned long long *overflow, int32_t *max_real, uint32_t *flags,
                                                float4 *__restrict__ rt32) {
  __shared__ __align__(16) FmtLds fmt_lds[FMT_WAVES];
  // uniform over the wave: the atom's data come by scalar loads
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * FMT_WAVES + wv;
  if (i >= n) return;
  unsigned long long *keys = fmt_lds[wv].keys;
  int32_t *jt = fmt_lds[wv].jt, *start = fmt_lds[wv].start;
  const int nb = FMT_NB / d.ntypes;
  const unsigned long long below = (1ull << lane) - 1ull;
  // keys stored and neighbours within rc per type, wave-uniform: ballot
  // prefix counts instead of atomics on one LDS address
  int kc = 0;
  int tc[MAXT];
#pragma unroll
  for (int t = 0; t < MAXT; ++t) tc[t] = 0;
  *(int4 *)(start + 4 * lane) = make_int4(0, 0, 0, 0);
  const double inv_w = 1.0 / (d.rcut - d.rcut_smth);
  const unsigned long long qlim = (unsigned long long)floor(d.rcut * 1e8) + 1ull;
  const float inv_qlim = 1.0f / (float)qlim;
  double4 p = xw[i];
  int nc = cand_n[i];
  const int32_t *ci = cand + i * (int64_t)cap;
  // pass 1: distances of all candidates; those within rc (r^2 <= rc2max,
  // the largest double whose square root is <= rc, so the same test as
  // sqrt(r^2) <= rc) are staged compactly, r^2 in their key slot
  for (int q0 = 0; q0 < nc; q0 += 64 * FMT_BATCH) {
    // issue the index loads, then the position gathers, of FMT_BATCH rounds
    // unconditional loads (lanes past the list reread its last entry and
    // are then masked), so none of them waits behind a branch
    int32_t jb[FMT_BATCH];
    double4 pb[FMT_BATCH];
#pragma unroll
    for (int u = 0; u < FMT_BATCH; ++u) {
      const int q = q0 + 64 * u + lane;
      jb[u] = ci[q < nc ? q : nc - 1];
    }
#pragma unroll
    for (int u = 0; u < FMT_BATCH; ++u) pb[u] = xw[jb[u]];
#pragma unroll
    for (int u = 0; u < FMT_BATCH; ++u)
      if (q0 + 64 * u + lane >= nc) {
        jb[u] = -1;
        pb[u] = p;
      }
#pragma unroll
    for (int u = 0; u < FMT_BATCH; ++u) {
      const int32_t j = jb[u];
      const double4 pj = pb[u];  // = p for lanes without a candidate (r = 0, not kept)
      double dx = min_image(pj.x - p.x, L0);
      double dy = min_image(pj.y - p.y, L1);
      double dz = min_image(pj.z - p.z, L2);
      double r2 = dx * dx + dy * dy;
      r2 = r2 + dz * dz;
      const bool keep = j >= 0 && r2 <= rc2max;
      const unsigned long long m = __ballot(keep);
      if (m == 0ull) continue;
      const int tj = (int)pj.w;
      const int slot = kc + __popcll(m & below);
      kc += __popcll(m);
      if (d.ntypes > 1) {
#pragma unroll
        for (int t = 0; t < MAXT; ++t)
          if (t < d.ntypes) tc[t] += __popcll(__ballot(keep && tj == t));
      }
      if (keep && slot < FMT_CAP) {
        keys[slot] = (unsigned long long)__double_as_longlong(r2);
        jt[slot] = j | (tj << 26);
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  int k = kc;
  if (k > FMT_CAP) {
    if (lane == 0) atomicOr(flags, FLAG_KEY_CAP);
    k = FMT_CAP;
  }
  if (d.ntypes == 1) tc[0] = kc;
  // pass 2, dense over the lanes: r, the key (type, floor(r 1e8), index), its
  // bucket and its place there
  unsigned long long key[FMT_KPL];
  int place[FMT_KPL];  // bucket << 16 | place
#pragma unroll
  for (int u = 0; u < FMT_KPL; ++u) {
    if (64 * u >= k) continue;
    const int q = 64 * u + lane;
    key[u] = 0;
    place[u] = -1;
    if (q < k) {
      const double r = sqrt(__longlong_as_double((long long)keys[q]));
      const int32_t v = jt[q];
      const uint32_t tj = (uint32_t)v >> 26, j = (uint32_t)v & ((1u << 26) - 1u);
      const uint32_t qd = (uint32_t)(r * 1e8);  // below 2^32 for every cutoff that is taken
      key[u] = ((unsigned long long)tj << 58) | ((unsigned long long)qd << 26) | j;
      const int b = fmt_bucket((int)tj, nb, qd, inv_qlim);
      place[u] = b << 16 | atomicAdd(&start[b], 1);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // exclusive scan of the bucket counts: lane takes four buckets
  {
    const int4 c = *(const int4 *)(start + 4 * lane);
    const int run = c.x + c.y + c.z + c.w;
    int incl = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    const int e = incl - run;
    *(int4 *)(start + 4 * lane) = make_int4(e, e + c.x, e + c.x + c.y, e + c.x + c.y + c.z);
    if (lane == 63) start[FMT_NB] = incl;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // the keys and their buckets in bucket order
#pragma unroll
  for (int u = 0; u < FMT_KPL; ++u) {
    if (64 * u >= k) continue;
    if (place[u] >= 0) {
      const int b = place[u] >> 16, at = start[b] + (place[u] & 0xffff);
      keys[at] = key[u];
      jt[at] = b;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  int tstart[MAXT], treal[MAXT];
  {
    int run = 0;
#pragma unroll
    for (int t = 0; t < MAXT; ++t) {
      const int c = t < d.ntypes ? tc[t] : 0;
      tstart[t] = run;
      run += c;
      treal[t] = t < d.ntypes ? (c < d.sel[t] ? c : d.sel[t]) : 0;
    }
  }
  int32_t *row = nlist + i * (int64_t)d.nnei;
  // exact rank of each key (keys are distinct)
  for (int q = lane; q < k; q += 64) {
    const unsigned long long key = keys[q];
    const int t = (int)(key >> 58);
    const int b = jt[q], m1 = start[b + 1];
    int rank = start[b];
    for (int m = rank; m < m1; ++m) rank += (keys[m] < key) ? 1 : 0;
    int ts = 0;
#pragma unroll
    for (int u = 0; u < MAXT; ++u)
      if (u == t) ts = tstart[u];
    int pos = rank - ts;
    // pos < 0 can only happen when the key buffer overflowed (flagged above)
    if (pos >= 0 && pos < d.sel[t]) {
      const int32_t j = (int32_t)(key & ((1ull << 26) - 1ull));
      row[d.off[t] + pos] = j;
      if (rt32) {
        // the slot's environment row (the mixed path's FP32 copy of FP64
        // values: from 1/r = rsqrt(r^2) with two Newton steps instead of the
        // environment kernel's square root and divisions, within an ulp or
        // two of its values before the rounding to FP32)
        const double4 D = pair_disp_sq(p, xw[j], L0, L1, L2);
        const double ir = rsqrt64(D.w), r = D.w * ir;
        const double x = fmin(fmax((r - d.rcut_smth) * inv_w, 0.0), 1.0);
        const double sv = (x * x * x * (-6.0 * x * x + 15.0 * x - 10.0) + 1.0) * ir, tv = sv * ir;
        rt32[i * (int64_t)d.nnei + d.off[t] + pos] =
            make_float4((float)sv, (float)(tv * D.x), (float)(tv * D.y), (float)(tv * D.z));
      }
    }
  }
  // only the real slots are written; k_pad_nlist fills the -1 padding when
  // the list is copied out (every device consumer stops at the real count)
  if (lane < d.ntypes) {
    int c = 0, cr = 0;
#pragma unroll
    for (int t = 0; t < MAXT; ++t)
      if (t == lane) {
        c = tc[t];
        cr = treal[t];
      }
    nreal[i * d.ntypes + lane] = cr;
    // the maximum only grows during the launch, so a stale read can only
    // cost an extra atomic; skipping the rest keeps 500k waves from
    // serialising on one address
    if (c > __hip_atomic_load(&max_real[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&max_real[lane], c);
    if (c > d.sel[lane]) atomicAdd(overflow, (unsigned long long)(c - d.sel[lane]));
  }
}

void launch_format(hipStream_t s, int64_t n, const double4 *xw, const Dims &d, const double *L, const int32_t *cand,
                   const int32_t *cand_n, int cand_cap, int32_t *nlist, int32_t *nreal, unsigned long long *overflow,
                   int32_t *max_real, uint32_t *flags, float4 *rt32) {
  if (n <= 0) return;
  // the largest double x with sqrt(x) <= rc (sqrt is correctly rounded and
  // monotone, so r^2 <= x exactly when sqrt(r^2) <= rc)
  double x = d.rcut * d.rcut;
  while (std::sqrt(x) > d.rcut) x = std::nextafter(x, 0.0);
  while (std::sqrt(std::nextafter(x, HUGE_VAL)) <= d.rcut) x = std::nextafter(x, HUGE_VAL);
  hipLaunchKernelGGL(k_format, dim3((unsigned)((n + FMT_WAVES - 1) / FMT_WAVES)), dim3(64 * FMT_WAVES), 0, s, n, xw,
                     d, L[0], L[1], L[2], x, cand, cand_n, cand_cap, nlist, nreal, overflow, max_real, flags, rt32);
}

// -1 in every slot past a type's real count
__global__ void k_pad_nlist(int64_t n, Dims d, const int32_t *__restrict__ nreal, int32_t *__restrict__ nlist) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;
  for (int t = 0; t < d.ntypes; ++t) {
    const int r = nreal[i * d.ntypes + t];
    for (int sl = r + lane; sl < d.sel[t]; sl += 64) nlist[i * (int64_t)d.nnei + d.off[t] + sl] = -1;
  }
}

void launch_pad_nlist(hipStream_t s, int64_t n, const Dims &d, const int32_t *nreal, int32_t *nlist) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_pad_nlist, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, n, d, nreal, nlist);
}

// ---------------------------------------------------------------------------
// skin check and reference copy for the MD driver
// ---------------------------------------------------------------------------
__global__ void k_max_disp(int64_t n, const double4 *__restrict__ xw, const double4 *__restrict__ xref, double L0,
                           double L1, double L2, double hs2, uint32_t *flags) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool far = false;
  if (i < n) {
    double4 a = xw[i], b = xref[i];
    double dx = min_image(a.x - b.x, L0), dy = min_image(a.y - b.y, L1), dz = min_image(a.z - b.z, L2);
    far = dx * dx + dy * dy + dz * dz > hs2;
  }
  if (__ballot(far) && (threadIdx.x & 63) == 0) atomicOr(flags, FLAG_REBUILD);
}

void launch_max_disp(hipStream_t s, int64_t n, const double4 *xw, const double4 *xref, const double *L,
                     double half_skin, uint32_t *flags) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_max_disp, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, xw, xref, L[0], L[1], L[2],
                     half_skin * half_skin, flags);
}

__global__ void k_copy_ref(int64_t n, const double4 *__restrict__ xw, double4 *__restrict__ xref,
                           const uint32_t *cond) {
  if (skip_build(cond)) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) xref[i] = xw[i];
}

void launch_copy_ref(hipStream_t s, int64_t n, const double4 *xw, double4 *xref, const uint32_t *cond) {
  if (n > 0)
    hipLaunchKernelGGL(k_copy_ref, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, xw, xref, cond);
}

__global__ void k_end_rebuild(uint32_t *flags, unsigned long long *nbuild) {
  if (threadIdx.x == 0 && (*flags & FLAG_REBUILD)) {
    *flags &= ~FLAG_REBUILD;
    *nbuild += 1ull;
  }
}

void launch_end_rebuild(hipStream_t s, uint32_t *flags, unsigned long long *nbuild) {
  hipLaunchKernelGGL(k_end_rebuild, dim3(1), dim3(64), 0, s, flags, nbuild);
}

}  // namespace dpk
