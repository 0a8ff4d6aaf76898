// neighbor.hip -- neighbour rows for the sums over j != i of Sec. II.B/II.C.
//
// The paper assumes neighbour counts NN_i and rows NL_im are given and uses
// the minimum image; it does not say how they are built.  Here:
//   1. atoms are binned into cells at least r_c wide along every cell vector
//      (fractional coordinates, float64; wider in a box that is mostly empty),
//      one cell per small structure;
//   2. a deterministic counting sort gives the internal atom order
//      (structure, cell, caller index): the atoms of a cell are contiguous;
//   3. the lanes of an atom walk the stencil cells in increasing cell index, or
//      the atoms and images of a small structure in order, and place members by
//      counts over the lanes, so every row comes out sorted by (j, image)
//      without a sort;
//   4. membership is the strict float64 test |d|^2 < r_c^2 on the canonical
//      displacement (no fused multiply-add), the same test for both cutoffs;
//   5. an exact radial row has the angular-range entries (|d|^2 < (r_c^A)^2)
//      first and the rest after, each part in order: the angular row of the sums
//      is the first nnA entries of the radial row.  A call without a skin builds
//      it at once; a run with a skin filters it at every step from candidate
//      rows (radius r_c^R + skin);
//   6. rev[m][i] locates i in the radial row of its m-th neighbour, so the force
//      pass can gather dU_j/dr_ji without atomics: a binary search on the sorted
//      parts of exact rows, or one on the candidate rows (once per candidate
//      build) and the candidate -> exact position map of every filter.
#include <algorithm>

#include "nep_kernels.h"

namespace nep {

// A grid stays below 2^32 threads.
constexpr int64_t kMaxBlocks = 1 << 22;

// Whether the row builder's blocks take ranges of atoms, see launch_cells.
__host__ __device__ inline bool rows_by_ranges(const BuildArgs& b) {
  return b.N < 2 * (int64_t)b.n_cells || b.n_cells > kMaxBlocks;
}

// Kernels of a rebuild take an optional gate: when it points to 0 they do
// nothing, so an MD step can issue a fixed kernel sequence and let the device
// decide whether the rows are rebuilt.
__device__ __forceinline__ bool gated_off(const int32_t* gate) { return gate && *gate == 0; }

__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// Structure id of every caller-order atom from the offsets array.
__global__ void k_assign_struct(const int64_t* __restrict__ offs, int32_t n_struct, int64_t N,
                                int32_t* __restrict__ sid) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  int lo = 0, hi = n_struct - 1;
  while (lo < hi) {  // last s with offs[s] <= i
    int mid = (lo + hi + 1) >> 1;
    if (offs[mid] <= i) lo = mid; else hi = mid - 1;
  }
  sid[i] = lo;
}

// Cell coordinates of a position inside structure st (fractional, wrapped
// along periodic directions, clamped along open ones).
__device__ inline void cell_coords(const StructInfo& st, double x, double y, double z,
                                   int& cx, int& cy, int& cz) {
  double s[3];
  s[0] = x * st.Hi[0] + y * st.Hi[3] + z * st.Hi[6];
  s[1] = x * st.Hi[1] + y * st.Hi[4] + z * st.Hi[7];
  s[2] = x * st.Hi[2] + y * st.Hi[5] + z * st.Hi[8];
  int c[3];
  for (int k = 0; k < 3; ++k) {
    double f = s[k];
    if (st.pbc[k]) f -= floor(f);
    f = fmin(fmax(f, 0.0), 1.0);
    int v = (int)(f * st.ncell[k]);
    c[k] = v < 0 ? 0 : (v >= st.ncell[k] ? st.ncell[k] - 1 : v);
  }
  cx = c[0];
  cy = c[1];
  cz = c[2];
}

// Structure of source atom e, and its cell in one with cells.
__device__ __forceinline__ int32_t struct_of(const BuildArgs& b, int64_t e) {
  return b.n_struct == 1 ? 0 : b.sid_ext[e];
}

__device__ __forceinline__ int cell_of(const StructInfo& st, double x, double y, double z) {
  int cx, cy, cz;
  cell_coords(st, x, y, z, cx, cy, cz);
  return st.cell_off + (cz * st.ncell[1] + cy) * st.ncell[0] + cx;
}

__global__ void k_cell_key(BuildArgs b) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= b.N || gated_off(b.gate)) return;
  const StructInfo& st = b.structs[struct_of(b, e)];
  if (st.mode != kModeCells) {  // one cell, in caller order (k_cell_scatter)
    b.key[e] = ~st.cell_off;
    if (e == st.start) b.cell_count[st.cell_off] = (int32_t)st.count;
    return;
  }
  const int k = cell_of(st, b.pos_ext[e], b.pos_ext[b.N + e], b.pos_ext[2 * b.N + e]);
  b.key[e] = k;
  atomicAdd(&b.cell_count[k], 1);
}

// Exclusive scan of n int32 counts by one block of 1024 threads.
__global__ void __launch_bounds__(1024) k_scan_1block(const int32_t* __restrict__ in,
                                                      int32_t* __restrict__ out, int32_t n,
                                                      const int32_t* gate) {
  __shared__ int32_t part[1024];
  if (gated_off(gate)) return;
  int t = threadIdx.x;
  int chunk = (n + 1023) / 1024;
  int lo = t * chunk, hi = min(n, lo + chunk);
  int32_t s = 0;
  for (int i = lo; i < hi; ++i) s += in[i];
  part[t] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    int32_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int32_t run = part[t] - s;
  for (int i = lo; i < hi; ++i) {
    int32_t c = in[i];
    out[i] = run;
    run += c;
  }
}

// A structure without cells keeps its order: its atoms come in caller order
// on the first call and stay so, and its cell needs no slots and no sort (its
// cell_fill stays 0).
__global__ void k_cell_scatter(BuildArgs b) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= b.N || gated_off(b.gate)) return;
  const int k = b.key[e];
  if (k < 0) {
    b.perm[b.cell_start[~k] + (e - b.structs[struct_of(b, e)].start)] = (int32_t)e;
    return;
  }
  int slot = atomicAdd(&b.cell_fill[k], 1);
  b.perm[b.cell_start[k] + slot] = (int32_t)e;
}

// Order the atoms of each cell by caller index (ext[source index], or the
// source index itself when ext is NULL).  The internal order is then a
// function of the positions and caller indices only: independent of the
// atomic slot assignment above and of the order the atoms came in.  One wave
// per cell: every lane holds up to kSortPerLane of the cell's atoms and
// counts, for each, the keys below its own (keys are distinct, so the counts
// are the sorted positions); the wave reads the cell's keys 64 at a time and
// passes them around with lane shuffles.  Cells above 64 kSortPerLane atoms
// (possible only for a structure that is one cell) are sorted by one lane.
constexpr int kSortPerLane = 16;

__global__ void __launch_bounds__(kBlock) k_cell_sort(const int32_t* __restrict__ cell_start,
                                                      const int32_t* __restrict__ cell_count,
                                                      const int32_t* __restrict__ cell_fill,
                                                      int32_t n_cells, const int32_t* __restrict__ ext,
                                                      int32_t* __restrict__ perm, const int32_t* gate) {
  const int lane = threadIdx.x & 63;
  const int64_t c = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (c >= n_cells || gated_off(gate)) return;  // the lanes of a wave leave together
  int32_t* p = perm + cell_start[c];
  const int n = cell_count[c];
  if (n <= 1 || cell_fill[c] == 0) return;  // (no slots taken: already in order)
  if (n > 64 * kSortPerLane) {
    if (lane != 0) return;
    for (int a = 1; a < n; ++a) {
      const int32_t v = p[a];
      const int32_t kv = ext ? ext[v] : v;
      int b = a - 1;
      while (b >= 0 && (ext ? ext[p[b]] : p[b]) > kv) {
        p[b + 1] = p[b];
        --b;
      }
      p[b + 1] = v;
    }
    return;
  }
  int32_t v[kSortPerLane], key[kSortPerLane], rank[kSortPerLane];
#pragma unroll
  for (int a = 0; a < kSortPerLane; ++a) {
    const int idx = lane + 64 * a;
    v[a] = idx < n ? p[idx] : 0;
    key[a] = idx < n ? (ext ? ext[v[a]] : v[a]) : INT32_MAX;
    rank[a] = 0;
  }
  for (int b0 = 0; b0 < n; b0 += 64) {
    const int idx = b0 + lane;
    int32_t kb = INT32_MAX;
    if (idx < n) {
      const int32_t u = p[idx];
      kb = ext ? ext[u] : u;
    }
    const int m = min(64, n - b0);
    for (int l = 0; l < m; ++l) {
      const int32_t k = __shfl(kb, l);
#pragma unroll
      for (int a = 0; a < kSortPerLane; ++a) rank[a] += k < key[a] ? 1 : 0;
    }
  }
  // every read of the cell's entries above has been consumed by the shuffles
#pragma unroll
  for (int a = 0; a < kSortPerLane; ++a)
    if (lane + 64 * a < n) p[rank[a]] = v[a];
}

// The same for cells that may hold any number of atoms, a thread to an atom: its
// place is the number of smaller keys in its cell (in b.cell, which k_gather_atoms
// takes the order from).  The whole cell by one lane, as above, would take n^2 / 4
// dependent steps for n atoms; here n / 8 for each of them at once.
__global__ void __launch_bounds__(kBlock) k_cell_rank(BuildArgs b) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= b.N || gated_off(b.gate)) return;
  const int32_t e = b.perm[k], c = b.key[e];
  if (c < 0) {  // a structure without cells: in order
    b.cell[k] = e;
    return;
  }
  const int32_t mine = b.ext_src ? b.ext_src[e] : e;
  const int32_t* p = b.perm + b.cell_start[c];
  const int n = b.cell_count[c];
  int rank = 0;
  for (int q = 0; q < n; q += 8) {
    int32_t other[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) other[u] = p[min(q + u, n - 1)];
    if (b.ext_src) {
#pragma unroll
      for (int u = 0; u < 8; ++u) other[u] = b.ext_src[other[u]];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) rank += q + u < n && other[u] < mine ? 1 : 0;
  }
  b.cell[b.cell_start[c] + rank] = e;
}

// `ranked`: the order is in b.cell (k_cell_rank), else in b.perm.
__global__ void k_gather_atoms(BuildArgs b, bool ranked) {
  const int64_t N = b.N;
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= N || gated_off(b.gate)) return;
  const int64_t e = ranked ? b.cell[k] : b.perm[k];
  if (ranked) b.perm[k] = (int32_t)e;
  const double x = b.pos_ext[e], y = b.pos_ext[N + e], z = b.pos_ext[2 * N + e];
  const int32_t t = b.types_ext[e];
  b.pos[k] = x;
  b.pos[N + k] = y;
  b.pos[2 * N + k] = z;
  b.types[k] = t;
  b.sid[k] = struct_of(b, e);
  if (rows_by_ranges(b)) b.cell[k] = b.key[e];
  if (b.vel_src)
    for (int c = 0; c < 3; ++c) b.vel_dst[c * N + k] = b.vel_src[c * N + e];
  if (b.ext_in) b.ext_out[k] = b.ext_in[e];
  if (!b.check) return;
  if (t < 0 || t >= b.n_types) atomicExch(&b.check[3], 1);
  if (!(isfinite(x) && isfinite(y) && isfinite(z))) atomicExch(&b.check[4], 1);
}

__global__ void k_fill_cells(BuildArgs b) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gated_off(b.gate)) return;
  if (b.check && i < 8) b.check[i] = 0;
  if (i < b.n_cells) {
    b.cell_count[i] = 0;
    b.cell_fill[i] = 0;
  }
}

__global__ void k_commit_rebuild(int64_t N, const double* __restrict__ pos2,
                                 const double* __restrict__ vel2, const int32_t* __restrict__ types2,
                                 const int32_t* __restrict__ ext2, double* __restrict__ pos,
                                 double* __restrict__ vel, int32_t* __restrict__ types,
                                 int32_t* __restrict__ ext, double* __restrict__ pos_ref,
                                 const int32_t* gate, double* mu_cum, int32_t* count,
                                 const StructInfo* __restrict__ st, StructInfo* __restrict__ st_ref) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= N || gated_off(gate)) return;
  if (k == 0 && mu_cum) *mu_cum = 1.0;  // the reference positions are the current ones
  if (k == 0 && st_ref) *st_ref = *st;  // and so is the reference cell
  if (k == 0 && count) atomicAdd(count, 1);  // rebuilds done
  for (int c = 0; c < 3; ++c) {
    const double x = pos2[c * N + k];
    pos[c * N + k] = x;
    pos_ref[c * N + k] = x;
    vel[c * N + k] = vel2[c * N + k];
  }
  types[k] = types2[k];
  ext[k] = ext2[k];
}

// The up-to-3 stencil cells along one cell vector in increasing order.
__device__ inline int stencil_1d(int c, int n, int periodic, int* out) {
  if (periodic) {
    if (n < 3) {
      for (int v = 0; v < n; ++v) out[v] = v;
      return n;
    }
    if (c == 0) {
      out[0] = 0; out[1] = 1; out[2] = n - 1;
    } else if (c == n - 1) {
      out[0] = 0; out[1] = n - 2; out[2] = n - 1;
    } else {
      out[0] = c - 1; out[1] = c; out[2] = c + 1;
    }
    return 3;
  }
  int k = 0;
  for (int v = c - 1; v <= c + 1; ++v)
    if (v >= 0 && v < n) out[k++] = v;
  return k;
}

// Set bits of m below this lane.
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Where a row builder puts the members it finds.  EXACT: the exact rows of a
// call without a skin, the angular-range members straight into L and the
// others parked in V's row (it is unused by such a call) until the number of
// angular ones is known; else the candidate rows V (radius r_c^R + skin).
// Members arrive in row order, so each part comes out sorted by (j, image).
template <bool EXACT>
struct RowSink {
  const Lists &V, &L;
  const int64_t N, i;
  const bool images;
  int32_t na = 0, no = 0;  // members found so far: angular, others (all of them: no, unless EXACT)
  __device__ __forceinline__ void put(bool angular, int32_t p, int32_t j, uint16_t code) const {
    const int64_t e = (int64_t)p * N + i;
    if (EXACT && angular) {
      if (p >= L.MR) return;
      L.nlR[e] = j;
      if (images) L.cdR[e] = code;
    } else {
      if (p >= V.MR) return;
      V.nlR[e] = j;
      if (!EXACT || images) V.cdR[e] = code;
    }
  }
  // after the last member, by the G lanes of the atom together
  template <int G>
  __device__ __forceinline__ void finish(int sub, int32_t* overflow) const {
    if constexpr (EXACT) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // the parked members are other lanes' stores
      const int32_t move = min(no, min(V.MR, L.MR - min(na, L.MR)));
      for (int32_t p = sub; p < move; p += G) {
        const int64_t from = (int64_t)p * N + i, to = (int64_t)(na + p) * N + i;
        L.nlR[to] = V.nlR[from];
        if (images) L.cdR[to] = V.cdR[from];
      }
      if (sub == 0) {
        L.nnR[i] = na + no;
        L.nnA[i] = na;
        if (na + no > L.MR) atomicMax(&overflow[0], na + no);
        if (na > L.MA) atomicMax(&overflow[1], na);
      }
    } else if (sub == 0) {
      V.nnR[i] = no;
      if (no > V.MR) atomicMax(&overflow[5], no);
    }
  }
};

// Rows of the atoms of cell-mode structures.  A block takes a part of a cell's
// atoms, G lanes each.  The atoms of the (up to 27) stencil cells are
// staged in LDS once, as float32 positions relative to one atom of the cell,
// in increasing internal index; every lane group walks them G at a
// time and lists those within the cutoff plus a bound of the float32 error,
// in order (ballot counts); the listed ones, about one in six, then take the
// float64 membership test that decides (the test is the same for every
// builder, so the rows are those of a sequential scan of the cells).
// Bound by instruction issue: the float64 tests and the staging's image
// arithmetic, then the walk.  A walk of each atom over its stencil, four
// lanes to it, was 510 dependent position loads and float64 tests per atom of
// the 4-species alloy: 179 us for 131,072 atoms and 58 us more to part the
// rows by cutoff, 87 us for 3,995.  This takes 130 and 14 us, parting included.
// Members staged in LDS and stored along consecutive atoms: 132 (and 75 for
// 66 us where the rows take a skin); one wave per cell: 158 to 162.
constexpr int kCellStage = 1024;  // staged candidates
constexpr int kCellList = 128;    // listed candidates of an atom between two exact passes
constexpr int kCellRun = 64;      // consecutive cells of an XCD

template <int G>
struct CellPart {  // LDS of a block of the row builder
  static constexpr int kAtoms = kBlock / G;  // atoms of a part of a cell
  float4 stage[kCellStage];
  int32_t list[kAtoms][kCellList];
  int32_t start[27], first[28];  // of the stencil's cells: first atom, running count of candidates
  float reach2[kBlock / 64];
};

// Starts and running counts of the cells around `cell` in increasing order, by a whole block.
template <int G>
__device__ __forceinline__ void cell_stencil(CellPart<G>& s, const StructInfo& st, int cell,
                                             const int32_t* __restrict__ cell_start,
                                             const int32_t* __restrict__ cell_count) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int c = cell - st.cell_off, cx = c % st.ncell[0], cy = c / st.ncell[0] % st.ncell[1],
            cz = c / (st.ncell[0] * st.ncell[1]);
  int sx[3], sy[3], sz[3];
  const int nx = stencil_1d(cx, st.ncell[0], st.pbc[0], sx), ny = stencil_1d(cy, st.ncell[1], st.pbc[1], sy),
            nz = stencil_1d(cz, st.ncell[2], st.pbc[2], sz);
  if (tid < 64) {
    int32_t n = 0;
    if (tid < nx * ny * nz) {
      const int x = tid % nx, y = tid / nx % ny, z = tid / (nx * ny);
      const int px = x == 0 ? sx[0] : (x == 1 ? sx[1] : sx[2]), py = y == 0 ? sy[0] : (y == 1 ? sy[1] : sy[2]),
                pz = z == 0 ? sz[0] : (z == 1 ? sz[1] : sz[2]);
      const int k = st.cell_off + (pz * st.ncell[1] + py) * st.ncell[0] + px;
      s.start[tid] = cell_start[k];
      n = cell_count[k];
    }
    int32_t run = n;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      const int32_t v = __shfl_up(run, off);
      if (lane >= off) run += v;
    }
    if (tid < 27) s.first[tid + 1] = run;
    if (tid == 0) s.first[0] = 0;
  }
}

// The rows of the atoms [a0, a0 + kBlock / G) of a cell of `count` atoms from `begin` on, by a whole block.
template <bool EXACT, int G>
__device__ __forceinline__ void cell_part_rows(CellPart<G>& s, const StructInfo& st, int begin, int count, int a0,
                                               const double* __restrict__ pos, int64_t N, double rcR2, double rcA2,
                                               const Lists& V, const Lists& L, int32_t* __restrict__ overflow) {
  const int tid = threadIdx.x, sub = tid & (G - 1), lane = tid & 63;
  const uint64_t gmask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1) << (lane & ~(G - 1));
  const float rc2 = (float)rcR2;
  const int total = s.first[27];
  const bool any_wrap = st.pbc[0] || st.pbc[1] || st.pbc[2];
  // float32 position relative to the cell's first atom (the nearest image of it)
  const double rx = pos[begin], ry = pos[N + begin], rz = pos[2 * N + begin];
  auto relative = [&](int64_t j, float& x, float& y, float& z) __attribute__((always_inline)) {
    double dx = pos[j] - rx, dy = pos[N + j] - ry, dz = pos[2 * N + j] - rz;
    if (any_wrap) {
      int n0, n1, n2;
      min_image(st, dx, dy, dz, n0, n1, n2);
      image_disp(st, dx, dy, dz, n0, n1, n2, dx, dy, dz);
    }
    x = (float)dx;
    y = (float)dy;
    z = (float)dz;
  };
  // A member j of i's row is less than one cell width from i, and i from the reference,
  // so the nearest image of j to the reference is the one next to i when two widths are
  // at most half the box; with fewer than four cells every staged candidate is listed.
  bool near_all = false;
  for (int k = 0; k < 3; ++k) near_all = near_all || (st.pbc[k] && st.ncell[k] < 4);
  const int a = a0 + tid / G;
  const bool live = a < count;
  const int64_t i = begin + min(a, count - 1);
  float xi, yi, zi;
  relative(i, xi, yi, zi);
  const double pxi = pos[i], pyi = pos[N + i], pzi = pos[2 * N + i];
  RowSink<EXACT> sink{V, L, N, i, false};
  int32_t* mine = s.list[tid / G];
  int listed = 0;
  // the float64 test of the listed candidates, G at a time
  auto exact_pass = [&]() __attribute__((always_inline)) {
    for (int q0 = 0; q0 < listed; q0 += G) {
      const int q = q0 + sub;
      bool ta = false, to = false;
      int32_t j = 0;
      if (q < listed) {
        j = mine[q];
        double Dx, Dy, Dz;
        {
#pragma clang fp contract(off)
          Dx = pos[j] - pxi;
          Dy = pos[N + j] - pyi;
          Dz = pos[2 * N + j] - pzi;
        }
        int n0, n1, n2;
        min_image(st, Dx, Dy, Dz, n0, n1, n2);
        if (!(j == i && n0 == 0 && n1 == 0 && n2 == 0)) {
          double dx, dy, dz;
          image_disp(st, Dx, Dy, Dz, n0, n1, n2, dx, dy, dz);
          const double r2 = norm2_exact(dx, dy, dz);
          ta = EXACT && r2 < rcA2;
          to = !ta && r2 < rcR2;
        }
      }
      const uint64_t ma = __ballot(ta) & gmask, mo = __ballot(to) & gmask;
      if (ta) sink.put(true, sink.na + lanes_below(ma), j, kCodeCenter);
      if (to) sink.put(false, sink.no + lanes_below(mo), j, kCodeCenter);
      sink.na += __popcll(ma);
      sink.no += __popcll(mo);
    }
    listed = 0;
  };
  for (int base = 0; base < total; base += kCellStage) {
    const int n = min(kCellStage, total - base);
    __syncthreads();  // the previous stage has been walked
    float far2 = 0.f;
    for (int k = tid; k < n; k += kBlock) {
      int l = 0, h = 26;  // last stencil cell whose first candidate is at or before base + k
      while (l < h) {
        const int mid = (l + h + 1) >> 1;
        if (s.first[mid] <= base + k) l = mid; else h = mid - 1;
      }
      const int32_t j = s.start[l] + base + k - s.first[l];
      float x, y, z;
      relative(j, x, y, z);
      far2 = fmaxf(far2, x * x + y * y + z * z);
      s.stage[k] = make_float4(x, y, z, __int_as_float(j));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) far2 = fmaxf(far2, __shfl_xor(far2, off));
    if (lane == 0) s.reach2[tid >> 6] = far2;
    __syncthreads();
    // the squared float32 distance of a pair is off by less than 1e-6 (r_c^2 + 4 of
    // the largest squared coordinate): two positions rounded to 2^-24, their
    // difference, and three products
    float m2 = s.reach2[0];
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) m2 = fmaxf(m2, s.reach2[w]);
    const float thr = near_all ? INFINITY : rc2 + 1e-6f * (rc2 + 8.f * (m2 + xi * xi + yi * yi + zi * zi));
    for (int k0 = 0; k0 < n; k0 += G) {
      const int k = k0 + sub;
      const float4 c = s.stage[min(k, n - 1)];
      const float dx = c.x - xi, dy = c.y - yi, dz = c.z - zi;
      // (written so that a non-finite distance lists the candidate)
      const bool near = live && k < n && !(dx * dx + dy * dy + dz * dz > thr);
      const uint64_t m = __ballot(near) & gmask;
      if (near) mine[listed + lanes_below(m)] = __float_as_int(c.w);
      listed += __popcll(m);
      if (listed > kCellList - G) {  // the same for the lanes of an atom
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        exact_pass();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    exact_pass();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (live) sink.template finish<G>(sub, overflow);
}

// The parts of a block's cell, the blocks along y sharing a cell.
template <bool EXACT, int G>
__global__ void __launch_bounds__(kBlock) k_build_rows_cells(
    const double* __restrict__ pos, int64_t N, const StructInfo* __restrict__ structs, int32_t n_struct,
    const int32_t* __restrict__ cell_start, const int32_t* __restrict__ cell_count, double rcR2, double rcA2, Lists V,
    Lists L, int32_t* __restrict__ overflow, const int32_t* gate) {
  __shared__ CellPart<G> s;
  if (gated_off(gate)) return;
  const int cell = (int)xcd_runs<kCellRun>();
  const int count = cell_count[cell], begin = cell_start[cell];
  if ((int)blockIdx.y * s.kAtoms >= count) return;
  // the structure this cell belongs to
  int lo = 0, hi = n_struct - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (structs[mid].cell_off <= cell) lo = mid; else hi = mid - 1;
  }
  const StructInfo& st = structs[lo];
  if (st.mode != kModeCells) return;
  cell_stencil(s, st, cell, cell_start, cell_count);
  __syncthreads();
  for (int a0 = blockIdx.y * s.kAtoms; a0 < count; a0 += gridDim.y * s.kAtoms)
    cell_part_rows<EXACT, G>(s, st, begin, count, a0, pos, N, rcR2, rcA2, V, L, overflow);
}

// The parts whose first atom lies in a block's range of half a part's atoms: mostly one or none in
// crowded cells, one for each cell where they hold an atom or two.
template <int G>
constexpr int cell_range() { return kBlock / G / 2; }

template <bool EXACT, int G>
__global__ void __launch_bounds__(kBlock) k_build_rows_ranges(
    const double* __restrict__ pos, int64_t N, const int32_t* __restrict__ sid, const StructInfo* __restrict__ structs,
    const int32_t* __restrict__ cell_id, const int32_t* __restrict__ cell_start, const int32_t* __restrict__ cell_count,
    double rcR2, double rcA2, Lists V, Lists L, int32_t* __restrict__ overflow, const int32_t* gate) {
  __shared__ CellPart<G> s;
  if (gated_off(gate)) return;
  constexpr int R = cell_range<G>();
  const int lane = threadIdx.x & 63;
  for (int64_t range = xcd_block() * R; range < N; range += (int64_t)gridDim.x * R) {
    int32_t my_cell = -1;
    bool head = false;
    if (lane < R && range + lane < N) {
      my_cell = cell_id[range + lane];
      if (my_cell >= 0) head = (range + lane - cell_start[my_cell]) % s.kAtoms == 0;
    }
    for (uint64_t heads = __ballot(head); heads; heads &= heads - 1) {  // the same in every wave
      const int at = __builtin_ctzll(heads);
      const int cell = __builtin_amdgcn_readfirstlane(__shfl(my_cell, at));
      const StructInfo& st = structs[sid[range + at]];
      const int begin = cell_start[cell];
      __syncthreads();  // the part before has been walked
      cell_stencil(s, st, cell, cell_start, cell_count);
      __syncthreads();
      cell_part_rows<EXACT, G>(s, st, begin, cell_count[cell], (int)(range + at - begin), pos, N, rcR2, rcA2, V, L,
                               overflow);
    }
  }
}

// Rows of the atoms of structures without cells (all-pairs and image modes:
// small cells), G lanes per atom.  The lanes take the structure's atoms j in
// order, G at a time; the images of j within the cutoff lie between two
// planes along every cell vector, |s_k + o_k| <= r_c / w_k with s the
// fractional nearest-image displacement and w_k the face width, so each lane
// lists the few offsets in that box (one or two per pair in cells of 100
// atoms, where the structure's image range holds 125), after the lanes
// below it; the listed (atom, image) pairs then take the float64 test of
// every builder, G at a time, and each member is placed by a count over the
// lanes' ballot bits.  The row is the one a sequential scan of the pairs
// writes: sorted by (j, image).  Testing the whole image range took 2.0 ms for
// the 132,000 atoms of 1,000 cells of the 3-species training model; this
// takes 0.24 ms.
constexpr int kWideList = 256;  // listed pairs of an atom between two exact passes

template <bool EXACT, int G>
__global__ void __launch_bounds__(kBlock) k_build_rows_wide(
    const double* __restrict__ pos, int64_t N, const int32_t* __restrict__ sid,
    const StructInfo* __restrict__ structs, double rcR2, double rcA2, Lists V, Lists L,
    int32_t* __restrict__ overflow, const int32_t* gate) {
  __shared__ int32_t list_j[kBlock / G][kWideList];
  __shared__ uint16_t list_c[kBlock / G][kWideList];
  const int sub = threadIdx.x & (G - 1);
  const int64_t i = (xcd_block() * blockDim.x + threadIdx.x) / G;
  if (i >= N || gated_off(gate)) return;  // the lanes of an atom leave together
  if (structs[sid[i]].mode == kModeCells) return;  // k_build_rows_cells' atoms
  const StructInfo st = structs[sid[i]];
  const int lane = threadIdx.x & 63;
  const uint64_t gmask = (G == 64 ? ~0ull : (1ull << (G & 63)) - 1) << (lane & ~(G - 1));
  int32_t* lj = list_j[threadIdx.x / G];
  uint16_t* lc = list_c[threadIdx.x / G];
  const double xi = pos[i], yi = pos[N + i], zi = pos[2 * N + i];
  const bool images = st.mode == kModeImages;
  RowSink<EXACT> sink{V, L, N, i, images};
  double bound[3] = {0.0, 0.0, 0.0};  // r_c / w_k, slightly enlarged
  if (images)
    for (int k = 0; k < 3; ++k)
      bound[k] = sqrt(rcR2 * (st.Hi[k] * st.Hi[k] + st.Hi[3 + k] * st.Hi[3 + k] + st.Hi[6 + k] * st.Hi[6 + k])) *
                     (1.0 + 1e-9) + 1e-9;
  int listed = 0;
  auto exact_pass = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int q0 = 0; q0 < listed; q0 += G) {
      const int q = q0 + sub;
      bool ta = false, to = false;
      int32_t j = 0;
      uint16_t code = kCodeCenter;
      if (q < listed) {
        j = lj[q];
        code = lc[q];
        double Dx, Dy, Dz;
        {
#pragma clang fp contract(off)
          Dx = pos[j] - xi;
          Dy = pos[N + j] - yi;
          Dz = pos[2 * N + j] - zi;
        }
        int n0, n1, n2, oa, ob, oc;
        min_image(st, Dx, Dy, Dz, n0, n1, n2);
        split_code(code, oa, ob, oc);
        n0 += oa;
        n1 += ob;
        n2 += oc;
        if (!(j == i && n0 == 0 && n1 == 0 && n2 == 0)) {
          double dx, dy, dz;
          image_disp(st, Dx, Dy, Dz, n0, n1, n2, dx, dy, dz);
          const double r2 = norm2_exact(dx, dy, dz);
          ta = EXACT && r2 < rcA2;
          to = !ta && r2 < rcR2;
        }
      }
      const uint64_t ma = __ballot(ta) & gmask, mo = __ballot(to) & gmask;
      if (ta) sink.put(true, sink.na + lanes_below(ma), j, code);
      if (to) sink.put(false, sink.no + lanes_below(mo), j, code);
      sink.na += __popcll(ma);
      sink.no += __popcll(mo);
    }
    listed = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  for (int64_t j0 = 0; j0 < st.count; j0 += G) {
    const bool have = j0 + sub < st.count;
    const int64_t j = st.start + min(j0 + sub, st.count - 1);
    int from[3] = {0, 0, 0}, n[3] = {1, 1, 1};
    if (images) {
      const double Dx = pos[j] - xi, Dy = pos[N + j] - yi, Dz = pos[2 * N + j] - zi;
      int n0, n1, n2;
      min_image(st, Dx, Dy, Dz, n0, n1, n2);
      const double s[3] = {Dx * st.Hi[0] + Dy * st.Hi[3] + Dz * st.Hi[6] + n0,
                           Dx * st.Hi[1] + Dy * st.Hi[4] + Dz * st.Hi[7] + n1,
                           Dx * st.Hi[2] + Dy * st.Hi[5] + Dz * st.Hi[8] + n2};
#pragma unroll
      for (int k = 0; k < 3; ++k) {  // (fmax and fmin keep the range for a NaN)
        from[k] = (int)fmax((double)-st.reach[k], ceil(-bound[k] - s[k]));
        n[k] = max((int)fmin((double)st.reach[k], floor(bound[k] - s[k])) - from[k] + 1, 0);
      }
    }
    const int c = have ? n[0] * n[1] * n[2] : 0;
    int32_t upto = c;  // pairs of the lanes up to this one
#pragma unroll
    for (int off = 1; off < G; off <<= 1) {
      const int32_t v = __shfl_up(upto, off, G);
      if (sub >= off) upto += v;
    }
    const int32_t all = __shfl(upto, G - 1, G);
    // list them, kWideList at most at a time
    for (int32_t first = 0; first < all;) {
      const int32_t room = min(kWideList - listed, all - first);
      for (int32_t q = max(upto - c, first); q < min(upto, first + room); ++q) {
        const int o = q - (upto - c), o2 = o % n[2], o1 = o / n[2] % n[1], o0 = o / (n[1] * n[2]);
        lj[listed + q - first] = (int32_t)j;
        lc[listed + q - first] = make_code(from[0] + o0, from[1] + o1, from[2] + o2);
      }
      listed += room;
      first += room;
      if (listed == kWideList) exact_pass();
    }
  }
  if (listed) exact_pass();
  sink.template finish<G>(sub, overflow);
}

// rev[m][i] = position of (i, -offset) in the row of j = nl[m][i] (rows
// sorted by (j, image)).
constexpr int kReverseLanes = 4;  // lanes per atom of k_reverse: lane s searches for entries s, s + 4, ...
constexpr int kReverseChunk = 4;  // entries whose searches a lane of k_reverse runs together

__global__ void k_reverse(int64_t N, const int32_t* __restrict__ nn, const int32_t* __restrict__ nl,
                          const uint16_t* __restrict__ cd, int32_t cap, int32_t* __restrict__ rev,
                          int32_t* __restrict__ err, const int32_t* gate) {
  const int sub = threadIdx.x & (kReverseLanes - 1);
  const int64_t i = (xcd_block() * blockDim.x + threadIdx.x) / kReverseLanes;
  if (i >= N || gated_off(gate)) return;
  const int cnt = min(nn[i], cap);
  bool bad = false;
  // kReverseChunk entries of the lane at a time: their binary searches advance
  // together, so each step has that many independent loads in flight
  constexpr int U = kReverseChunk;
  for (int m0 = sub; m0 < cnt; m0 += U * kReverseLanes) {
    int32_t j[U];
    uint32_t key[U];
    int lo[U], hi[U], found[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * kReverseLanes;
      j[u] = 0;
      key[u] = 0;
      lo[u] = 0;
      hi[u] = -1;  // an empty search for entries past the row
      found[u] = -1;
      if (m < cnt) {
        j[u] = nl[(int64_t)m * N + i];
        int a, b, c;
        split_code(cd[(int64_t)m * N + i], a, b, c);
        key[u] = (uint32_t)make_code(-a, -b, -c);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (m0 + u * kReverseLanes < cnt) hi[u] = min(nn[j[u]], cap) - 1;
    for (;;) {
      bool any = false;
      int mid[U];
      int32_t jj[U];
      uint32_t kk[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool live = found[u] < 0 && lo[u] <= hi[u];
        any |= live;
        mid[u] = live ? (lo[u] + hi[u]) >> 1 : -1;
        jj[u] = 0;
        kk[u] = 0;
        if (live) {
          jj[u] = nl[(int64_t)mid[u] * N + j[u]];
          kk[u] = cd[(int64_t)mid[u] * N + j[u]];
        }
      }
      if (!any) break;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (mid[u] < 0) continue;
        if (jj[u] == (int32_t)i && kk[u] == key[u]) found[u] = mid[u];
        else if (jj[u] < (int32_t)i || (jj[u] == (int32_t)i && kk[u] < key[u])) lo[u] = mid[u] + 1;
        else hi[u] = mid[u] - 1;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * kReverseLanes;
      if (m >= cnt) continue;
      if (found[u] < 0) {
        bad = true;
        found[u] = 0;
      }
      rev[(int64_t)m * N + i] = found[u];
    }
  }
  if (bad) atomicExch(err, 1);
}

// Reverse index of exact rows built without candidates: rev[m][i] = position
// of (i, -image) in the row of j, searched in the part of that row (angular
// or other) the entry belongs to -- membership of a pair is the same bits seen
// from either atom -- and with it the invariants of k_check_rows: counts, the
// neighbour inside the structure, the entry found pointing back with the
// opposite image code, codes within the image reach (*bad, the same bits).
// G lanes per atom; a lane's searches advance together, kReverseChunk at a
// time.  Bound by the latency of the searches' dependent reads: with 4, 8 and 16
// lanes 31, 23 and 28 us for 32,000 atoms, 82, 78 and 92 for 131,072, and 223,
// 209 and 226 for a batch of 132,000.  For a batch (DISP) it also writes every entry's displacement and
// species.
template <bool DISP, int G>
__global__ void __launch_bounds__(kBlock) k_reverse_exact(
    int64_t N, Lists L, const double* __restrict__ pos, const int32_t* __restrict__ types,
    const int32_t* __restrict__ sid, const StructInfo* __restrict__ structs, float4* __restrict__ disp,
    int32_t* __restrict__ err, int32_t* __restrict__ bad) {
  constexpr int U = kReverseChunk;
  const int sub = threadIdx.x & (G - 1);
  const int64_t i = (xcd_block() * blockDim.x + threadIdx.x) / G;
  if (i >= N) return;
  const int32_t* __restrict__ nl = L.nlR;
  const uint16_t* __restrict__ cd = L.cdR;
  // a row that overflowed (reported by the builder) is truncated, and so are its partners': an
  // MD step evaluates it before the host knows, so its entries need a position in bounds too
  const int all = L.nnR[i], part = L.nnA[i];
  const int nn = min(all, L.MR), na = min(part, nn);
  const StructInfo& st = structs[sid[i]];
  const bool images = st.mode == kModeImages;
  const int64_t s_lo = st.start, s_hi = st.start + st.count;
  int32_t b = part < 0 || all < 0 || part > all ? 1 : 0;
  bool lost = false;
  double xi = 0.0, yi = 0.0, zi = 0.0;
  if (DISP) {
    xi = pos[i];
    yi = pos[N + i];
    zi = pos[2 * N + i];
  }
  for (int m0 = sub; m0 < nn; m0 += U * G) {
    int32_t j[U];
    uint16_t code[U];
    uint32_t key[U];
    int lo[U], hi[U], found[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * G;
      const int64_t e = m < nn ? (int64_t)m * N + i : i;
      j[u] = nl[e];
      code[u] = images ? cd[e] : kCodeCenter;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * G;
      lo[u] = 0;
      hi[u] = -1;  // an empty search for entries past the row
      found[u] = -1;
      int oa, ob, oc;
      split_code(code[u], oa, ob, oc);
      key[u] = (uint32_t)make_code(-oa, -ob, -oc);
      if (m >= nn) continue;
      if (j[u] < s_lo || j[u] >= s_hi) {
        b |= 2;
        j[u] = (int32_t)i;
        continue;
      }
      if (images && (abs(oa) > st.reach[0] || abs(ob) > st.reach[1] || abs(oc) > st.reach[2])) b |= 16;
      const int nj = min(L.nnR[j[u]], L.MR), aj = min(L.nnA[j[u]], nj);
      lo[u] = m < na ? 0 : aj;
      hi[u] = (m < na ? aj : nj) - 1;
    }
    double px[U], py[U], pz[U];
    int32_t tj[U];
    if constexpr (DISP) {  // on their way during the searches
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t q = m0 + u * G < nn ? j[u] : (int32_t)i;
        px[u] = pos[q];
        py[u] = pos[N + q];
        pz[u] = pos[2 * N + q];
        tj[u] = types[q];
      }
    }
    for (;;) {
      bool any = false;
      int mid[U];
      int32_t jj[U];
      uint32_t kk[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool open = found[u] < 0 && lo[u] <= hi[u];
        any |= open;
        mid[u] = open ? (lo[u] + hi[u]) >> 1 : -1;
        jj[u] = 0;
        kk[u] = key[u];
        if (open) {
          jj[u] = nl[(int64_t)mid[u] * N + j[u]];
          if (images) kk[u] = cd[(int64_t)mid[u] * N + j[u]];
        }
      }
      if (!any) break;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (mid[u] < 0) continue;
        if (jj[u] == (int32_t)i && kk[u] == key[u]) found[u] = mid[u];
        else if (jj[u] < (int32_t)i || (jj[u] == (int32_t)i && kk[u] < key[u])) lo[u] = mid[u] + 1;
        else hi[u] = mid[u] - 1;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * G;
      if (m >= nn) continue;
      const int64_t e = (int64_t)m * N + i;
      if (found[u] < 0) {
        lost = true;
        found[u] = 0;
      }
      L.revR[e] = found[u];
      if constexpr (DISP) {
        double Dx, Dy, Dz;
        {
#pragma clang fp contract(off)
          Dx = px[u] - xi;
          Dy = py[u] - yi;
          Dz = pz[u] - zi;
        }
        int n0, n1, n2, oa, ob, oc;
        min_image(st, Dx, Dy, Dz, n0, n1, n2);
        split_code(code[u], oa, ob, oc);
        double dx, dy, dz;
        image_disp(st, Dx, Dy, Dz, n0 + oa, n1 + ob, n2 + oc, dx, dy, dz);
        disp[e] = make_float4((float)dx, (float)dy, (float)dz, __int_as_float(tj[u]));
      }
    }
  }
  if (lost) atomicExch(err, 1);
  if (b) atomicOr(bad, b);
}

// ---- row order for the network pass: atoms grouped by species in
// increasing internal index, each group padded to whole kRowGroup-row groups
// (padding rows hold -1).  Counting sort by blocks of kBlock atoms:
// per-block species counts, one exclusive scan over [species][block], then
// every atom takes its rank inside the block from wave ballots. ----

// Species of atom i for the row order, clamped into [0, Tn): a type out of
// range is reported by its own check, and the rows stay in bounds meanwhile.
__device__ __forceinline__ int row_species(const int32_t* types, int64_t i, int32_t Tn,
                                           int32_t per_type) {
  return per_type ? min(max(types[i], 0), Tn - 1) : 0;
}

__global__ void __launch_bounds__(kBlock) k_type_block_count(const int32_t* __restrict__ types,
                                                             int64_t N, int32_t Tn, int32_t per_type,
                                                             int32_t nb, int32_t* __restrict__ tblk,
                                                             int32_t* __restrict__ rows,
                                                             int64_t rows_len, const int32_t* gate) {
  __shared__ int32_t hist[kMaxTypes];
  if (gated_off(gate)) return;
  const int t = threadIdx.x;
  // every row slot starts as padding (-1); the scatter kernel fills the atoms
  for (int64_t r = (int64_t)blockIdx.x * kBlock + t; r < rows_len; r += (int64_t)nb * kBlock) rows[r] = -1;
  if (t < kMaxTypes) hist[t] = 0;
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * kBlock + t;
  if (i < N) atomicAdd(&hist[row_species(types, i, Tn, per_type)], 1);
  __syncthreads();
  if (t < Tn) tblk[(int64_t)t * nb + blockIdx.x] = hist[t];
}


__global__ void __launch_bounds__(kBlock) k_type_block_scatter(
    const int32_t* __restrict__ types, int64_t N, int32_t Tn, int32_t per_type, int32_t nb,
    const int32_t* __restrict__ tex, int32_t* __restrict__ rows, const int32_t* gate) {
  constexpr int kWaves = kBlock / 64;
  __shared__ int32_t wcount[kWaves][kMaxTypes], shift[kMaxTypes];
  if (gated_off(gate)) return;
  if (threadIdx.x == 0) {  // species t's rows start at a multiple of kRowGroup
    int32_t o = 0;
    for (int t = 0; t < Tn; ++t) {
      const int32_t first = tex[(int64_t)t * nb];
      const int32_t next = t + 1 < Tn ? tex[(int64_t)(t + 1) * nb] : (int32_t)N;
      shift[t] = o - first;
      o += (next - first + kRowGroup - 1) / kRowGroup * kRowGroup;
    }
  }
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t i = (int64_t)blockIdx.x * kBlock + t;
  const bool live = i < N;
  const int sp = live ? row_species(types, i, Tn, per_type) : -1;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  int rank = 0;
  for (int q = 0; q < Tn; ++q) {
    const uint64_t m = __ballot(sp == q);
    if (sp == q) rank = __popcll(m & below);
    if (lane == 0) wcount[w][q] = __popcll(m);
  }
  __syncthreads();
  if (!live) return;
  for (int v = 0; v < w; ++v) rank += wcount[v][sp];
  rows[tex[(int64_t)sp * nb + blockIdx.x] + shift[sp] + rank] = (int32_t)i;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

static inline dim3 grid_for(int64_t n, int b = kBlock) { return dim3((unsigned)div_up(n, b)); }

void launch_fill_i32(int32_t* a, int64_t n, int32_t v, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill_i32, grid_for(n), dim3(kBlock), 0, s, a, n, v);
}

void launch_assign_struct(const int64_t* offs, int32_t n_struct, int64_t N, int32_t* sid,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_assign_struct, grid_for(N), dim3(kBlock), 0, s, offs, n_struct, N, sid);
}

void launch_commit_rebuild(int64_t N, const double* pos2, const double* vel2, const int32_t* types2,
                           const int32_t* ext2, double* pos, double* vel, int32_t* types, int32_t* ext,
                           double* pos_ref, const int32_t* gate, hipStream_t s, double* mu_cum,
                           int32_t* count, const StructInfo* st, StructInfo* st_ref) {
  hipLaunchKernelGGL(k_commit_rebuild, grid_for(N), dim3(kBlock), 0, s, N, pos2, vel2, types2, ext2,
                     pos, vel, types, ext, pos_ref, gate, mu_cum, count, st, st_ref);
}

// Below this many atoms the row kernels give an atom more lanes: a whole wave
// in the builders (by cells 14 us against 17 with sixteen lanes for 3,995
// atoms, 24 against 34 for ten cells of 100 to 1,000; at 131,072 atoms the
// wave per atom takes 185 us against 136), sixteen lanes in the reverse
// searches and the filter: each lane then has one or two steps, where the chip
// is not full anyway.  Rows of the 4-species alloy, few lanes against many, in
// us: 46 : 25 at 4,000 atoms, 50 : 43 at 10,976, 65 : 62 at 19,652, 78 : 89 at
// 32,000.
constexpr int64_t kFewAtoms = 16384;

// Blocks to cells, in runs of cells to an XCD (with an eighth of the grid to each,
// a slab of 64,000 atoms in four times its volume left most of them idle: 576 us
// for the evaluation, 418 now).  Blocks to ranges of atoms where the cells hold
// fewer than two on average: most are empty then, and the others crowded where
// a box that is mostly empty has larger cells (5,562 atoms in a thousand times
// their volume: 6,970 us for the evaluation with blocks to cells, 430 with
// ranges; 64,000 in twenty times: 909 and 615).  In full cells the ranges are the
// slower: 186 us against 130 for 131,072 atoms, 14 registers more for the loop
// over parts and two parts to some blocks.
template <bool EXACT, int G>
static void launch_cells(const BuildArgs& b, const Lists& V, const Lists& L, hipStream_t s) {
  if (rows_by_ranges(b)) {
    const int64_t blocks = std::min<int64_t>(div_up(b.N, cell_range<G>()), kMaxBlocks);
    hipLaunchKernelGGL((k_build_rows_ranges<EXACT, G>), dim3((unsigned)blocks), dim3(kBlock), 0, s, b.pos, b.N, b.sid,
                       b.structs, b.cell, b.cell_start, b.cell_count, b.rcR2, b.rcA2, V, L, b.overflow, b.gate);
    return;
  }
  // blocks along y share a cell's atoms: enough for cells of half as many again
  // as the average (fuller ones take another turn)
  const int64_t per = b.N * 3 / (2 * (int64_t)b.n_cells) + 1;
  const int64_t y = std::min<int64_t>(div_up(per, kBlock / G), 64);
  hipLaunchKernelGGL((k_build_rows_cells<EXACT, G>), dim3((unsigned)b.n_cells, (unsigned)y), dim3(kBlock), 0, s, b.pos,
                     b.N, b.structs, b.n_struct, b.cell_start, b.cell_count, b.rcR2, b.rcA2, V, L, b.overflow, b.gate);
}

template <bool EXACT>
static void launch_members(const BuildArgs& b, const Lists& V, const Lists& L, hipStream_t s) {
  if (b.cell_rows) {
    if (b.N < kFewAtoms) launch_cells<EXACT, 64>(b, V, L, s);
    else launch_cells<EXACT, 16>(b, V, L, s);
  }
  if (b.wide_rows) {
    if (b.N < kFewAtoms)
      hipLaunchKernelGGL((k_build_rows_wide<EXACT, 64>), grid_for(b.N * 64), dim3(kBlock), 0, s, b.pos, b.N, b.sid,
                         b.structs, b.rcR2, b.rcA2, V, L, b.overflow, b.gate);
    else
      hipLaunchKernelGGL((k_build_rows_wide<EXACT, 16>), grid_for(b.N * 16), dim3(kBlock), 0, s, b.pos, b.N, b.sid,
                         b.structs, b.rcR2, b.rcA2, V, L, b.overflow, b.gate);
  }
}

template <bool DISP, int G>
static void launch_reverse_exact(const BuildArgs& b, const Lists& L, float4* disp, hipStream_t s) {
  hipLaunchKernelGGL((k_reverse_exact<DISP, G>), grid_for(b.N * G), dim3(kBlock), 0, s, b.N, L, b.pos, b.types, b.sid,
                     b.structs, disp, b.overflow + 2, b.overflow + 6);
}

void launch_build_rows(const BuildArgs& b0, const Lists& V, const Lists& L, float4* disp, hipStream_t s) {
  BuildArgs b = b0;
  b.gate = nullptr;
  launch_members<true>(b, V, L, s);
  const bool wide = b.N < kFewAtoms;
  if (disp) wide ? launch_reverse_exact<true, 16>(b, L, disp, s) : launch_reverse_exact<true, 8>(b, L, disp, s);
  else wide ? launch_reverse_exact<false, 16>(b, L, disp, s) : launch_reverse_exact<false, 8>(b, L, disp, s);
}

void launch_reverse(int64_t N, const Lists& L, int32_t* err, const int32_t* gate, hipStream_t s) {
  hipLaunchKernelGGL(k_reverse, grid_for(N * kReverseLanes), dim3(kBlock), 0, s, N, L.nnR, L.nlR, L.cdR, L.MR,
                     L.revR, err, gate);
}

// Candidate rows at sqrt(b.rcR2) and their reverse index, rebuilt when the
// gate is set.
void launch_build_verlet(const BuildArgs& b, const Lists& V, hipStream_t s) {
  launch_members<false>(b, V, V, s);
  launch_reverse(b.N, V, b.overflow + 2, b.gate, s);
}

// Exact radial row from the candidate row with the same float64 membership
// test: the entries with |d|^2 < (r_c^A)^2 first, then the others, each part
// in candidate order; nnA = size of the first part.  V.fmap[m][i] = exact
// position of candidate m (or -1).  G lanes per atom take the candidates m =
// s, s + G, ...: with four the 16 atoms of a wave read and write whole
// 64-byte runs of a row, and with many atoms the loads are what the kernel
// takes (its address units are busy for three quarters of it; 117 us for 131,072
// atoms); with few it is a chain of steps, shorter with sixteen lanes (18 us
// to 8.5 for 2,048 atoms).  Both passes walk a lane's candidates in
// chunks of kFilterChunk: the index words of a chunk are loaded together,
// then the positions (pass 1) or the row words (pass 2), so a lane has a
// chunk's loads in flight at once instead of one dependent chain per
// candidate.  Pass 1 classifies, counts the members and keeps the classes in
// register bit masks; pass 2 goes through the candidates in order, and
// counts over wave ballots of the class flags give each member its exact position.
// The rows are the same as those of a single sequential pass.
// With images a candidate's code counts from the nearest image at the build, and
// an atom near half a cell vector has another one as soon as it moves: the
// entry is the same image all the same, so its offset comes from the reference
// positions (and cell, st_ref, where the cell changes), and the exact entry's code
// counts from the nearest image now, which its readers take.
constexpr int kFilterChunk = 4;

struct ImageOffset {
  int n[3];
};

// Offset of the candidate of code `code`, from the difference of the reference positions.
__device__ __forceinline__ ImageOffset offset_at_build(const StructInfo& st, const double* __restrict__ ref, int64_t N,
                                                       int64_t i, int64_t j, uint16_t code) {
  ImageOffset o;
  int a, b, c;
  min_image(st, ref[j] - ref[i], ref[N + j] - ref[N + i], ref[2 * N + j] - ref[2 * N + i], o.n[0], o.n[1], o.n[2]);
  split_code(code, a, b, c);
  o.n[0] += a;
  o.n[1] += b;
  o.n[2] += c;
  return o;
}

template <bool BATCH, bool IMAGES, int G>
__global__ void __launch_bounds__(kBlock) k_filter_rows(const double* __restrict__ pos, int64_t N,
                                                        const int32_t* __restrict__ sid,
                                                        const StructInfo* __restrict__ structs,
                                                        StructInfo st0, const double* __restrict__ ref,
                                                        const StructInfo* __restrict__ st_ref, Lists V, double rcR2,
                                                        double rcA2, Lists L,
                                                        int32_t* __restrict__ overflow) {
  constexpr int U = kFilterChunk;
  constexpr int32_t kOuter = -2, kAngular = -3;
  const int sub = threadIdx.x & (G - 1);
  const int64_t i = (xcd_block() * blockDim.x + threadIdx.x) / G;
  if (i >= N) return;  // the lanes of an atom leave together
  const StructInfo& st = BATCH ? structs[sid[i]] : st0;
  const StructInfo& st_built = BATCH ? *st_ref : st0;
  const int32_t* __restrict__ vnl = V.nlR;
  const uint16_t* __restrict__ vcd = V.cdR;
  const int32_t* __restrict__ vrev = V.revR;
  int32_t* __restrict__ fmap = V.fmap;
  int32_t* __restrict__ lnl = L.nlR;
  int32_t* __restrict__ lrev = L.revR;
  uint16_t* __restrict__ lcd = L.cdR;
  const int nv = min(V.nnR[i], V.MR);
  const int steps = (nv + G - 1) / G;  // the same for every lane of an atom
  constexpr bool images = IMAGES;  // the structure's, one for all (a run's)
  const double xi = pos[i], yi = pos[N + i], zi = pos[2 * N + i];
  int32_t na = 0, no = 0;
  // classes of the lane's first 64 candidates (t = local index) as bit masks;
  // later ones (rows over 64 G candidates) go through V.fmap
  uint64_t mask_a = 0, mask_o = 0;
  // the index words of chunk t0 + U are loaded while chunk t0's positions
  // are in flight
  int32_t jn[U];
  uint16_t cn[U];
  auto load_words = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = (t0 + u) * G + sub;
      jn[u] = (int32_t)i;  // past the row: the atom itself, in bounds and never classified
      cn[u] = kCodeCenter;
      if (m < nv) {
        jn[u] = vnl[(int64_t)m * N + i];
        if (images) cn[u] = vcd[(int64_t)m * N + i];
      }
    }
  };
  load_words(0);
  for (int t0 = 0; t0 < steps; t0 += U) {
    int32_t j[U];
    uint16_t code[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      j[u] = jn[u];
      code[u] = cn[u];
    }
    double px[U], py[U], pz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      px[u] = pos[j[u]];
      py[u] = pos[N + j[u]];
      pz[u] = pos[2 * N + j[u]];
    }
    if (t0 + U < steps) load_words(t0 + U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u, m = t * G + sub;
      if (m >= nv) continue;
      double Dx, Dy, Dz;
      {
#pragma clang fp contract(off)
        Dx = px[u] - xi;
        Dy = py[u] - yi;
        Dz = pz[u] - zi;
      }
      int n0, n1, n2;
      if (images) {
        const ImageOffset o = offset_at_build(st_built, ref, N, i, j[u], code[u]);
        n0 = o.n[0];
        n1 = o.n[1];
        n2 = o.n[2];
      } else {
        min_image(st, Dx, Dy, Dz, n0, n1, n2);
      }
      double dx, dy, dz;
      image_disp(st, Dx, Dy, Dz, n0, n1, n2, dx, dy, dz);
      const double r2 = norm2_exact(dx, dy, dz);
      int32_t f = -1;
      if (r2 < rcA2) {
        f = kAngular;
        ++na;
      } else if (r2 < rcR2) {
        f = kOuter;
        ++no;
      }
      if (t < 64) {
        if (f == kAngular) mask_a |= 1ull << t;
        if (f == kOuter) mask_o |= 1ull << t;
      } else {
        fmap[(int64_t)m * N + i] = f;
      }
    }
  }
  int32_t a_all = na, o_all = no;
#pragma unroll
  for (int off = 1; off < G; off <<= 1) {
    a_all += __shfl_xor(a_all, off);
    o_all += __shfl_xor(o_all, off);
  }
  // pass 2: candidate m = G t + s is lane s's t-th; every lane of the atom's
  // group runs every step, so the group's ballot bits are whole at each step
  const int lane = threadIdx.x & 63;
  const uint64_t gmask = (G == 64 ? ~0ull : ((1ull << G) - 1)) << (lane & ~(G - 1));
  const uint64_t below = (1ull << lane) - 1;
  int32_t pa = 0, po = a_all;  // next angular / outer position
  // the members' words of chunk t0 + U are loaded while chunk t0 is placed
  int32_t cq[U], jq[U], rq[U];
  uint16_t kq[U];
  auto load_members = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u, m = t * G + sub;
      const int64_t e = (int64_t)m * N + i;
      cq[u] = -1;
      if (m < nv) {
        if (t < 64) cq[u] = ((mask_a >> t) & 1) ? kAngular : (((mask_o >> t) & 1) ? kOuter : -1);
        else cq[u] = fmap[e];
      }
      jq[u] = 0;
      rq[u] = 0;
      kq[u] = kCodeCenter;
      if (cq[u] != -1) {
        jq[u] = vnl[e];
        rq[u] = vrev[e];
        if (images) {  // the same image, counted from the nearest one now
          const ImageOffset o = offset_at_build(st_built, ref, N, i, jq[u], vcd[e]);
          int n0, n1, n2;
          min_image(st, pos[jq[u]] - xi, pos[N + jq[u]] - yi, pos[2 * N + jq[u]] - zi, n0, n1, n2);
          kq[u] = make_code(o.n[0] - n0, o.n[1] - n1, o.n[2] - n2);
        }
      }
    }
  };
  load_members(0);
  for (int t0 = 0; t0 < steps; t0 += U) {
    int32_t c[U], jn[U], rn[U];
    uint16_t cn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = cq[u];
      jn[u] = jq[u];
      rn[u] = rq[u];
      cn[u] = kq[u];
    }
    if (t0 + U < steps) load_members(t0 + U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = (t0 + u) * G + sub;
      const int64_t e = (int64_t)m * N + i;
      const int32_t fa = c[u] == kAngular, fo = c[u] == kOuter;
      const uint64_t ma = __ballot(fa) & gmask, mo = __ballot(fo) & gmask;
      const int32_t ta = __popcll(ma), to = __popcll(mo);
      const int32_t ba = __popcll(ma & below), bo = __popcll(mo & below);
      if (m < nv && !(fa | fo)) fmap[e] = -1;
      if (fa | fo) {
        const int32_t p = fa ? pa + ba : po + bo;
        fmap[e] = p;
        if (p < L.MR) {
          lnl[(int64_t)p * N + i] = jn[u];
          lrev[(int64_t)p * N + i] = rn[u];  // candidate position, resolved by its reader
          if (images) lcd[(int64_t)p * N + i] = cn[u];
        }
      }
      pa += ta;
      po += to;
    }
  }
  if (sub == 0) {
    const int32_t total = a_all + o_all;
    L.nnR[i] = total;
    L.nnA[i] = a_all;
    if (total > L.MR) atomicMax(&overflow[0], total);
    if (a_all > L.MA) atomicMax(&overflow[1], a_all);
  }
}

// rev of the exact rows: the filter left in L.revR[p][i] the candidate
// position of i in the row of j = L.nlR[p][i]; the exact position there is
// V.fmap of that candidate entry, written in place.  G lanes per atom
// take exact entries p = s, s + G, ..., four or sixteen as in the filter; a lane
// loads the words of kFilterChunk entries, then their map
// entries, then writes them.  For a batch (DISP) it also writes every
// entry's float32 displacement and species (as bits), read by each parameter
// set's passes.
template <bool DISP, int G>
__global__ void __launch_bounds__(kBlock) k_reverse_from_candidates(
    int64_t N, Lists V, Lists L, const double* __restrict__ pos, const int32_t* __restrict__ types,
    const int32_t* __restrict__ sid, const StructInfo* __restrict__ structs, float4* __restrict__ disp,
    int32_t* __restrict__ err) {
  constexpr int U = kFilterChunk;
  const int sub = threadIdx.x & (G - 1);
  const int64_t i = (xcd_block() * blockDim.x + threadIdx.x) / G;
  if (i >= N) return;
  const int32_t* __restrict__ fmap = V.fmap;
  const int32_t* __restrict__ lnl = L.nlR;
  int32_t* __restrict__ lrev = L.revR;
  const int nn = min(L.nnR[i], L.MR);
  bool broken = false;
  StructInfo st;
  double xi = 0.0, yi = 0.0, zi = 0.0;
  if (DISP) {
    st = structs[sid[i]];
    xi = pos[i];
    yi = pos[N + i];
    zi = pos[2 * N + i];
  }
  // the words of chunk p0 + U G are loaded while chunk p0's map entries are in flight
  int32_t jq[U], rq[U];
  auto load_words = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u * G;
      jq[u] = 0;
      rq[u] = 0;
      if (p < nn) {
        jq[u] = lnl[(int64_t)p * N + i];
        rq[u] = lrev[(int64_t)p * N + i];
      }
    }
  };
  load_words(sub);
  for (int p0 = sub; p0 < nn; p0 += U * G) {
    int32_t j[U], r[U], g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      j[u] = jq[u];
      r[u] = rq[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] = p0 + u * G < nn ? fmap[(int64_t)r[u] * N + j[u]] : 0;
    if (p0 + U * G < nn) load_words(p0 + U * G);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u * G;
      if (p >= nn) continue;
      if (g[u] < 0) {
        broken = true;
        g[u] = 0;
      }
      lrev[(int64_t)p * N + i] = min(g[u], L.MR - 1);
    }
    if constexpr (DISP) {
      double px[U], py[U], pz[U];
      int32_t t[U];
      uint16_t code[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // past the row: word 0, an atom in bounds
        px[u] = pos[j[u]];
        py[u] = pos[N + j[u]];
        pz[u] = pos[2 * N + j[u]];
        t[u] = types[j[u]];
        code[u] = kCodeCenter;
        if (st.mode == kModeImages && p0 + u * G < nn) code[u] = L.cdR[(int64_t)(p0 + u * G) * N + i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + u * G;
        if (p >= nn) continue;
        double Dx, Dy, Dz;
        {
#pragma clang fp contract(off)
          Dx = px[u] - xi;
          Dy = py[u] - yi;
          Dz = pz[u] - zi;
        }
        int n0, n1, n2, oa, ob, oc;
        min_image(st, Dx, Dy, Dz, n0, n1, n2);
        split_code(code[u], oa, ob, oc);
        double dx, dy, dz;
        image_disp(st, Dx, Dy, Dz, n0 + oa, n1 + ob, n2 + oc, dx, dy, dz);
        disp[(int64_t)p * N + i] = make_float4((float)dx, (float)dy, (float)dz, __int_as_float(t[u]));
      }
    }
  }
  if (broken) atomicExch(err, 1);
}

// Checks, for every atom i of the exact rows, the invariants under which the
// evaluation kernels only touch memory inside their buffers: nnA <= nnR <= MR;
// every neighbour j lies in i's structure; its reverse position r lies in
// j's row (r < nnR[j]) and that entry points back to i with the opposite
// image code; image codes stay within the structure's image reach.  Any
// violation sets a bit of *bad (1: counts, 2: neighbour index, 4: reverse
// position, 8: reverse entry, 16: image code); rows that overflowed their
// capacity are reported by the overflow flags instead.
constexpr int kCheckLanes = 4;  // lanes per atom of k_check_rows (entries s, s + 4, ...)
constexpr int kCheckChunk = 4;  // entries a lane checks together

__global__ void __launch_bounds__(kBlock) k_check_rows(int64_t N, const int32_t* __restrict__ sid,
                                                       const StructInfo* __restrict__ structs,
                                                       StructInfo st0, int32_t batch, Lists L,
                                                       const int32_t* __restrict__ fmap, int32_t MV,
                                                       int32_t* __restrict__ bad) {
  constexpr int G = kCheckLanes, U = kCheckChunk;
  const int sub = threadIdx.x & (G - 1);
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  if (i >= N) return;
  const StructInfo& st = batch ? structs[sid[i]] : st0;
  const int nn = L.nnR[i], na = L.nnA[i];
  if (nn > L.MR) return;  // overflow: reported and handled by the caller
  int32_t b = 0;
  if (sub == 0 && (na < 0 || nn < 0 || na > nn)) b |= 1;
  const bool images = st.mode == kModeImages;
  const int64_t lo = st.start, hi = st.start + st.count;
  // a chunk's index words first, then the partners' row lengths and reverse
  // entries (each read only when the words before it are in bounds)
  for (int m0 = sub; m0 < max(nn, 0); m0 += U * G) {
    int32_t j[U], r[U];
    bool jok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * G;
      j[u] = 0;
      r[u] = 0;
      if (m < nn) {
        j[u] = L.nlR[(int64_t)m * N + i];
        r[u] = L.revR[(int64_t)m * N + i];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      jok[u] = m0 + u * G < nn && j[u] >= lo && j[u] < hi;
      if (m0 + u * G < nn && !jok[u]) b |= 2;
      if (fmap && jok[u]) r[u] = r[u] >= 0 && r[u] < MV ? fmap[(int64_t)r[u] * N + j[u]] : -1;
    }
    int nj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) nj[u] = jok[u] ? L.nnR[j[u]] : 0;
    int32_t back[U];
    bool rok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      rok[u] = jok[u] && r[u] >= 0 && r[u] < min(nj[u], L.MR);
      if (jok[u] && !rok[u]) b |= 4;
      back[u] = rok[u] ? L.nlR[(int64_t)r[u] * N + j[u]] : (int32_t)i;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!rok[u]) continue;
      if (back[u] != (int32_t)i) b |= 8;
      if (images) {
        const int64_t e = (int64_t)(m0 + u * G) * N + i, er = (int64_t)r[u] * N + j[u];
        int oa, ob, oc, ra, rb, rc;
        split_code(L.cdR[e], oa, ob, oc);
        split_code(L.cdR[er], ra, rb, rc);
        if (oa != -ra || ob != -rb || oc != -rc) b |= 8;
        if (abs(oa) > st.reach[0] || abs(ob) > st.reach[1] || abs(oc) > st.reach[2]) b |= 16;
      }
    }
  }
  if (b) atomicOr(bad, b);
}

void launch_check_rows(int64_t N, const int32_t* sid, const StructInfo* structs, const StructInfo& st0,
                       bool batch, const Lists& L, const Lists* V, int32_t* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_check_rows, grid_for(N * kCheckLanes), dim3(kBlock), 0, s, N, sid, structs, st0,
                     (int32_t)(batch ? 1 : 0), L, V ? V->fmap : nullptr, V ? V->MR : 0, bad);
}

// Few atoms: the gather looks the positions up itself, a launch less (a step of
// 5,323 atoms 89 -> 86 us).  Many: its random reads of the map would fill the caches
// that it reads the partial forces through (131,072 atoms: 124 us against 43 + 58).
bool rev_in_candidates(int64_t N, bool batch) { return !batch && N < kFewAtoms; }

template <bool BATCH, int G>
static void launch_filter_rows_g(const BuildArgs& b, const StructInfo& st0, const double* ref, const StructInfo* st_ref,
                                 const Lists& V, const Lists& L, hipStream_t s) {
  const auto kernel = st0.mode == kModeImages ? k_filter_rows<BATCH, true, G> : k_filter_rows<BATCH, false, G>;
  hipLaunchKernelGGL(kernel, grid_for(b.N * G), dim3(kBlock), 0, s, b.pos, b.N, b.sid, b.structs, st0, ref, st_ref, V,
                     b.rcR2, b.rcA2, L, b.overflow);
}

template <int G>
static void launch_filter_g(const BuildArgs& b, const StructInfo& st0, bool batch, const double* ref,
                            const StructInfo* st_ref, const Lists& V, const Lists& L, float4* disp, hipStream_t s) {
  const dim3 grid = grid_for(b.N * G);
  batch ? launch_filter_rows_g<true, G>(b, st0, ref, st_ref, V, L, s)
        : launch_filter_rows_g<false, G>(b, st0, ref, st_ref, V, L, s);
  if (batch)
    hipLaunchKernelGGL((k_reverse_from_candidates<true, G>), grid, dim3(kBlock), 0, s, b.N, V, L,
                       b.pos, b.types, b.sid, b.structs, disp, b.overflow + 2);
  else if (!rev_in_candidates(b.N, batch))
    hipLaunchKernelGGL((k_reverse_from_candidates<false, G>), grid, dim3(kBlock), 0, s, b.N, V, L,
                       (const double*)nullptr, (const int32_t*)nullptr, (const int32_t*)nullptr,
                       (const StructInfo*)nullptr, (float4*)nullptr, b.overflow + 2);
}

void launch_filter_rows(const BuildArgs& b, const StructInfo& st0, bool batch, const double* ref,
                        const StructInfo* st_ref, const Lists& V, const Lists& L, float4* disp, hipStream_t s) {
  if (b.N < kFewAtoms) launch_filter_g<16>(b, st0, batch, ref, st_ref, V, L, disp, s);
  else launch_filter_g<4>(b, st0, batch, ref, st_ref, V, L, disp, s);
}

// flag = any atom whose displacement since the last build, plus horizon
// times its speed when vel is given, exceeds half the skin: |r_i - r_i(build)|
// + horizon |v_i| > sqrt(thr2) (the plain test |r_i - r_i(build)|^2 > thr2
// when horizon is 0).  With a box scaled by mu since the build (NPT), a pair
// within r_c now was within r_c + skin then as long as every
// |r_i - mu r_i(build)| <= (mu (r_c + skin) - r_c) / 2.
__global__ void k_check_displacement(const double* __restrict__ pos, const double* __restrict__ ref,
                                     const double* __restrict__ vel, int64_t N, double thr2,
                                     double horizon, int32_t* __restrict__ flag,
                                     const double* __restrict__ mu_cum, double rc, double rl) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double m = 1.0, t2 = thr2;
  if (mu_cum) {
    m = *mu_cum;
    const double a = fmax(0.0, 0.5 * (m * rl - rc));
    t2 = a * a;
  }
  const double dx = pos[i] - m * ref[i], dy = pos[N + i] - m * ref[N + i],
               dz = pos[2 * N + i] - m * ref[2 * N + i];
  const double d2 = dx * dx + dy * dy + dz * dz;
  bool out = d2 > t2;
  if (vel && horizon > 0.0) {
    const double vx = vel[i], vy = vel[N + i], vz = vel[2 * N + i];
    out = sqrt(d2) + horizon * sqrt(vx * vx + vy * vy + vz * vz) > sqrt(t2);
  }
  if (out) atomicExch(flag, 1);
}

void launch_check_displacement(const double* pos, const double* ref, const double* vel, int64_t N,
                               double thr2, double horizon, int32_t* flag, hipStream_t s,
                               const double* mu_cum, double rc, double rl) {
  hipLaunchKernelGGL(k_check_displacement, grid_for(N), dim3(kBlock), 0, s, pos, ref, vel, N, thr2, horizon,
                     flag, mu_cum, rc, rl);
}

int64_t type_row_blocks(int64_t N) { return div_up(N, kBlock); }

// A thread block of 1024 orders the atoms of a call this small by itself.
// Bound by the latency of its few dependent passes: LDS holds the cell
// counts and the caller indices in cell order; each atom's place in its cell
// is the number of smaller caller indices there, so the order is that of the
// other kernels.  Two launches (k_gather_atoms moves the atoms: with their
// scattered stores in the block they were no faster) for the others' nine, each
// of which is mostly its own launch at these sizes.
constexpr int kOneThreads = 1024, kOnePerThread = 6;
constexpr int kOneAtoms = kOneThreads * kOnePerThread;  // atoms, and cells

__global__ void __launch_bounds__(kOneThreads) k_order_one_block(BuildArgs b) {
  constexpr int kWaves = kOneThreads / 64, P = kOnePerThread;
  __shared__ int32_t cell[kOneAtoms], ext[kOneAtoms];
  __shared__ int32_t wsum[kWaves], wtypes[kWaves][kMaxTypes], base[kMaxTypes];
  if (gated_off(b.gate)) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int N = (int)b.N;
  const int turns = (N + kOneThreads - 1) / kOneThreads;  // atoms of a thread: t, t + 1024, ...
  // every pass below loads for all of a thread's atoms before it uses any of them
  double x[P], y[P], z[P];
  int32_t type[P], sid[P], mine[P];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q >= turns) break;
    const int e = min(t + q * kOneThreads, N - 1);
    x[q] = b.pos_ext[e];
    y[q] = b.pos_ext[N + e];
    z[q] = b.pos_ext[2 * N + e];
    type[q] = b.types_ext[e];
    sid[q] = struct_of(b, e);
    mine[q] = b.ext_src ? b.ext_src[e] : e;  // its caller index
  }
  for (int c = t; c < b.n_cells; c += kOneThreads) cell[c] = 0;
  if (b.check && t < 8) {
    b.check[t] = 0;
    __threadfence();  // before other threads' atomics on them
  }
  __syncthreads();
  int key[P];   // cell of the thread's atoms; ~cell in a structure without cells, whose atoms keep
  int from[P];  // their order from its first
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q >= turns) break;
    const int e = t + q * kOneThreads;
    const StructInfo& st = b.structs[sid[q]];
    from[q] = (int)st.start;
    key[q] = ~st.cell_off;
    if (st.mode == kModeCells) key[q] = cell_of(st, x[q], y[q], z[q]);
    if (e >= N) continue;
    if (rows_by_ranges(b)) b.key[e] = key[q];
    if (key[q] >= 0) atomicAdd(&cell[key[q]], 1);
    else if (e == st.start) cell[st.cell_off] = (int32_t)st.count;
  }
  __syncthreads();
  // exclusive scan of the counts, a run of cells to a thread
  {
    const int per = (b.n_cells + kOneThreads - 1) / kOneThreads, lo = min(t * per, b.n_cells),
              hi = min(lo + per, b.n_cells);
    int32_t sum = 0;
    for (int c = lo; c < hi; ++c) sum += cell[c];
    int32_t run = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t v = __shfl_up(run, off);
      if (lane >= off) run += v;
    }
    if (lane == 63) wsum[w] = run;
    __syncthreads();
    run -= sum;
    for (int v = 0; v < w; ++v) run += wsum[v];
    for (int c = lo; c < hi; ++c) {
      const int32_t n = cell[c];
      b.cell_start[c] = run;
      b.cell_count[c] = n;
      cell[c] = run;
      run += n;
    }
  }
  __syncthreads();
  int begin[P];  // first place of the atom's cell
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q >= turns) break;
    begin[q] = b.cell_start[key[q] < 0 ? ~key[q] : key[q]];
  }
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q >= turns) break;
    if (t + q * kOneThreads < N && key[q] >= 0) ext[atomicAdd(&cell[key[q]], 1)] = mine[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q >= turns) break;
    const int e = t + q * kOneThreads;
    if (e >= N) continue;
    int k = begin[q];
    if (key[q] < 0) {
      k += e - from[q];
    } else {
      const int end = cell[key[q]];  // where its last atom went
      for (int p = begin[q]; p < end; p += 4) {
        int32_t other[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) other[u] = ext[min(p + u, end - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) k += p + u < end && other[u] < mine[q] ? 1 : 0;
      }
    }
    begin[q] = k;  // from here on: its place
  }
  __syncthreads();
  const int Tn = b.per_type ? b.n_types : 1;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q >= turns) break;
    const int e = t + q * kOneThreads;
    if (e < N) cell[begin[q]] = e | (b.per_type ? min(max(type[q], 0), Tn - 1) : 0) << 16;
  }
  __syncthreads();
  int sp[P];  // species of the internal atoms t, t + 1024, ...
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int k = t + q * kOneThreads;
    sp[q] = -1;
    if (k >= N) continue;
    b.perm[k] = cell[k] & 0xffff;
    sp[q] = cell[k] >> 16;
  }
  if (!b.rows) return;
  // the species-grouped rows: species counts, their starts, then ranks in internal order
  for (int64_t r = t; r < b.rows_len; r += kOneThreads) b.rows[r] = -1;
  if (t < kMaxTypes) base[t] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < P; ++q)
    for (int s = 0; s < Tn; ++s) {
      const uint64_t m = __ballot(sp[q] == s);
      if (lane == 0 && m) atomicAdd(&base[s], (int32_t)__popcll(m));
    }
  __syncthreads();
  if (t == 0) {
    int32_t o = 0;
    for (int s = 0; s < Tn; ++s) {
      const int32_t n = base[s];
      base[s] = o;
      o += (n + kRowGroup - 1) / kRowGroup * kRowGroup;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (q * kOneThreads >= N) break;
    int rank = 0;
    for (int s = 0; s < Tn; ++s) {
      const uint64_t m = __ballot(sp[q] == s);
      if (sp[q] == s) rank = lanes_below(m);
      if (lane == 0) wtypes[w][s] = __popcll(m);
    }
    __syncthreads();
    if (sp[q] >= 0) {
      for (int v = 0; v < w; ++v) rank += wtypes[v][sp[q]];
      b.rows[base[sp[q]] + rank] = t + q * kOneThreads;
    }
    __syncthreads();
    if (t < Tn)
      for (int v = 0; v < kWaves; ++v) base[t] += wtypes[v][t];
    __syncthreads();
  }
}

void launch_order_atoms(const BuildArgs& b, hipStream_t s) {
  const int32_t* g = b.gate;
  // one block up to the size where the chip's share of the work makes up for the launches:
  // 12 us against 28 for 256 atoms, 20 : 41 for 2,048, 28 : 42 for 4,000, 35 : 41 for 5,324,
  // 42 : 40 for 6,912 (and its LDS holds a word per cell and per atom)
  if (b.N <= kOneAtoms && b.n_cells <= kOneAtoms) {
    hipLaunchKernelGGL(k_order_one_block, dim3(1), dim3(kOneThreads), 0, s, b);
    hipLaunchKernelGGL(k_gather_atoms, grid_for(b.N), dim3(kBlock), 0, s, b, false);
    return;
  }
  hipLaunchKernelGGL(k_fill_cells, grid_for(std::max<int64_t>(b.n_cells, 8)), dim3(kBlock), 0, s, b);
  hipLaunchKernelGGL(k_cell_key, grid_for(b.N), dim3(kBlock), 0, s, b);
  hipLaunchKernelGGL(k_scan_1block, dim3(1), dim3(1024), 0, s, b.cell_count, b.cell_start, b.n_cells, g);
  hipLaunchKernelGGL(k_cell_scatter, grid_for(b.N), dim3(kBlock), 0, s, b);
  // cells as large as the cutoff asks for hold tens of atoms: a wave each
  const bool ranked = b.cell_rows && (b.coarse || b.n_cells > kMaxBlocks);
  if (ranked)
    hipLaunchKernelGGL(k_cell_rank, grid_for(b.N), dim3(kBlock), 0, s, b);
  else if (b.cell_rows)
    hipLaunchKernelGGL(k_cell_sort, dim3(div_up(b.n_cells, kBlock / 64)), dim3(kBlock), 0, s, b.cell_start,
                       b.cell_count, b.cell_fill, b.n_cells, b.ext_src, b.perm, g);
  hipLaunchKernelGGL(k_gather_atoms, grid_for(b.N), dim3(kBlock), 0, s, b, ranked);
  if (!b.rows) return;
  const int32_t Tn = b.per_type ? b.n_types : 1;
  const int32_t nb = (int32_t)type_row_blocks(b.N);
  hipLaunchKernelGGL(k_type_block_count, dim3(nb), dim3(kBlock), 0, s, b.types, b.N, Tn, b.per_type, nb, b.tblk,
                     b.rows, b.rows_len, g);
  hipLaunchKernelGGL(k_scan_1block, dim3(1), dim3(1024), 0, s, b.tblk, b.tex, Tn * nb, g);
  hipLaunchKernelGGL(k_type_block_scatter, dim3(nb), dim3(kBlock), 0, s, b.types, b.N, Tn, b.per_type, nb, b.tex,
                     b.rows, g);
}

}  // namespace nep
