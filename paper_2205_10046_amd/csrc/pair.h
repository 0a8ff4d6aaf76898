// pair.h -- what the descriptor and partial-force kernels share: the radial
// basis of a bond, the walk over an atom's row, and the matrix products of
// one atom's bonds on the 16-block 4x4 MFMA.
//
// Both kernels give a quad of four adjacent lanes to an atom (or Q = 4 quads
// to each when the atoms are too few to fill the chip): lane s of a quad
// takes the row entries m = s, s + 4, ...  v_mfma_f32_4x4x1_16b_f32 multiplies
// sixteen independent 4x1 by 1x4 products, one per quad: lane s of a quad
// supplies element s of the column and of the row, and holds column s of the
// 4x4 result, one row per register.  The contractions of NEP's angular part
// (n_A radial functions by (l_max + 1)^2 - 1 polynomials per bond) are sums
// of such products, so every quad works on its own atom with no padding
// beyond multiples of four, float32 multiply-adds in the order of the row,
// and the per-atom blocks (sums S, derivatives D) spread over four lanes.
// The matrix instructions ignore the execution mask: the loops below run the
// same number of times in every lane of a wave, and entries past a row add
// zero.
#pragma once
#include <type_traits>

#include "angular.h"
#include "nep_kernels.h"

namespace nep {

typedef float quad4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ quad4 quad_mfma(float a, float b, quad4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// Lane x's value in every lane of its quad.
template <int X>
__device__ __forceinline__ int quad_bcast(int v) {
  return __builtin_amdgcn_mov_dpp(v, X * 0x55, 0xF, 0xF, false);
}
template <int X>
__device__ __forceinline__ float quad_bcast(float v) {
  return __int_as_float(quad_bcast<X>(__float_as_int(v)));
}

// The 4x4 transpose within a quad: lane i holds x0..x3 of row i, the result's
// register i in lane j is element j of row i.  id[c] is 1 in lane c of the
// quad and 0 elsewhere, so every product is exact.
struct QuadIdentity {
  float id[4];
  __device__ __forceinline__ QuadIdentity() {
#pragma unroll
    for (int c = 0; c < 4; ++c) id[c] = (threadIdx.x & 3) == c ? 1.f : 0.f;
  }
  // (only the first C of the four columns are not zero)
  template <int C>
  __device__ __forceinline__ quad4 transpose(float x0, float x1, float x2, float x3) const {
    quad4 c = {0.f, 0.f, 0.f, 0.f};
    c = quad_mfma(x0, id[0], c);
    if constexpr (C > 1) c = quad_mfma(x1, id[1], c);
    if constexpr (C > 2) c = quad_mfma(x2, id[2], c);
    if constexpr (C > 3) c = quad_mfma(x3, id[3], c);
    return c;
  }
};

// Sum of v over the Q quads of an atom (lane s of each; Q = 1 or 4, the four
// quads being one DPP row).  Every quad gets the same bits: the first add
// pairs quads two apart, so the second one adds the same two values in
// either order.
template <int Q>
__device__ __forceinline__ float quads_sum(float v) {
  if constexpr (Q == 4) {
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, false));  // row_ror:8
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xF, 0xF, false));  // row_ror:4
  }
  return v;
}

// The largest v of the wave, in a scalar register.
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off));
  return __builtin_amdgcn_readfirstlane(v);
}

// Cutoff function and Chebyshev basis state for one bond.
struct Basis {
  float fc, dfc, x, dxdr;
};

__device__ __forceinline__ Basis make_basis(float r, float rc) {
  Basis b;
  const float rr = r * (1.0f / rc);
  // cos(pi r / rc) with the hardware cosine (argument in revolutions)
  b.fc = 0.5f + 0.5f * __builtin_amdgcn_cosf(0.5f * rr);
  b.dfc = -0.5f * (3.14159265358979f / rc) * __builtin_amdgcn_sinf(0.5f * rr);
  const float t = rr - 1.0f;
  b.x = 2.0f * t * t - 1.0f;
  b.dxdr = 4.0f * t * (1.0f / rc);
  return b;
}

// Geometry of a single structure in the form the walk uses: the inverse is
// zeroed along open directions, so no test is left in the loop.
struct Frame {
  double H[9], Hi[9];
  bool images, ortho;
  __host__ __device__ __forceinline__ explicit Frame(const StructInfo& st)
      : images(st.mode == kModeImages), ortho(st.ortho != 0) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      H[k] = st.H[k];
      Hi[k] = st.pbc[k % 3] ? st.Hi[k] : 0.0;
    }
  }
  // Displacement of an entry from the difference of the positions: the nearest
  // image, min_image's to the bit, plus the offset of its code.  The fused
  // multiply-adds of a diagonal cell round like image_disp's separate operations
  // for offsets up to two cells, where the products are exact.
  __host__ __device__ __forceinline__ void displacement(double Dx, double Dy, double Dz, uint16_t code, double& dx,
                                                        double& dy, double& dz) const {
    double n0, n1, n2;
    if (ortho) {
      n0 = rint(Dx * Hi[0]);
      n1 = rint(Dy * Hi[4]);
      n2 = rint(Dz * Hi[8]);
    } else {
      n0 = rint(bond_fraction(Hi, Dx, Dy, Dz));
      n1 = rint(bond_fraction(Hi + 1, Dx, Dy, Dz));
      n2 = rint(bond_fraction(Hi + 2, Dx, Dy, Dz));
    }
    if (images) {
      int oa, ob, oc;
      split_code(code, oa, ob, oc);
      n0 -= (double)oa;
      n1 -= (double)ob;
      n2 -= (double)oc;
    }
    dx = fma(-n0, H[0], Dx);
    dy = fma(-n1, H[4], Dy);
    dz = fma(-n2, H[8], Dz);
    if (!ortho) {
      dx -= n1 * H[3] + n2 * H[6];
      dy -= n0 * H[1] + n2 * H[7];
      dz -= n0 * H[2] + n1 * H[5];
    }
  }
};

// Visit the row entries m = sub + step k < nn of atom i, k = 0 .. iters - 1
// (iters the same in every lane of the wave), with the loads software-
// pipelined.  body(k, m, e, tj, x, y, z) gets the float32 displacement of an
// entry and its species; past the row the displacement is (1, 0, 0).
// One structure: the index of entry k + 2 and the position and species of
// entry k + 1 are in flight while entry k is computed; the displacement is the
// float64 one of the frame rounded once.
// A batch: rows come with their displacements and species (a.disp), one
// 16-byte load per entry two steps ahead: every parameter set and both
// kernels walk the same rows, and a lane then needs no structure.
template <bool BATCH, class Body>
__device__ __forceinline__ void walk_row(const EvalArgs& a, const Frame& fr, int64_t i, int sub, int nn, int step,
                                         int iters, Body&& body) {
  const int64_t N = a.N;
  if constexpr (BATCH) {
    const float4* __restrict__ disp = a.disp;
    auto entry = [&](int m) { return disp[m < nn ? (int64_t)m * N + i : i]; };
    float4 d0 = entry(sub), d1 = entry(sub + step);
    int m = sub;
    for (int k = 0; k < iters; ++k, m += step) {
      const float4 d = d0;
      d0 = d1;
      d1 = entry(m + 2 * step);
      const bool in = m < nn;
      body(k, m, (int64_t)m * N + i, in ? __float_as_int(d.w) : 0, in ? d.x : 1.f, in ? d.y : 0.f, in ? d.z : 0.f);
    }
  } else {
    const double* __restrict__ pos = a.pos;
    const int32_t* __restrict__ nl = a.L.nlR;
    const uint16_t* __restrict__ cd = a.L.cdR;
    const double xi = pos[i], yi = pos[N + i], zi = pos[2 * N + i];
    // the words of entry m as they are; replaced past the row when they are used
    auto words = [&](int m, uint16_t& code) -> int32_t {
      const int64_t e = m < nn ? (int64_t)m * N + i : i;
      code = kCodeCenter;
      if (fr.images) code = cd[e];
      return nl[e];
    };
    uint16_t c0, c1;
    int32_t j0 = words(sub, c0), j1 = words(sub + step, c1);
    j0 = sub < nn ? j0 : (int32_t)i;
    double px = pos[j0], py = pos[N + j0], pz = pos[2 * N + j0];
    int32_t t0 = a.types[j0];
    int m = sub;
    for (int k = 0; k < iters; ++k, m += step) {
      const int32_t tc = t0;
      const uint16_t cc = c0;
      const double Dx = px - xi, Dy = py - yi, Dz = pz - zi;
      j0 = m + step < nn ? j1 : (int32_t)i;
      c0 = c1;
      px = pos[j0];
      py = pos[N + j0];
      pz = pos[2 * N + j0];
      t0 = a.types[j0];
      j1 = words(m + 2 * step, c1);
      double dx, dy, dz;
      fr.displacement(Dx, Dy, Dz, cc, dx, dy, dz);
      const bool in = m < nn;
      body(k, m, (int64_t)m * N + i, tc, in ? (float)dx : 1.f, in ? (float)dy : 0.f, in ? (float)dz : 0.f);
    }
  }
}

// Length of a bond and its inverse from the squared length: the hardware
// inverse square root and one residual step for each, correctly rounded but
// for rare last-bit cases.
__device__ __forceinline__ void length_of(float r2, float& r, float& rinv) {
  const float y = __builtin_amdgcn_rsqf(r2);
  const float x = r2 * y;
  r = fmaf(fmaf(-x, x, r2), 0.5f * y, x);
  rinv = fmaf(fmaf(-r, y, 1.f), y, y);
}

// LDS: the radial table [T][T][KR][nR rounded up to 4], then an angular table
// [T x T pairs, cA_pair floats apart][KA][4 NT], both as they are in memory.
__host__ __device__ inline int radial_table_floats(const DevModel& M) {
  return M.T * M.T * M.KR * round4(M.nR);
}

__device__ __forceinline__ void load_tables(const DevModel& M, const float* angular, float* sR, float* sA) {
  const int n_r = radial_table_floats(M) / 4, n_a = M.T * M.T * M.cA_pair / 4;  // the pair stride is a multiple of 4
  const float4* __restrict__ r = reinterpret_cast<const float4*>(M.cR);
  const float4* __restrict__ g = reinterpret_cast<const float4*>(angular);
#pragma unroll 2
  for (int k = threadIdx.x; k < n_r; k += blockDim.x) reinterpret_cast<float4*>(sR)[k] = r[k];
#pragma unroll 2
  for (int k = threadIdx.x; k < n_a; k += blockDim.x) reinterpret_cast<float4*>(sA)[k] = g[k];
}

// The 4 NT coefficients at one basis index (16-byte aligned rows).
template <int NT>
__device__ __forceinline__ void load_group(const float* p, float (&c)[4 * NT]) {
#pragma unroll
  for (int v = 0; v < NT; ++v) {
    const float4 x = reinterpret_cast<const float4*>(p)[v];
    c[4 * v] = x.x;
    c[4 * v + 1] = x.y;
    c[4 * v + 2] = x.z;
    c[4 * v + 3] = x.w;
  }
}

// Basis sizes the kernels can take as constants: shape 1 is n_R = K_R = 9
// and n_A = K_A = 7 (n_max 8/6 with N_bas 8/6); with them the basis loops
// have fixed trip counts and the same arithmetic in the same order as with
// shape 0, which reads the sizes from the model.
template <int S> struct BasisShape {
  static constexpr int nR = 0, KR = 0, nA = 0, KA = 0;
};
template <> struct BasisShape<1> {
  static constexpr int nR = 9, KR = 9, nA = 7, KA = 7;
};

// Stored sums S: float4 of k = 4t .. 4t + 3 of radial function n = 4u + s at
// ((u NBT + t) N + i) 4 + s, zero beyond n_A and NB: one coalesced 16-byte
// access per lane and tile.
__device__ __forceinline__ int64_t sums_slot(int tile, int64_t N, int64_t i, int s) {
  return ((int64_t)tile * N + i) * 4 + s;
}

// Bytes of the tables above.
inline size_t pair_table_bytes(const DevModel& M) {
  return ((size_t)radial_table_floats(M) + (size_t)M.T * M.T * M.cA_pair) * sizeof(float);
}

// launch(NT, L, BATCH, Q, SH) with the constants of this model and call: NT
// tiles of four radial functions, Q quads per atom.
template <class Launch>
bool dispatch_pair(const EvalArgs& a, Launch&& launch) {
  const DevModel& M = a.M;
  const int nt = (M.nA + 3) / 4;
  const bool shape1 = M.nR == BasisShape<1>::nR && M.KR == BasisShape<1>::KR && M.nA == BasisShape<1>::nA &&
                      M.KA == BasisShape<1>::KA;
  auto with = [&](auto NT, auto L, auto SH) {
    using B0 = std::false_type;
    using B1 = std::true_type;
    using Q1 = std::integral_constant<int, 1>;
    using Q4 = std::integral_constant<int, 4>;
    if (a.quads == 4) return a.batch ? launch(NT, L, B1{}, Q4{}, SH) : launch(NT, L, B0{}, Q4{}, SH);
    if (a.quads == 1) return a.batch ? launch(NT, L, B1{}, Q1{}, SH) : launch(NT, L, B0{}, Q1{}, SH);
    return false;
  };
  auto with_l = [&](auto NT, auto SH) {
    switch (M.L) {
#define NEP_CASE(l) \
  case l: return with(NT, std::integral_constant<int, l>{}, SH);
      NEP_CASE(1) NEP_CASE(2) NEP_CASE(3) NEP_CASE(4) NEP_CASE(5) NEP_CASE(6)
#undef NEP_CASE
    }
    return false;
  };
  using S0 = std::integral_constant<int, 0>;
  if (shape1) return with_l(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
  switch (nt) {
    case 1: return with_l(std::integral_constant<int, 1>{}, S0{});
    case 2: return with_l(std::integral_constant<int, 2>{}, S0{});
    case 3: return with_l(std::integral_constant<int, 3>{}, S0{});
    case 4: return with_l(std::integral_constant<int, 4>{}, S0{});
  }
  return false;
}

}  // namespace nep
