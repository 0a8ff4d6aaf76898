// descriptor.hip -- descriptor pass of NEP3 (eqs. qin, g_n, f_n, S_nk and the
// explicit q_{nl}, q_{n222}, q_{n1111}; Sec. II.B-II.D).
//
//   * radial: q_n = sum_j sum_k c^{t_i t_j}_{nk} f_k(r_ij) is regrouped as
//     sum_t sum_k c^{t_i t}_{nk} F_{t,k} with F_{t,k} = sum_{j of species t}
//     f_k(r_ij); a bond adds the outer product of its species' unit vector
//     and its f to F, lane s of the quad holding species s;
//   * angular: S_{n,k} += g_n(r) b_k(u), the outer product of the bond's
//     radial functions and polynomials; lane s of the quad holds n = 4u + s,
//     which is what q_{nl}, q_{n222}, q_{n1111} of one n need.
// One walk over the row: its angular prefix feeds both sums, the rest F
// alone.  The four bonds of a quad are computed one per lane, transposed
// (lane = component) and accumulated in row order, so S and F are the same
// bits as a sequential sum over the row.
//
// Bound by instruction issue: about 265 vector and 100 matrix instructions
// per 64 bonds at l_max = 4, n_A = 7.  With the sums in registers of one lane
// per atom (168 of them) or repeated in four lanes the same work took 126 us
// for 131,072 atoms of the 4-species alloy and 40 us for 2,048; with the quad
// it takes 102 and 10 us (2,000,000 atoms, l_max = 6: 3.23 -> 2.07 ms), at
// three waves per SIMD (163 registers).
#include "pair.h"

namespace nep {

template <int NT, int L, bool BATCH, int Q, int SH>
__global__ void __launch_bounds__(kBlock, 2) k_descriptor(EvalArgs a, StructInfo st0) {
  if (rows_refused(a)) return;
  constexpr int NB = num_poly(L), NBT = (NB + 3) / 4;
  using Sh = BasisShape<SH>;
  constexpr int KT = SH ? (Sh::KR + 3) / 4 : kMaxBasis / 4;  // basis tiles of F
  extern __shared__ float4 lds_v4[];  // 16-byte aligned base
  float* sR = reinterpret_cast<float*>(lds_v4);
  const DevModel& M = a.M;
  const int T = M.T;
  const int KR = SH ? Sh::KR : M.KR, KA = SH ? Sh::KA : M.KA, nR = SH ? Sh::nR : M.nR, nA = SH ? Sh::nA : M.nA;
  const int WR = round4(nR);
  constexpr int W = 4 * NT;
  float* sA = sR + radial_table_floats(M);
  load_tables(M, M.cA, sR, sA);
  __syncthreads();
  const int64_t N = a.N;
  const int sub = threadIdx.x & (4 * Q - 1), s = threadIdx.x & 3, quad = sub >> 2;
  const int64_t i0 = (xcd_block() * kBlock + threadIdx.x) / (4 * Q);
  const bool live = i0 < N;
  const int64_t i = live ? i0 : N - 1;  // lanes past the last atom compute on no entries
  const int ti = a.types[i];
  const int nnR = live ? min(a.L.nnR[i], a.L.MR) : 0, nnA = live ? min(a.L.nnA[i], a.L.MR) : 0;
  const int steps = wave_max((nnR + 4 * Q - 1) / (4 * Q)), stepsA = wave_max((nnA + 4 * Q - 1) / (4 * Q));
  const QuadIdentity I;
  const Frame fr(st0);
  const float rcR = M.rcR, rcA = M.rcA;

  quad4 F[KT];  // of the species t_first + lane
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) F[kt] = quad4{0.f, 0.f, 0.f, 0.f};
  // F_{t,k} += [t_j = t] f_k of the quad's four bonds, in row order
  auto add_radial = [&](bool in, int32_t tj, float r, int t_first) __attribute__((always_inline)) {
    const Basis bs = make_basis(r, rcR);
    float f[4 * KT];
    f[0] = bs.fc;
    float Tm1 = 1.f, Tk = bs.x;
#pragma unroll
    for (int k = 1; k < 4 * KT; ++k) {
      f[k] = 0.f;
      if (k >= KR) continue;
      f[k] = fmaf(Tk, 0.5f, 0.5f) * bs.fc;
      const float Tn = 2.f * bs.x * Tk - Tm1;
      Tm1 = Tk;
      Tk = Tn;
    }
    const int32_t tq = in ? tj - t_first : -1;
    const float o0 = quad_bcast<0>(tq) == s ? 1.f : 0.f, o1 = quad_bcast<1>(tq) == s ? 1.f : 0.f;
    const float o2 = quad_bcast<2>(tq) == s ? 1.f : 0.f, o3 = quad_bcast<3>(tq) == s ? 1.f : 0.f;
    static_for<0, KT>([&](auto tile) __attribute__((always_inline)) {
      constexpr int kt = decltype(tile)::value;
      if (!SH && 4 * kt >= KR) return;
      constexpr int live_k = SH ? (Sh::KR - 4 * kt < 4 ? Sh::KR - 4 * kt : 4) : 4;
      const quad4 x = I.transpose<live_k>(f[4 * kt], f[4 * kt + 1], f[4 * kt + 2], f[4 * kt + 3]);
      F[kt] = quad_mfma(x[0], o0, F[kt]);
      F[kt] = quad_mfma(x[1], o1, F[kt]);
      F[kt] = quad_mfma(x[2], o2, F[kt]);
      F[kt] = quad_mfma(x[3], o3, F[kt]);
    });
  };
  // S_{n,k} += g_n(r) b_k(u) of the quad's four bonds, in row order
  quad4 S[NT][NBT];
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int t = 0; t < NBT; ++t) S[u][t] = quad4{0.f, 0.f, 0.f, 0.f};
  auto add_angular = [&](bool in, int32_t tj, float r, float x, float y, float z) __attribute__((always_inline)) {
    const Basis bs = make_basis(r, rcA);
    const float* c = sA + (ti * T + tj) * M.cA_pair;
    float gq[W];
    {
      float cv[W];
      load_group<NT>(c, cv);
#pragma unroll
      for (int q = 0; q < W; ++q) gq[q] = cv[q] * bs.fc;
    }
    float Tm1 = 1.f, Tk = bs.x;
#pragma unroll
    for (int k = 1; k < kMaxBasis; ++k) {
      if (k >= KA) break;
      float cv[W];
      load_group<NT>(c + k * W, cv);
      const float f = fmaf(Tk, 0.5f, 0.5f) * bs.fc;
#pragma unroll
      for (int q = 0; q < W; ++q)
        if (!SH || q < nA) gq[q] += cv[q] * f;
      const float Tn = 2.f * bs.x * Tk - Tm1;
      Tm1 = Tk;
      Tk = Tn;
    }
    quad4 gT[NT];
    static_for<0, NT>([&](auto tile) __attribute__((always_inline)) {
      constexpr int u = decltype(tile)::value;
      constexpr int live_n = SH ? (Sh::nA - 4 * u < 4 ? Sh::nA - 4 * u : 4) : 4;
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = in ? gq[4 * u + q] : 0.f;
      gT[u] = I.transpose<live_n>(v[0], v[1], v[2], v[3]);
    });
    float b4[4] = {0.f, 0.f, 0.f, 0.f};
    angular_values<L>(x, y, z, [&](int k, float b) __attribute__((always_inline)) {
      b4[k & 3] = b;
      if ((k & 3) == 3 || k == NB - 1) {
        const quad4 bT = I.transpose<4>(b4[0], b4[1], b4[2], b4[3]);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int u = 0; u < NT; ++u) S[u][k / 4] = quad_mfma(bT[v], gT[u][v], S[u][k / 4]);
        b4[0] = b4[1] = b4[2] = b4[3] = 0.f;
      }
    });
  };
  walk_row<BATCH>(a, fr, i, sub, nnR, 4 * Q, steps,
                  [&](int k, int m, int64_t, int32_t tj, float fx, float fy, float fz) __attribute__((always_inline)) {
    float r, rinv;
    length_of(fx * fx + fy * fy + fz * fz, r, rinv);
    add_radial(m < nnR, tj, r, 0);
    if (k < stepsA) add_angular(m < nnA, tj, r, fx * rinv, fy * rinv, fz * rinv);
  });

  // ---- q_n = sum_t sum_k c^{t_i t}_{nk} F_{t,k}: lane s takes n = 4s .. 4s + 3 ----
  float qr[4] = {0.f, 0.f, 0.f, 0.f};
  auto contract_radial = [&](int t_first) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int k = 0; k < 4; ++k) F[kt][k] = quads_sum<Q>(F[kt][k]);
    static_for<0, 4>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      const int t = t_first + X;
      if (t >= T) return;
      const float* c = sR + (ti * T + t) * KR * WR + min(4 * s, WR - 4);
      static_for<0, 4 * KT>([&](auto kk) __attribute__((always_inline)) {
        constexpr int k = decltype(kk)::value;
        if (k >= KR) return;
        const float Ftk = quad_bcast<X>(F[k / 4][k % 4]);
        const float4 c4 = *reinterpret_cast<const float4*>(c + k * WR);
        qr[0] += c4.x * Ftk;
        qr[1] += c4.y * Ftk;
        qr[2] += c4.z * Ftk;
        qr[3] += c4.w * Ftk;
      });
    });
  };
  contract_radial(0);
  if (T > 4) {  // models of more than four species walk the row again for the others
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) F[kt] = quad4{0.f, 0.f, 0.f, 0.f};
    walk_row<BATCH>(a, fr, i, sub, nnR, 4 * Q, steps,
                    [&](int, int m, int64_t, int32_t tj, float fx, float fy, float fz) __attribute__((always_inline)) {
      float r, rinv;
      length_of(fx * fx + fy * fy + fz * fz, r, rinv);
      add_radial(m < nnR, tj, r, 4);
    });
    contract_radial(4);
  }
  float* __restrict__ qrow = a.q + i * M.NDp;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (live && 4 * s + u < nR && quad == (Q > 1 ? u % Q : 0)) qrow[4 * s + u] = qr[u];

  // ---- q_{nl} = sum_{k in l} C3_k S_{nk}^2; q_{n222}; q_{n1111}: lane s takes n = 4u + s ----
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    float z[4 * NBT];
#pragma unroll
    for (int t = 0; t < NBT; ++t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) z[4 * t + k] = quads_sum<Q>(S[u][t][k]);
      if (live && quad == (Q > 1 ? t % Q : 0))
        reinterpret_cast<float4*>(a.sums)[sums_slot(u * NBT + t, N, i, s)] =
            make_float4(z[4 * t], z[4 * t + 1], z[4 * t + 2], z[4 * t + 3]);
    }
    const int n = 4 * u + s;
    if (!live || n >= nA || quad != 0) continue;
    float v[L];
#pragma unroll
    for (int l = 0; l < L; ++l) v[l] = 0.f;
#pragma unroll
    for (int k = 0; k < NB; ++k) v[degree_of(k) - 1] += M.C3[k] * z[k] * z[k];
#pragma unroll
    for (int l = 1; l <= L; ++l) qrow[nR + (l - 1) * nA + n] = v[l - 1];
    if constexpr (L >= 2) {
      if (M.has4b) {
        const float v4 = M.C4[0] * z[3] * z[3] * z[3] + M.C4[1] * z[3] * (z[4] * z[4] + z[5] * z[5]) +
                         M.C4[2] * z[3] * (z[6] * z[6] + z[7] * z[7]) +
                         M.C4[3] * z[6] * (z[5] * z[5] - z[4] * z[4]) + M.C4[4] * z[4] * z[5] * z[7];
        qrow[nR + L * nA + n] = v4;
      }
    }
    if (M.has5b) {
      const float z12 = z[1] * z[1] + z[2] * z[2];
      const float v5 = M.C5[0] * z[0] * z[0] * z[0] * z[0] + M.C5[1] * z[0] * z[0] * z12 + M.C5[2] * z12 * z12;
      qrow[nR + (L + M.has4b) * nA + n] = v5;
    }
  }
  if (live && sub == 0)
    for (int c = M.ND; c < M.NDp; ++c) qrow[c] = 0.f;
}

bool launch_descriptor(const EvalArgs& a, hipStream_t s) {
  return dispatch_pair(a, [&](auto nt, auto l, auto batch, auto q, auto sh) {
    constexpr int NT = decltype(nt)::value, L = decltype(l)::value, Q = decltype(q)::value, S = decltype(sh)::value;
    constexpr bool B = decltype(batch)::value;
    const size_t lds = pair_table_bytes(a.M);
    if (lds > 64 * 1024) return false;
    hipLaunchKernelGGL((k_descriptor<NT, L, B, Q, S>), dim3((unsigned)div_up(a.N * 4 * Q, kBlock)), dim3(kBlock), lds, s,
                       a, a.st0);
    return true;
  });
}

}  // namespace nep
