// force.hip -- partial forces dU_i/dr_ij (eq. partial_force) and the force and
// virial gather (eqs. F_ij, F_i, virial) of NEP3.
//
// Partial forces: dU_i/dr_ij for every radial entry.  The radial part uses
// per-atom tables A_{t,k} = sum_n dU/dq_n c^{t_i t}_{nk} in LDS.  The angular
// part of a bond is
//   sum_{n,k} D_{nk} [g'_n b_k u + g_n d b_k / d r_ij],  D_{nk} = dU/dS_{nk},
// two products with the atom's D: w_k = sum_n g_n D_{nk}, the weights of the
// polynomials' gradients, and w'_k = sum_n g'_n D_{nk}, those of the
// polynomials themselves.  Both run on the quad's matrix product with the
// quad's four bonds as columns, so every lane gets the w and w' of its own
// bond without moving data, and D is spread over the quad, lane = polynomial
// (a lane per bond would hold all of it: 168 registers for n_A = 7, l_max =
// 4, where the quad holds 42).
// Bound by instruction issue: about 360 vector and 84 matrix instructions
// per 64 bonds at l_max = 4, n_A = 7, in one walk over the row.  Two walks with
// a lane per atom (half of D in registers each time) took 218 us for 131,072
// atoms of the 4-species alloy and 37 us for 2,048; this takes 128 and 11.6 us
// (2,000,000 atoms, l_max = 6: 7.2 -> 2.6 ms).  The sums over n and the
// gradients would not fit one lane: D alone is 168 registers.
// Gather: F_i = sum_j dU_i/dr_ij - dU_j/dr_ji and W_i = sum_j r_ij (x)
//   dU_j/dr_ji over the radial row, reading dU_j/dr_ji through the reverse
//   index: no atomics, so results are bitwise reproducible.  The first sum
//   comes from the force pass.  Bound by the cache lines its reads touch: the
//   partial forces lie in rows of an atom, where the entries next to the one
//   an atom reads belong to the atoms next to it (131,072 atoms: 73 us with
//   the entries of neighbouring atoms side by side and both sums read, 68 with
//   one sum, 58 in rows; 2,000,000 atoms: 1295, 1208, 1064).
#include "pair.h"

namespace nep {

// Sum of v over the G adjacent lanes of one atom (4 or 16); every lane of the
// group gets the same bits (the pairwise adds commute).
template <int G>
__device__ __forceinline__ float group_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false));
  if constexpr (G == 16) {  // the mirrored half row, then the mirrored row
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, false));
  }
  return v;
}

// Three waves per SIMD where D leaves the registers for them: 72 words of it do
// with two or three spilled (132,000 atoms of the 3-species training model: 171 us
// against 193 with two waves), the 96 of n_A = 8, l_max = 6 would spill 18 (2.94 ms
// against 2.66 for 2,000,000 atoms).
template <int NT, int L, bool BATCH, int Q, int SH>
__global__ void __launch_bounds__(kBlock, NT * num_poly(L) <= 72 ? 3 : 2) k_partial_forces(EvalArgs a, StructInfo st0) {
  constexpr int NB = num_poly(L), NBT = (NB + 3) / 4;
  constexpr int kAtoms = 64 / (4 * Q);  // atoms of a wave
  using Sh = BasisShape<SH>;
  extern __shared__ float4 lds_v4[];  // 16-byte aligned base
  if (rows_refused(a)) return;
  float* sR = reinterpret_cast<float*>(lds_v4);
  const DevModel& M = a.M;
  const int T = M.T;
  const int KR = SH ? Sh::KR : M.KR, KA = SH ? Sh::KA : M.KA, nR = SH ? Sh::nR : M.nR, nA = SH ? Sh::nA : M.nA;
  const int WR = round4(nR);
  constexpr int W = 4 * NT;
  float* sA = sR + radial_table_floats(M);
  const int KRp = KR | 1;  // an odd stride spreads the species over the banks
  const int lane = threadIdx.x & 63;
  float* At = sA + T * T * M.cA_pair + (threadIdx.x >> 6) * (T * KRp * kAtoms) + lane / (4 * Q);
  const int64_t N = a.N;
  const int sub = lane & (4 * Q - 1), s = lane & 3;
  const int64_t i0 = (xcd_block() * kBlock + threadIdx.x) / (4 * Q);
  const bool live = i0 < N;
  const int64_t i = live ? i0 : N - 1;  // lanes past the last atom compute on no entries
  // the atom's words are on their way while the block stages the tables
  const int ti = a.types[i];
  const float* __restrict__ fprow = a.fp + i * M.NDp;
  const int nnR = live ? min(a.L.nnR[i], a.L.MR) : 0, nnA = live ? min(a.L.nnA[i], a.L.MR) : 0;
  float fpr[kMaxBasis];
#pragma unroll
  for (int n = 0; n < kMaxBasis; ++n) fpr[n] = n < nR ? fprow[n] : 0.f;
  float4 z4[NT][NBT];
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int t = 0; t < NBT; ++t) z4[u][t] = reinterpret_cast<const float4*>(a.sums)[sums_slot(u * NBT + t, N, i, s)];
  load_tables(M, M.cS, sR, sA);
  __syncthreads();
  const QuadIdentity I;
  const Frame fr(st0);
  const float rcR = M.rcR, rcA = M.rcA;
  const int steps = wave_max((nnR + 4 * Q - 1) / (4 * Q)), stepsA = wave_max((nnA + 4 * Q - 1) / (4 * Q));

  // ---- radial: A_{t,k} = sum_n dU/dq_n c^{t_i t}_{nk}; dU_i/dr_ij = (sum_k A f'_k) u, as a
  // Chebyshev series like the angular table; a lane takes whole species, and only
  // the wave's own lanes read them ----
  for (int t = sub; t < T; t += 4 * Q) {
    const float* c = sR + (ti * T + t) * KR * WR;
    float sum = 0.f;
    for (int k = KR - 1; k >= 0; --k) {
      float v = 0.f;
#pragma unroll
      for (int n4 = 0; n4 < kMaxBasis / 4; ++n4) {
        if (4 * n4 >= nR) break;
        const float4 x = *reinterpret_cast<const float4*>(c + k * WR + 4 * n4);
        v += fpr[4 * n4] * x.x;
        v += fpr[4 * n4 + 1] * x.y;
        v += fpr[4 * n4 + 2] * x.z;
        v += fpr[4 * n4 + 3] * x.w;
      }
      if (k > 0) {
        v *= 0.5f;
        sum += v;
      } else {
        v += sum;
      }
      At[(t * KRp + k) * kAtoms] = v;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // radial scalar v with dU_i/dr_ij (radial part) = v r_ij: the series h of
  // T_k and dh of T'_k = k U_{k-1}, times the cutoff's f_c' and x' f_c
  auto radial_scalar = [&](int32_t tj, float r, float rinv) __attribute__((always_inline)) {
    const Basis bs = make_basis(r, rcR);
    const float* At_j = At + tj * KRp * kAtoms;
    float h = At_j[0], dh = 0.f;
    const float x2 = 2.f * bs.x;
    float Tm = 1.f, Tk = bs.x, Um = 0.f, Uk = 1.f;
#pragma unroll
    for (int k = 1; k < kMaxBasis; ++k) {
      if (k >= KR) break;
      const float A = At_j[k * kAtoms];
      h += A * Tk;
      dh += A * ((float)k * Uk);
      const float Tn = x2 * Tk - Tm, Un = x2 * Uk - Um;
      Tm = Tk;
      Tk = Tn;
      Um = Uk;
      Uk = Un;
    }
    return (h * bs.dfc + dh * (bs.dxdr * bs.fc)) * rinv;
  };

  // ---- D_{nk} = dU/dS_{nk} through q_{nl}, q_{n222}, q_{n1111}: lane s takes n = 4u + s,
  // then spread with lane = polynomial: D[t][u][r] is that of n = 4u + r and the
  // scaled polynomial of slot 4t + s ----
  quad4 D[NBT][NT];
  {
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int n = min(4 * u + s, nA - 1);
      const bool on = 4 * u + s < nA;
      float z[4 * NBT], d[4 * NBT];
#pragma unroll
      for (int t = 0; t < NBT; ++t) {
        z[4 * t] = z4[u][t].x;
        z[4 * t + 1] = z4[u][t].y;
        z[4 * t + 2] = z4[u][t].z;
        z[4 * t + 3] = z4[u][t].w;
      }
      float f3[L];
#pragma unroll
      for (int l = 1; l <= L; ++l) f3[l - 1] = on ? fprow[nR + (l - 1) * nA + n] : 0.f;
#pragma unroll
      for (int k = 0; k < NB; ++k) d[k] = 2.f * M.C3[k] * f3[degree_of(k) - 1] * z[k];
      if constexpr (L >= 2) {
        if (M.has4b) {
          const float f = on ? fprow[nR + L * nA + n] : 0.f;
          const float* C = M.C4;
          d[3] += f * (3.f * C[0] * z[3] * z[3] + C[1] * (z[4] * z[4] + z[5] * z[5]) +
                       C[2] * (z[6] * z[6] + z[7] * z[7]));
          d[4] += f * (2.f * C[1] * z[3] * z[4] - 2.f * C[3] * z[6] * z[4] + C[4] * z[5] * z[7]);
          d[5] += f * (2.f * C[1] * z[3] * z[5] + 2.f * C[3] * z[6] * z[5] + C[4] * z[4] * z[7]);
          d[6] += f * (2.f * C[2] * z[3] * z[6] + C[3] * (z[5] * z[5] - z[4] * z[4]));
          d[7] += f * (2.f * C[2] * z[3] * z[7] + C[4] * z[4] * z[5]);
        }
      }
      if (M.has5b) {
        const float f = on ? fprow[nR + (L + M.has4b) * nA + n] : 0.f;
        const float* C = M.C5;
        const float z12 = z[1] * z[1] + z[2] * z[2];
        d[0] += f * (4.f * C[0] * z[0] * z[0] * z[0] + 2.f * C[1] * z[0] * z12);
        d[1] += f * (2.f * C[1] * z[0] * z[0] * z[1] + 4.f * C[2] * z12 * z[1]);
        d[2] += f * (2.f * C[1] * z[0] * z[0] * z[2] + 4.f * C[2] * z12 * z[2]);
      }
      static_for<0, NBT>([&](auto tile) __attribute__((always_inline)) {
        constexpr int t = decltype(tile)::value;
        float x[4] = {0.f, 0.f, 0.f, 0.f};
        static_for<0, 4>([&](auto j) __attribute__((always_inline)) {
          constexpr int slot = 4 * t + decltype(j)::value;
          if constexpr (slot < NB) {
            constexpr Harmonic o = harmonic_at(slot, L);
            x[decltype(j)::value] = (float)o.scale * d[o.k];
          }
        });
        D[t][u] = I.transpose<4>(x[0], x[1], x[2], x[3]);
      });
    }
  }

  // angular part of a bond: dU_i/dr_ij = (returned) r_ij + V / r
  auto angular = [&](int32_t tj, float r, float rinv, float x, float y, float z, float on, float& Vx, float& Vy,
                     float& Vz) __attribute__((always_inline)) {
    // g_n = f_c G_n and g'_n = f_c' G_n + x' f_c H_n with G the series of T_k, H that of T'_k
    float G[W], H[W];
    {
      const Basis bs = make_basis(r, rcA);
      const float* c = sA + (ti * T + tj) * M.cA_pair;
      load_group<NT>(c, G);
#pragma unroll
      for (int q = 0; q < W; ++q) H[q] = 0.f;
      const float x2 = 2.f * bs.x;
      float Tm = 1.f, Tk = bs.x, Um = 0.f, Uk = 1.f;
#pragma unroll
      for (int k = 1; k < kMaxBasis; ++k) {
        if (k >= KA) break;
        float cv[W];
        load_group<NT>(c + k * W, cv);
        const float dT = (float)k * Uk;
#pragma unroll
        for (int q = 0; q < W; ++q) {
          if (SH && q >= nA) continue;
          G[q] += cv[q] * Tk;
          H[q] += cv[q] * dT;
        }
        const float Tn = x2 * Tk - Tm, Un = x2 * Uk - Um;
        Tm = Tk;
        Tk = Tn;
        Um = Uk;
        Uk = Un;
      }
      const float fc = on * bs.fc, dfc = on * bs.dfc, hx = bs.dxdr * fc;
#pragma unroll
      for (int q = 0; q < W; ++q) {
        H[q] = dfc * G[q] + hx * H[q];
        G[q] = fc * G[q];
      }
    }
    // per m: sums over l of w Q (A for cos, B for sin), of w dQ/dz (Az, Bz) and
    // of w' Q, w_k = sum_n g_n D_nk and w'_k = sum_n g'_n D_nk
    const float zz = z * z;
    float v = 0.f;  // sum_k w'_k b_k; V: grad sum_k w_k b_k
    float Cm = 1.f, Sm = 0.f, Cp = 0.f, Sp = 0.f;  // of this m, and of m - 1
    quad4 w4, d4;
    static_for<0, L + 1>([&](auto mm) __attribute__((always_inline)) {
      constexpr int m = decltype(mm)::value;
      constexpr int l0 = m > 1 ? m : 1;
      // slots before this m: m = 0 has L, every m' > 0 has 2 (L - m' + 1)
      constexpr int first = m == 0 ? 0 : L + (m - 1) * (2 * L - m + 2);
      float A[2] = {0.f, 0.f}, Az[2] = {0.f, 0.f}, dA[2] = {0.f, 0.f};
      static_for<0, (m ? 2 : 1) * (L - l0 + 1)>([&](auto jj) __attribute__((always_inline)) {
        constexpr int slot = first + decltype(jj)::value;
        constexpr Harmonic o = harmonic_at(slot, L);
        static_assert(o.m == m, "slot order");
        if constexpr (slot % 4 == 0) {
          w4 = d4 = quad4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < W; ++q) {
            if (SH && q >= nA) continue;
            w4 = quad_mfma(D[slot / 4][q / 4][q % 4], G[q], w4);
            d4 = quad_mfma(D[slot / 4][q / 4][q % 4], H[q], d4);
          }
        }
        const float w = w4[slot % 4], dw = d4[slot % 4];
        const float Q0 = monic<o.l, m>(z, zz);
        if constexpr (m > 0) A[o.sine] += w * Q0;
        if constexpr (o.l > m) Az[o.sine] += w * ((float)(o.l - m) * monic<o.l, (o.l > m ? m + 1 : m)>(z, zz));
        dA[o.sine] += dw * Q0;
      });
      if constexpr (m == 0) {
        Vz = Az[0];
        v = dA[0];
      } else {
        Vx += (float)m * (A[0] * Cp + A[1] * Sp);
        Vy += (float)m * (A[1] * Cp - A[0] * Sp);
        Vz += Az[0] * Cm + Az[1] * Sm;
        v += dA[0] * Cm + dA[1] * Sm;
      }
      Cp = Cm;
      Sp = Sm;
      Cm = x * Cp - y * Sp;
      Sm = x * Sp + y * Cp;
    });
    return (v - (x * Vx + y * Vy + z * Vz) * rinv) * rinv;  // v u + (V - (u V) u) / r
  };
  // ---- the row: the radial part of every entry, the angular part of the prefix.  A result is
  // stored while the next entry is computed, so no step waits for its own store; their sum is
  // the atom's own part of its force, which the gather then need not read again ----
  float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
  int64_t out_e = -1;
  float own[3] = {0.f, 0.f, 0.f};
  auto put = [&]() __attribute__((always_inline)) {
    if (out_e < 0) return;
    a.P[out_e] = out;
    own[0] += out.x;
    own[1] += out.y;
    own[2] += out.z;
  };
  walk_row<BATCH>(a, fr, i, sub, nnR, 4 * Q, steps,
                  [&](int k, int m, int64_t e, int32_t tj, float fx, float fy, float fz) __attribute__((always_inline)) {
    put();
    float r, rinv;
    length_of(fx * fx + fy * fy + fz * fz, r, rinv);
    float along = radial_scalar(tj, r, rinv), Vx = 0.f, Vy = 0.f, Vz = 0.f;
    if (k < stepsA) along += angular(tj, r, rinv, fx * rinv, fy * rinv, fz * rinv, m < nnA ? 1.f : 0.f, Vx, Vy, Vz);
    out = make_float4(along * fx + Vx * rinv, along * fy + Vy * rinv, along * fz + Vz * rinv, 0.f);
    out_e = m < nnR ? i * a.L.MR + m : -1;
  });
  put();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float v = group_sum<4 * Q>(own[c]);
    if (c == sub && live) a.F[(int64_t)c * N + i] = v;
  }
}

bool launch_partial_forces(const EvalArgs& a, hipStream_t s) {
  return dispatch_pair(a, [&](auto nt, auto l, auto batch, auto q, auto sh) {
    constexpr int NT = decltype(nt)::value, L = decltype(l)::value, Q = decltype(q)::value, S = decltype(sh)::value;
    constexpr bool B = decltype(batch)::value;
    // the tables, then A_{t,k} of every atom the block has at a time
    const size_t lds = pair_table_bytes(a.M) + (size_t)a.M.T * (a.M.KR | 1) * (kBlock / (4 * Q)) * sizeof(float);
    if (lds > 64 * 1024) return false;
    hipLaunchKernelGGL((k_partial_forces<NT, L, B, Q, S>), dim3((unsigned)div_up(a.N * 4 * Q, kBlock)), dim3(kBlock),
                       lds, s, a, a.st0);
    return true;
  });
}

// ---------------------------------------------------------------------------
// force and virial gather (eqs. F_ij, F_i, virial)
// ---------------------------------------------------------------------------

// G lanes per atom (4 or 16) walk its radial row (lane s takes entries
// s, s + G, ...); dU_j/dr_ji sits at position rev[m][i] of row j, and F holds
// sum_j dU_i/dr_ij.  The index words of a lane's entry after next and the partial forces (and neighbour
// position, for the virial) of its next entry are loaded while the current
// one is accumulated; the lane sums are combined with DPP sums.  Four lanes
// read whole 64-byte runs of a row; sixteen, where a quad per atom leaves
// SIMDs without a wave, shorten the chain: in us, four against sixteen, with the
// virial, 12.1 : 7.6 at 4,000 atoms, 12.5 : 12.5 at 10,976, 19.5 : 17.3 at
// 19,652, 20.8 : 25.8 at 32,000; without it 9.3 : 4.6 at 2,048.
// VIRIAL = false leaves W untouched (MD steps without a thermo row).
template <bool BATCH, bool VIRIAL, bool CAND, int G>
__global__ void __launch_bounds__(kBlock) k_gather(EvalArgs a, StructInfo st0) {
  if (rows_refused(a)) return;
  const int64_t N = a.N;
  const int sub = threadIdx.x & (G - 1);
  const int64_t i = (xcd_block() * blockDim.x + threadIdx.x) / G;
  if (i >= N) return;  // the lanes of an atom leave together
  const int nn = min(a.L.nnR[i], a.L.MR);
  // the virial's displacements: stored with the rows of a batch, else the minimum image
  const double* __restrict__ pos = a.pos;
  double xi = 0.0, yi = 0.0, zi = 0.0;
  if (VIRIAL && !BATCH) {
    xi = pos[i];
    yi = pos[N + i];
    zi = pos[2 * N + i];
  }
  struct Words {
    int32_t j, r;
    uint16_t code;
  };
  auto words = [&](int m) -> Words {
    Words w{0, 0, kCodeCenter};
    if (m < nn) {
      const int64_t e = (int64_t)m * N + i;
      w.j = a.L.nlR[e];
      w.r = a.L.revR[e];
      if (VIRIAL && !BATCH && st0.mode == kModeImages) w.code = a.L.cdR[e];
    }
    return w;
  };
  // position of the entry in its partner's row: with CAND through the filter's map of the
  // partner's candidates (its -1 is an entry without a partner: an error, kept in bounds)
  bool broken = false;
  auto position = [&](const Words& w) -> int32_t {
    if constexpr (CAND) return a.fmap[(int64_t)w.r * N + w.j];
    else return w.r;
  };
  auto partial = [&](const Words& w, int32_t p, bool in) -> float4 {
    if constexpr (CAND) {
      broken = broken || (in && p < 0);
      p = min(max(p, 0), a.L.MR - 1);
    }
    return a.P[(int64_t)w.j * a.L.MR + p];
  };
  Words w0 = words(sub), w1 = words(sub + G), w2;
  int32_t p1 = position(w0);
  float4 pji = partial(w0, p1, sub < nn);
  if constexpr (CAND) {
    w2 = words(sub + 2 * G);
    p1 = position(w1);
  }
  double px = 0.0, py = 0.0, pz = 0.0;
  float4 dq = make_float4(0.f, 0.f, 0.f, 0.f);
  if (VIRIAL && BATCH) dq = a.disp[(int64_t)min(sub, max(nn - 1, 0)) * N + i];
  if (VIRIAL && !BATCH) {
    px = pos[w0.j];
    py = pos[N + w0.j];
    pz = pos[2 * N + w0.j];
  }
  float F[3] = {0.f, 0.f, 0.f}, W[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int m = sub; m < nn; m += G) {
    const Words c = w0;
    const float4 cji = pji;
    const double cx = px, cy = py, cz = pz;
    const float4 cd = dq;
    w0 = w1;
    if constexpr (CAND) {
      w1 = w2;
      w2 = words(m + 3 * G);
      pji = partial(w0, p1, m + G < nn);
      p1 = position(w1);
    } else {
      w1 = words(m + 2 * G);
      pji = partial(w0, w0.r, true);
    }
    if (VIRIAL && BATCH) dq = a.disp[(int64_t)min(m + G, nn - 1) * N + i];
    if (VIRIAL && !BATCH) {
      px = pos[w0.j];
      py = pos[N + w0.j];
      pz = pos[2 * N + w0.j];
    }
    F[0] += cji.x;
    F[1] += cji.y;
    F[2] += cji.z;
    if constexpr (VIRIAL) {
      float d[3] = {cd.x, cd.y, cd.z};
      if constexpr (!BATCH) {
        double Dx, Dy, Dz;
        {
#pragma clang fp contract(off)
          Dx = cx - xi;
          Dy = cy - yi;
          Dz = cz - zi;
        }
        int n0, n1, n2;
        min_image(st0, Dx, Dy, Dz, n0, n1, n2);
        if (c.code != kCodeCenter) {
          int oa, ob, oc;
          split_code(c.code, oa, ob, oc);
          n0 += oa;
          n1 += ob;
          n2 += oc;
        }
        double dx, dy, dz;
        image_disp(st0, Dx, Dy, Dz, n0, n1, n2, dx, dy, dz);
        d[0] = (float)dx;
        d[1] = (float)dy;
        d[2] = (float)dz;
      }
      const float q[3] = {cji.x, cji.y, cji.z};
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) W[x * 3 + y] += d[x] * q[y];
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float other = group_sum<G>(F[c]);
    if (c == sub) {
      const float v = a.F[(int64_t)c * N + i] - other;  // the atom's own part is there
      a.F[(int64_t)c * N + i] = v;
      if (a.kick_vel) a.kick_vel[(int64_t)c * N + i] += 0.5 * a.kick_dt * a.kick_inv_mass[a.types[i]] * (double)v;
    }
  }
  if constexpr (VIRIAL) {
#pragma unroll
    for (int v = 0; v < 9; ++v) {
      const float x = group_sum<G>(W[v]);
      if (v % G == sub) a.W[(int64_t)v * N + i] = x;
    }
  }
  if (CAND && broken) atomicExch(a.rev_err, 1);
}

template <int G>
static void launch_gather_g(const EvalArgs& a, bool virial, hipStream_t s) {
  dim3 grid((unsigned)div_up(a.N * G, kBlock));
  if (a.batch) {
    if (virial) hipLaunchKernelGGL((k_gather<true, true, false, G>), grid, dim3(kBlock), 0, s, a, a.st0);
    else hipLaunchKernelGGL((k_gather<true, false, false, G>), grid, dim3(kBlock), 0, s, a, a.st0);
  } else if (a.fmap) {
    if (virial) hipLaunchKernelGGL((k_gather<false, true, true, G>), grid, dim3(kBlock), 0, s, a, a.st0);
    else hipLaunchKernelGGL((k_gather<false, false, true, G>), grid, dim3(kBlock), 0, s, a, a.st0);
  } else {
    if (virial) hipLaunchKernelGGL((k_gather<false, true, false, G>), grid, dim3(kBlock), 0, s, a, a.st0);
    else hipLaunchKernelGGL((k_gather<false, false, false, G>), grid, dim3(kBlock), 0, s, a, a.st0);
  }
}

void launch_gather_forces(const EvalArgs& a, bool virial, hipStream_t s) {
  if (a.quads == 4) launch_gather_g<16>(a, virial, s);
  else launch_gather_g<4>(a, virial, s);
}

}  // namespace nep
