// params.hip -- the float32 / bf16 model tables of many parameter vectors
// built on the device from their float64 vectors (the SNES population of
// Sec. II.E never leaves the GPU).  The tables are the same, bit for bit, as
// the ones the host builds for a single vector (api.cpp upload_model): the
// same layout, float64 -> float32 by round to nearest, bf16 by round to
// nearest even of the float32 value.
#include "nep_kernels.h"

namespace nep {

namespace {

__device__ __forceinline__ uint16_t bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);  // inf / nan
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Value of network weight w0[t][mu][v] of the parameter vector (0 outside
// the N_neu x N_des block: padding neurons and padding descriptor slots).
__device__ __forceinline__ double w0_of(const double* p, const TableLayout& L, int t, int mu, int v) {
  if (mu >= L.NN || v >= L.ND) return 0.0;
  return p[(int64_t)t * (L.ND + 2) * L.NN + (int64_t)mu * L.ND + v];
}

}  // namespace

// One thread per table element of one parameter set (blockIdx.y = set).
__global__ void k_model_tables(const double* __restrict__ params, int64_t npar, TableLayout L,
                               unsigned char* __restrict__ base, int64_t set_stride) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double* p = params + (int64_t)blockIdx.y * npar;
  unsigned char* out = base + (int64_t)blockIdx.y * set_stride;
  int64_t k = g;
  // w0 [nets][NNp][ND] and w0t [nets][ND][NNp]
  const int64_t n_w0 = (int64_t)L.nets * L.NNp * L.ND;
  if (k < n_w0) {
    const int t = (int)(k / ((int64_t)L.NNp * L.ND)), r = (int)(k % ((int64_t)L.NNp * L.ND));
    const int mu = r / L.ND, v = r % L.ND;
    const float x = (float)w0_of(p, L, t, mu, v);
    ((float*)(out + L.at_w0))[k] = x;
    ((float*)(out + L.at_w0t))[((int64_t)t * L.ND + v) * L.NNp + mu] = x;
    return;
  }
  k -= n_w0;
  // b0 [nets][NNp] then b1; w1 [nets][NNp]
  const int64_t n_b = (int64_t)L.nets * L.NNp;
  if (k < n_b) {
    const int t = (int)(k / L.NNp), mu = (int)(k % L.NNp);
    const int64_t o = (int64_t)t * (L.ND + 2) * L.NN + (int64_t)L.NN * L.ND;
    ((float*)(out + L.at_b0))[k] = mu < L.NN ? (float)p[o + mu] : 0.f;
    ((float*)(out + L.at_w1))[k] = mu < L.NN ? (float)p[o + L.NN + mu] : 0.f;
    if (k == 0) ((float*)(out + L.at_b0))[n_b] = (float)p[L.off_b1];
    return;
  }
  k -= n_b;
  // bf16 w0b [nets][NNp][NDp32] and w0tb [nets][NDp32][NNp]
  const int64_t n_wb = (int64_t)L.nets * L.NNp * L.NDp32;
  if (k < n_wb) {
    const int t = (int)(k / ((int64_t)L.NNp * L.NDp32)), r = (int)(k % ((int64_t)L.NNp * L.NDp32));
    const int mu = r / L.NDp32, v = r % L.NDp32;
    const uint16_t b = bf16_bits((float)w0_of(p, L, t, mu, v));
    ((uint16_t*)(out + L.at_w0b))[k] = b;
    ((uint16_t*)(out + L.at_w0tb))[((int64_t)t * L.NDp32 + v) * L.NNp + mu] = b;
    return;
  }
  k -= n_wb;
  // radial coefficients c^R [T][T][KR][n_R rounded up to 4]
  const int wR = round4(L.nR);
  const int64_t n_cR = (int64_t)L.T * L.T * L.KR * wR;
  if (k < n_cR) {
    const int n = (int)(k % wR), kk = (int)(k / wR % L.KR);
    const int64_t a = k / wR / L.KR;
    ((float*)(out + L.at_cR))[k] = n < L.nR ? (float)p[L.off_cR + (a * L.nR + n) * L.KR + kk] : 0.f;
    return;
  }
  k -= n_cR;
  // angular coefficients [T x T pairs, pair stride apart][KA][n_A rounded up to 4]
  // and their Chebyshev series
  if (k < L.n_cA) {
    const int w = round4(L.nA);
    const int a = (int)(k / L.cA_pair), q = (int)(k % L.cA_pair), kk = q / w, n = q % w;
    float x = 0.f, y = 0.f;
    if (kk < L.KA && n < L.nA) {
      const double* c = p + L.off_cA + ((int64_t)a * L.nA + n) * L.KA;
      x = (float)c[kk];
      if (kk > 0) {
        y = 0.5f * x;
      } else {
        float sum = 0.f;
        for (int v = L.KA - 1; v > 0; --v) sum += 0.5f * (float)c[v];
        y = x + sum;
      }
    }
    ((float*)(out + L.at_cA))[k] = x;
    ((float*)(out + L.at_cS))[k] = y;
  }
}

int64_t table_elements(const TableLayout& L) {
  return (int64_t)L.nets * L.NNp * L.ND + (int64_t)L.nets * L.NNp + (int64_t)L.nets * L.NNp * L.NDp32 +
         (int64_t)L.T * L.T * L.KR * round4(L.nR) + L.n_cA;
}

void launch_model_tables(const double* params, int64_t npar, int32_t P, const TableLayout& L,
                         unsigned char* base, int64_t set_stride, hipStream_t s) {
  const int64_t n = table_elements(L);
  dim3 grid((unsigned)div_up(n, kBlock), (unsigned)P);
  hipLaunchKernelGGL(k_model_tables, grid, dim3(kBlock), 0, s, params, npar, L, base, set_stride);
}

}  // namespace nep
