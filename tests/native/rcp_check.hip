// GPU check of the reciprocal of the face code (rcp_nr in physics.hpp): its
// estimate is off by less than 2^-24, the third-order correction leaves 2^-72 of
// it, and what the correction's own operations add is below 2^-76, so before the
// final rounding the value is within 2^-71.9 of 1/b and after it within
// 1/2 + 2^-18 ulp. Operands over the exponents that the products of two
// reconstruction normalisers take (1e-94 to 1e306), random mantissas, and values
// next to powers of two. The error in ulps comes from the residual 1 - b q, which
// one fma gives to 2^-53 of itself. Prints the worst; exit 1 above the bound.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2203_13760_amd/csrc/physics.hpp"

__global__ void k_rcp(const double* __restrict__ b, double* __restrict__ q, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) q[i] = cfd::rcp_nr(b[i]);
}

int main() {
  const int n = 1 << 22;
  std::mt19937_64 rng(1403);
  std::uniform_real_distribution<double> mant(1.0, 2.0), e(-312.0, 1016.0);
  std::vector<double> b(n), q(n);
  for (int i = 0; i < n; ++i) b[i] = std::ldexp((rng() & 1 ? 1.0 : -1.0) * mant(rng), (int)std::floor(e(rng)));
  for (int i = 0; i < 4096; ++i) {
    b[i] = std::ldexp(1.0 + i * 0x1p-52, (i % 1300) - 312);
    b[4096 + i] = std::ldexp(2.0 - (i + 1) * 0x1p-52, (i % 1300) - 312);
  }
  double *db = nullptr, *dq = nullptr;
  const size_t bytes = sizeof(double) * (size_t)n;
  if (hipMalloc(&db, bytes) != hipSuccess || hipMalloc(&dq, bytes) != hipSuccess ||
      hipMemcpy(db, b.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
    std::printf("allocation or upload failed\n");
    return 1;
  }
  hipLaunchKernelGGL(k_rcp, dim3((n + 255) / 256), dim3(256), 0, 0, db, dq, n);
  if (hipGetLastError() != hipSuccess || hipMemcpy(q.data(), dq, bytes, hipMemcpyDeviceToHost) != hipSuccess) {
    std::printf("kernel failed\n");
    return 1;
  }
  double worst = 0.0, at = 0.0;
  long long bad = 0;
  for (int i = 0; i < n; ++i) {
    int x;
    std::frexp(q[i], &x);  // |q| in [2^(x-1), 2^x): ulp 2^(x-53)
    const double ulps = std::fabs(std::fma(-b[i], q[i], 1.0)) / std::fabs(std::ldexp(b[i], x - 53));
    if (!(ulps <= 0.5 + 0x1p-18)) ++bad;
    if (!(ulps <= worst)) {
      worst = ulps;
      at = b[i];
    }
  }
  std::printf("samples %d worst_ulp %.7f at %.17g above_bound %lld\n", n, worst, at, bad);
  (void)hipFree(db);
  (void)hipFree(dq);
  return bad == 0 ? 0 : 1;
}
