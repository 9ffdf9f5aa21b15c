// Runs each form of the rounding helpers of csrc/wcc_rn.hpp on its own (the
// general ones, the near ones with their range tests, and the operations that
// choose between them), and the limiter's weights of csrc/wcc_cell.hpp in both
// forms, on operands read from files.  Test infrastructure:
// tests/test_gpu_rounding_forms.py generates the operands and compares.
//
//   rn_forms <div.bin> <sqrt.bin> <weights.bin> <out.bin>
//
// div.bin: n numerators, then n denominators (binary64); sqrt.bin: m operands;
// weights.bin: k each of b0, b1, b2, st, eps.  out.bin: n each of div_rn,
// div_rn_any, div_near, its range test (1 or 0), rcp_rn, rcp_near, its range
// test; m each of sqrt_rn, sqrt_rn_any, sqrt_near, its range test; then for
// P = 1 and P = 3: k each of w0, w1, w2 (near), their range test, w0, w1, w2
// (general).  Exit status 0 on success, 1 on a HIP error, 2 on unreadable
// input.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#include "wcc_cell.hpp"
#include "wcc_rn.hpp"

__global__ void k_div(const double* a, const double* b, double* out, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double x = a[i], y = b[i];
    out[i] = wcc::div_rn(x, y);
    out[n + i] = wcc::div_rn_any(x, y);
    out[2 * n + i] = wcc::div_near(x, y, wcc::rcp_near(y));
    out[3 * n + i] = wcc::near_num(x) && wcc::near_den(y) ? 1.0 : 0.0;
    out[4 * n + i] = wcc::rcp_rn(y);
    out[5 * n + i] = wcc::rcp_near(y);
    out[6 * n + i] = wcc::near_rcp(y) ? 1.0 : 0.0;
  }
}

__global__ void k_sqrt(const double* x, double* out, long m) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < m; i += (long)gridDim.x * blockDim.x) {
    out[i] = wcc::sqrt_rn(x[i]);
    out[m + i] = wcc::sqrt_rn_any(x[i]);
    out[2 * m + i] = wcc::sqrt_near(x[i]);
    out[3 * m + i] = wcc::near_sqrt(x[i]) ? 1.0 : 0.0;
  }
}

template <int P>
__global__ void k_weights(const double* in, double* out, long k) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < k; i += (long)gridDim.x * blockDim.x) {
    const double eps = in[4 * k + i];
    double w[3];
    bool ok = wcc::near_eps(eps), unused = true;
    wcc::limiter_weights<P, true>(in[i], in[k + i], in[2 * k + i], in[3 * k + i], eps, w[0], w[1], w[2], ok);
    for (int j = 0; j < 3; ++j) out[j * k + i] = w[j];
    out[3 * k + i] = ok ? 1.0 : 0.0;
    wcc::limiter_weights<P, false>(in[i], in[k + i], in[2 * k + i], in[3 * k + i], eps, w[0], w[1], w[2], unused);
    for (int j = 0; j < 3; ++j) out[(4 + j) * k + i] = w[j];
  }
}

static bool read_all(const char* path, std::vector<double>& v) {
  FILE* f = fopen(path, "rb");
  if (!f) return false;
  fseek(f, 0, SEEK_END);
  const long bytes = ftell(f);
  fseek(f, 0, SEEK_SET);
  if (bytes <= 0 || bytes % 8) {
    fclose(f);
    return false;
  }
  v.resize(bytes / 8);
  const bool ok = fread(v.data(), 8, v.size(), f) == v.size();
  fclose(f);
  return ok;
}

#define HIP_OK(call)                                                       \
  do {                                                                     \
    hipError_t e_ = (call);                                                \
    if (e_ != hipSuccess) {                                                \
      fprintf(stderr, "%s: %s\n", #call, hipGetErrorString(e_));          \
      return 1;                                                            \
    }                                                                      \
  } while (0)

int main(int argc, char** argv) {
  if (argc != 5) {
    fprintf(stderr, "usage: %s div.bin sqrt.bin weights.bin out.bin\n", argv[0]);
    return 2;
  }
  std::vector<double> ab, x, w;
  if (!read_all(argv[1], ab) || !read_all(argv[2], x) || !read_all(argv[3], w) || ab.size() % 2 || w.size() % 5) {
    fprintf(stderr, "cannot read the operands\n");
    return 2;
  }
  const long n = (long)ab.size() / 2, m = (long)x.size(), k = (long)w.size() / 5;
  std::vector<double> out(7 * n + 4 * m + 14 * k);
  double *d_ab = nullptr, *d_x = nullptr, *d_w = nullptr, *d_out = nullptr;
  HIP_OK(hipMalloc(&d_ab, ab.size() * sizeof(double)));
  HIP_OK(hipMalloc(&d_x, x.size() * sizeof(double)));
  HIP_OK(hipMalloc(&d_w, w.size() * sizeof(double)));
  HIP_OK(hipMalloc(&d_out, out.size() * sizeof(double)));
  HIP_OK(hipMemcpy(d_ab, ab.data(), ab.size() * sizeof(double), hipMemcpyHostToDevice));
  HIP_OK(hipMemcpy(d_x, x.data(), x.size() * sizeof(double), hipMemcpyHostToDevice));
  HIP_OK(hipMemcpy(d_w, w.data(), w.size() * sizeof(double), hipMemcpyHostToDevice));
  // grid-stride loops: any grid covers every element
  k_div<<<1024, 256>>>(d_ab, d_ab + n, d_out, n);
  HIP_OK(hipGetLastError());
  k_sqrt<<<1024, 256>>>(d_x, d_out + 7 * n, m);
  HIP_OK(hipGetLastError());
  k_weights<1><<<1024, 256>>>(d_w, d_out + 7 * n + 4 * m, k);
  HIP_OK(hipGetLastError());
  k_weights<3><<<1024, 256>>>(d_w, d_out + 7 * n + 4 * m + 7 * k, k);
  HIP_OK(hipGetLastError());
  HIP_OK(hipMemcpy(out.data(), d_out, out.size() * sizeof(double), hipMemcpyDeviceToHost));
  HIP_OK(hipFree(d_ab));
  HIP_OK(hipFree(d_x));
  HIP_OK(hipFree(d_w));
  HIP_OK(hipFree(d_out));
  FILE* f = fopen(argv[4], "wb");
  if (!f || fwrite(out.data(), sizeof(double), out.size(), f) != out.size()) {
    fprintf(stderr, "cannot write %s\n", argv[4]);
    return 2;
  }
  fclose(f);
  printf("rn_forms: %ld quotients, %ld square roots, %ld sets of weights\n", n, m, k);
  return 0;
}
