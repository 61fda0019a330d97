// What the hardware's functions are off by, for the bounds that the signature
// kernels rest on: the fp32 logarithm, square root, sine and cosine over every
// Philox word, and the matrix instructions' sums.  Built beside the library and
// called by test_gpu_bounds.py.
#include "../../paper_1110_1328_amd/csrc/srp_entries.h"

using namespace blsh;

namespace {

__device__ inline void keep_max(double *to, double v) {   // v >= 0: its bits order as it does
  atomicMax(reinterpret_cast<unsigned long long *>(to), __builtin_bit_cast(unsigned long long, v));
}

__global__ __launch_bounds__(256) void k_entry_errors(double *out) {
  double radius = 0, most = 0, cosine = 0, sine = 0;
  for (uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x; i < uint64_t(1) << 32; i += uint64_t(gridDim.x) * 256) {
    const uint32_t w = uint32_t(i);
    const double u = (double(w) + 0.5) / 4294967296.0;
    double sn, cs;
    sincos(6.283185307179586476925286766559 * u, &sn, &cs);
    const float a = __builtin_fmaf(float(w), 0x1p-32f, 0x1p-33f), r = srp_fast_radius(w);
    radius = fmax(radius, fabs(double(r) - sqrt(-2.0 * log(u))));
    most = fmax(most, double(r));
    cosine = fmax(cosine, fabs(double(__builtin_amdgcn_cosf(a)) - cs));
    sine = fmax(sine, fabs(double(__builtin_amdgcn_sinf(a)) - sn));
  }
  keep_max(out, radius);
  keep_max(out + 1, most);
  keep_max(out + 2, cosine);
  keep_max(out + 3, sine);
}

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// D = C + A B, one 32 x 32 problem per block of 64 lanes; A [32][K], B [K][32].
__global__ __launch_bounds__(64) void k_bf16(const uint16_t *A, const uint16_t *B, const float *C, float *D) {
  const int lane = threadIdx.x, i = lane & 31, h = lane >> 5;
  A += size_t(blockIdx.x) * 512;
  B += size_t(blockIdx.x) * 512;
  bf16x8 a, b;
  for (int k = 0; k < 8; ++k) {
    a[k] = __builtin_bit_cast(__bf16, A[i * 16 + 8 * h + k]);
    b[k] = __builtin_bit_cast(__bf16, B[(8 * h + k) * 32 + i]);
  }
  floatx16 acc;
  for (int v = 0; v < 16; ++v) acc[v] = C[size_t(blockIdx.x) * 1024 + (8 * (v >> 2) + 4 * h + (v & 3)) * 32 + i];
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
  for (int v = 0; v < 16; ++v) D[size_t(blockIdx.x) * 1024 + (8 * (v >> 2) + 4 * h + (v & 3)) * 32 + i] = acc[v];
}

__global__ __launch_bounds__(64) void k_f32(const float *A, const float *B, const float *C, float *D) {
  const int lane = threadIdx.x, i = lane & 31, h = lane >> 5;
  floatx16 acc;
  for (int v = 0; v < 16; ++v) acc[v] = C[size_t(blockIdx.x) * 1024 + (8 * (v >> 2) + 4 * h + (v & 3)) * 32 + i];
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A[size_t(blockIdx.x) * 64 + i * 2 + h], B[size_t(blockIdx.x) * 64 + h * 32 + i], acc,
                                             0, 0, 0);
  for (int v = 0; v < 16; ++v) D[size_t(blockIdx.x) * 1024 + (8 * (v >> 2) + 4 * h + (v & 3)) * 32 + i] = acc[v];
}

}  // namespace

extern "C" {

// out[4] (device, zeroed): largest error of the radius, largest radius, largest
// error of the cosine and of the sine.
int entry_errors(double *out) {
  k_entry_errors<<<4096, 256>>>(out);
  return int(hipGetLastError()) | int(hipDeviceSynchronize());
}
float entry_bound() { return kFastErr; }
float entry_unit() { return kUnit; }

int product_bf16(const uint16_t *A, const uint16_t *B, const float *C, float *D, int n) {
  k_bf16<<<n, 64>>>(A, B, C, D);
  return int(hipGetLastError()) | int(hipDeviceSynchronize());
}
int product_f32(const float *A, const float *B, const float *C, float *D, int n) {
  k_f32<<<n, 64>>>(A, B, C, D);
  return int(hipGetLastError()) | int(hipDeviceSynchronize());
}
}
