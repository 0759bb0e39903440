// The SwiGLU epilogue's product over every fp32 gate that a product can come to, beside the plain expression and beside 64 bits: one line per `up` with the
// gates tried, the halves that differ (a zero's sign aside), the floats that differ where the half is not zero, and the largest relative error there.
#include <cstdio>

#include "../paper_2602_02192_amd/csrc/echo_device.h"

using namespace echo;

constexpr float LARGEST = 65504.0f * 65504.0f * 32768.0f;   // operands and packed weights saturate at 65504; 32768 of their products
struct Result { unsigned long long tried, halves, floats; unsigned rel; };

__global__ __launch_bounds__(256) void sweep(Result *out, float u) {
  unsigned long long tried = 0, halves = 0, floats = 0;
  float rel = 0.f;
  const uint32_t n = gridDim.x * 256, first = blockIdx.x * 256 + threadIdx.x;   // n divides 2^32
  for (uint32_t k = 0; k < (uint32_t)((1ull << 32) / n); ++k) {
    const float g = __uint_as_float(first + k * n);
    if (!(fabsf(g) <= LARGEST)) continue;   // (infinities, NaN)
    ++tried;
    const float x = g * W_UNSCALE, plain = x / (1.0f + expf(-x)) * (u * W_UNSCALE), got = swiglu(g, u);
    const uint16_t a = f32_to_h16_bits(plain), b = f32_to_h16_bits(got);
    halves += a != b && ((a | b) & 0x7fff) != 0;
    if ((a & 0x7fff) == 0) continue;
    floats += plain != got;
    const double exact = (double)x / (1.0 + exp(-(double)x)) * ((double)u * W_UNSCALE);
    rel = fmaxf(rel, (float)fabs(got / exact - 1.0));
  }
  atomicAdd(&out->tried, tried);
  atomicAdd(&out->halves, halves);
  atomicAdd(&out->floats, floats);
  atomicMax(&out->rel, __float_as_uint(rel));   // (floats of one sign order as their bits do)
}

int main() {
  Result *out, r;
  if (hipMalloc((void **)&out, sizeof r) != hipSuccess) return 1;
  // of size one, of the size the layers have, below it, beyond half, the largest
  for (float u : {W_SCALE, -3.7f * W_SCALE, 0.37f, 6.4e6f, LARGEST}) {
    if (hipMemset(out, 0, sizeof r) != hipSuccess) return 1;
    hipLaunchKernelGGL(sweep, dim3(4096), dim3(256), 0, 0, out, u);
    if (hipGetLastError() != hipSuccess || hipMemcpy(&r, out, sizeof r, hipMemcpyDeviceToHost) != hipSuccess) return 1;
    float rel;
    __builtin_memcpy(&rel, &r.rel, 4);
    printf("%.9g %llu %llu %llu %.4g\n", u, r.tried, r.halves, r.floats, rel);
    fflush(stdout);
  }
  return 0;
}
