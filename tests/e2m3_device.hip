// Device checks of the operand encoders and turns in lp_ops.h
// (test_gpu_encoders.py): libe2m3_device.so.
#include "lp_ops.h"

namespace mps {
namespace {

// e2m3x4 of (x, y, z, w) / 64 against e2m3_code of each, for every float x with
// bits lo .. hi - 1 in each of the four positions, both signs; the other
// positions hold other values of the same range.
__global__ void check_codes(uint32_t lo, uint32_t hi, unsigned long long* bad) {
  unsigned long long n = 0;
  for (uint64_t i = lo + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t u = (uint32_t)i;
    const uint32_t o = lo + (hi - 1 - u);  // the range backwards
    const uint32_t b[4] = {u, u | 0x80000000u, o, o | 0x80000000u};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x[4];
      uint32_t want = 0;
      for (int e = 0; e < 4; ++e) {
        x[e] = __builtin_bit_cast(float, b[(r + e) & 3]);
        want |= e2m3_code(x[e]) << (6 * e);
      }
      n += e2m3x4(x[0] * 0.015625f, x[1] * 0.015625f, x[2] * 0.015625f, x[3] * 0.015625f) != want;
    }
  }
  if (n) atomicAdd(bad, n);
}

// Turned operands: 20 dwords a thread (32-byte pair-plane row of E4M3 codes, 32-byte E2M3
// record, 16 bytes of 16-bit values), their turned forms.
__global__ void do_turns(const int* in, int* out) {
  const int t = threadIdx.x;
  in += t * 20;
  out += t * 20;
  intx8 a, b;
  for (int i = 0; i < 8; ++i) {
    a[i] = in[i];
    b[i] = in[8 + i];
  }
  const intx4 c = {in[16], in[17], in[18], in[19]};
  const intx8 ta = turn_e4m3(a), tb = turn_e2m3(b);
  const intx4 tc = turn(c);
  for (int i = 0; i < 8; ++i) {
    out[i] = ta[i];
    out[8 + i] = tb[i];
  }
  for (int i = 0; i < 4; ++i) out[16 + i] = tc[i];
}

// Left vectors to fp16 planes and E2M3 records: v[16] floats a thread (8 complex).
__global__ void do_split8(const float* in, uint32_t* out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  float2 v[8];
  uint32_t h[8], w[8];
  for (int i = 0; i < 8; ++i) v[i] = make_float2(in[16 * t + 2 * i], in[16 * t + 2 * i + 1]);
  split8_e2m3(v, h, w);
  for (int i = 0; i < 8; ++i) {
    out[16 * t + i] = h[i];
    out[16 * t + 8 + i] = w[i];
  }
}

}  // namespace
}  // namespace mps

extern "C" {

// All on the null stream of the current device; device pointers.
int check_e2m3_codes(uint32_t lo, uint32_t hi, unsigned long long* bad) {
  hipLaunchKernelGGL(mps::check_codes, dim3(2048), dim3(256), 0, nullptr, lo, hi, bad);
  return (int)hipGetLastError();
}
int turn_operands(const int* in, int* out, int n) {  // n <= 1024 sets of 20 dwords
  if (n < 1 || n > 1024) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(mps::do_turns, dim3(1), dim3(n), 0, nullptr, in, out);
  return (int)hipGetLastError();
}
int split_slices(const float* in, uint32_t* out, int blocks) {  // 64 slices a block
  if (blocks < 1) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(mps::do_split8, dim3(blocks), dim3(64), 0, nullptr, in, out);
  return (int)hipGetLastError();
}

}  // extern "C"
