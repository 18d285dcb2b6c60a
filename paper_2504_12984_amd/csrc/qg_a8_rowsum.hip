// Row sums of int8 activations per scale group, for the zero-point term of the tiled int8 kernel:
// out[g][m] = sum of A8[m, k] over the rows k of group g, as three bf16 terms (r0 | r1 << 16,
// r2 | r2 << 16) whose sum is the integer (up to 2^24 exactly), in the order the matrix instruction takes them.
#include "qg_common.h"

namespace qg {

typedef int i4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef __bf16 b2_t __attribute__((ext_vector_type(2)));

// A team of TEAM lanes adds one (row, group), 16 bytes per lane and step.  Bound by reading A once
// (M = 1000, K = 8192: 8 MB).
template <int TEAM>
__global__ __launch_bounds__(256) void a8_rowsum_kernel(const int8_t* __restrict__ A, int M, int K, int group, uint2* __restrict__ out) {
  const int G = K / group;
  const int64_t job = ((int64_t)blockIdx.x * 256 + threadIdx.x) / TEAM;
  const int lane = threadIdx.x % TEAM;
  if (job >= (int64_t)M * G) return;
  const int m = (int)(job / G), g = (int)(job % G);
  const int8_t* src = A + (int64_t)m * K + (int64_t)g * group;
  int sum = 0;
  for (int o = 16 * lane; o < group; o += 16 * TEAM) {
    const i4_t v = *reinterpret_cast<const i4_t*>(src + o);
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_sdot4(v[i], 0x01010101, sum, false);
  }
#pragma unroll
  for (int d = TEAM / 2; d >= 1; d /= 2) sum += __shfl_xor(sum, d, 64);
  if (lane == 0) {
    const float x = (float)sum, r0 = (float)(__bf16)x, r1 = (float)(__bf16)(x - r0), r2 = (x - r0) - r1;
    auto pk = [](float lo, float hi) { f2_t f = {lo, hi}; return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t)); };
    out[(int64_t)g * M + m] = make_uint2(pk(r0, r1), pk(r2, r2));
  }
}

int launch_a8_rowsum(const int8_t* A, int M, int K, int group, uint2* out, hipStream_t st) {
  const int64_t jobs = (int64_t)M * (K / group);
  if (group >= 1024)
    hipLaunchKernelGGL(a8_rowsum_kernel<64>, dim3((unsigned)((jobs + 3) / 4)), dim3(256), 0, st, A, M, K, group, out);
  else
    hipLaunchKernelGGL(a8_rowsum_kernel<4>, dim3((unsigned)((jobs + 63) / 64)), dim3(256), 0, st, A, M, K, group, out);
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

}  // namespace qg
