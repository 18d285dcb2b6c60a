// Second half of a split-K call of the tiled kernel: adds the K-slabs of every partial tile in slab
// order (the result does not depend on which workgroup finished first) and rounds once to the output type.
// A workgroup owns 16 rows of a tile; a thread has 16 consecutive columns of one row, as in the tiled
// kernel, so a slab costs it four 16-byte loads, the loads of four slabs in flight together.
// Bound by the traffic of the partial sums, which stay in the memory-side cache.
#include "qg_common.h"

namespace qg {

typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef __bf16 b2_t __attribute__((ext_vector_type(2)));

template <int ROUTE>
__global__ __launch_bounds__(256) void reduce_tiles_kernel(const float* __restrict__ ws, uint16_t* __restrict__ C, int M, int N,
                                                           int bm, int splitk, int tiles_m, int tiles_n) {
  const int mts = bm / 16, tile = blockIdx.x / mts, mt = blockIdx.x % mts;
  int tm = tiles_m, tn = tile - tiles_m * tiles_n;        // behind the others: the last row tile of 64 rows
  if (tn < 0) tile_position<LARGE_GROUP_M>(tile, tiles_m, tiles_n, &tm, &tn);
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const int m = tm * bm + mt * 16 + (l & 15);
  const int nc = tn * (LARGE_BN / TILE_N) + w;
  if (m >= M || nc >= N / TILE_N) return;                 // not stored by the tiled kernel
  const int64_t slab = (int64_t)bm * (LARGE_BN / 4);      // in 16-byte pieces
  const f4_t* src = reinterpret_cast<const f4_t*>(ws) + (int64_t)tile * splitk * slab + mt * 1024 + tid;
  f4_t sum[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) sum[nt] = (f4_t){0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < splitk; sp += 4) {
    f4_t v[4][4];
#pragma unroll
    for (int y = 0; y < 4; ++y)
      if (sp + y < splitk) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) v[y][nt] = __builtin_nontemporal_load(src + (sp + y) * slab + nt * 256);
      }
#pragma unroll
    for (int y = 0; y < 4; ++y)
      if (sp + y < splitk) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) sum[nt] += v[y][nt];
      }
  }
  uint32_t o[8];
#pragma unroll
  for (int r = 0; r < 4; ++r)                             // column offset 4r + nt
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f2_t f = {sum[2 * h][r], sum[2 * h + 1][r]};
      if constexpr (ROUTE == ROUTE_F16) o[2 * r + h] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, h2_t));
      else o[2 * r + h] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t));
    }
  u4_t* dst = reinterpret_cast<u4_t*>(C + (int64_t)m * N + TILE_N * nc + 16 * (l >> 4));
  dst[0] = (u4_t){o[0], o[1], o[2], o[3]};
  dst[1] = (u4_t){o[4], o[5], o[6], o[7]};
}

int launch_reduce_tiles(const GemmParams& p, int route, int bm, hipStream_t st) {
  const int all_m = (p.M + bm - 1) / bm, tiles_n = (p.N + LARGE_BN - 1) / LARGE_BN;
  const int tiles_m = bm == 128 && large_last64(p.M) ? all_m - 1 : all_m;
  auto kern = route == ROUTE_F16 ? reduce_tiles_kernel<ROUTE_F16> : reduce_tiles_kernel<ROUTE_BF16>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(all_m * tiles_n * (bm / 16))), dim3(256), 0, st, p.ws, p.C, p.M, p.N, bm, p.splitk, tiles_m, tiles_n);
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

// Memory to zero by a kernel: a memset does not go into a captured graph.
__global__ __launch_bounds__(256) void clear_kernel(u4_t* __restrict__ dst, int64_t pieces) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < pieces) dst[i] = (u4_t){0, 0, 0, 0};
}

// bytes: a multiple of 16
int launch_clear(void* dst, size_t bytes, hipStream_t st) {
  const int64_t pieces = (int64_t)(bytes / 16);
  hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, static_cast<u4_t*>(dst), pieces);
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

}  // namespace qg
