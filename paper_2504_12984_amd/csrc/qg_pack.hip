// Compact storage and the offline re-layout of the weight.
//   pack_codes_kernel : one code per byte -> canonical gap-free bit stream
//                       (paper, Section "Storage of Low-Precision Data")
//   repack_kernel     : canonical [K,N] stream -> tiled device layout
//                       (paper, Section "Efficient Low-Precision Weight Loading",
//                       the "Change Layout" pre-processing step)
// A weight passes through each once when a model is loaded.
#include "qg_common.h"
#include "qg_static_for.h"

namespace qg {

// Vector loads and stores that assume no alignment (the hardware takes any address; the
// canonical stream and the codes may start anywhere).
typedef uint32_t u4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u2_any __attribute__((ext_vector_type(2), aligned(1)));

// Four codes, one per byte of x, as 4*BITS adjacent bits.
template <int BITS>
__device__ __forceinline__ uint32_t squeeze4(uint32_t x) {
  if constexpr (BITS == 8) return x;
  constexpr uint32_t M = (1u << BITS) - 1u;
  const uint32_t p = (x & (M * 0x00010001u)) | ((x >> (8 - BITS)) & ((M << BITS) * 0x00010001u));
  constexpr uint32_t M2 = (1u << (2 * BITS)) - 1u;
  return (p & M2) | ((p >> (16 - 2 * BITS)) & (M2 << (2 * BITS)));
}

// 32 consecutive codes fill exactly BITS dwords.  A thread squeezes 32 codes (two 16-byte loads)
// and a workgroup meets in LDS so that the stream leaves in 16-byte stores of whole cache lines.
// Bound by memory: on K = 8192, N = 28672 the codes of 5 bits take 68 us = 5.6 TB/s read and written
// (4 bits 61, 8 bits 79; a device copy of 256 MiB moves 5.4 TB/s, one of 2 GiB 4.9).  With a thread that gathered eight
// codes byte by byte and stored bytes it was 207 (187, 253) us: byte-wide accesses.
constexpr int PACK_CODES = 256 * 32;      // codes per workgroup
template <int BITS>
__global__ __launch_bounds__(256) void pack_codes_kernel(const uint8_t* __restrict__ codes, int64_t count,
                                                         uint8_t* __restrict__ out, int64_t out_bytes) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[256 * BITS];
  const int tid = threadIdx.x;
  const int64_t e0 = (int64_t)blockIdx.x * PACK_CODES;
  const uint8_t* src = codes + e0 + 32 * tid;
  uint32_t x[8];
  const bool whole = e0 + PACK_CODES <= count;
  if (whole) {
    const u4_any a = reinterpret_cast<const u4_any*>(src)[0], b = reinterpret_cast<const u4_any*>(src)[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[i] = a[i]; x[4 + i] = b[i]; }
  } else {                                // the last workgroup: codes past the end count as zero
    const int64_t left = count - e0 - 32 * tid;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * i + e < left) x[i] |= (uint32_t)src[4 * i + e] << (8 * e);
    }
  }
  uint32_t r[BITS];
#pragma unroll
  for (int d = 0; d < BITS; ++d) r[d] = 0;
  static_for<8>([&](auto Ic) __attribute__((always_inline)) {
    constexpr int bit = decltype(Ic)::value * 4 * BITS, h = bit >> 5, p = bit & 31;
    const uint32_t q = squeeze4<BITS>(x[decltype(Ic)::value]);
    r[h] |= q << p;
    if constexpr (p + 4 * BITS > 32) r[h + 1] |= q >> (32 - p);
  });
#pragma unroll
  for (int d = 0; d < BITS; ++d) lds[tid * BITS + d] = r[d];
  __syncthreads();
  uint8_t* dst = out + (int64_t)blockIdx.x * (1024 * BITS);
  if (whole) {
    for (int u = tid; u < 64 * BITS; u += 256)
      reinterpret_cast<u4_any*>(dst)[u] = reinterpret_cast<const u4_any*>(lds)[u];
  } else {
    const int64_t left = out_bytes - (int64_t)blockIdx.x * (1024 * BITS);
    for (int i = tid; i < 1024 * BITS && i < left; i += 256) dst[i] = reinterpret_cast<const uint8_t*>(lds)[i];
  }
}

// How the codes of a lane are arranged (see qg_common.h for the element <-> (chunk, lane, pair) maps).
enum RepackMode {
  REPACK_STREAMS = 0,   // first layout, two 16-bit streams
  REPACK_PLAIN = 1,     // first layout, plain order (types with a hardware convert, codebook indices)
  REPACK_R32 = 2,       // second layout, two 16-bit streams
  REPACK_R32_PLAIN = 3,
  REPACK_I8 = 4,        // third layout, four byte streams
  NUM_REPACK = 5
};

// One wavefront builds one chunk.  A lane's columns are adjacent (four of them, two in the second
// layout), so what it needs of a row is ONE field of the canonical stream, and the four wavefronts of a workgroup
// take adjacent strips of the same 128 rows.  Their part of a row, 32*BITS bytes, goes to LDS in 16-byte loads
// (a last workgroup of fewer than four strips: 8-byte ones, which no row is a fraction of), and a lane picks the two dwords with its field
// from each of its 32 (64) rows there.  Workgroups are dealt out so that one XCD gets a run of
// them: the parts of a cache line that two of them need meet in that XCD's L2.
// Bound by memory from 4 bits on (K = 8192, N = 28672: 41 us = 5.7 TB/s at 4 bits, 48 = 6.1 at 5, 94 = 5.0 at 8; every byte is read and
// written once), below that by the placing of the codes (24.5 us = 2.4 TB/s at 1 bit).  When each lane fetched its 8-byte
// windows from global memory, an address per lane and row, their issue took 60, 68, 97 and 32 us (second layout 89, 101, 122, 54).
template <int BITS, int MODE>
__global__ __launch_bounds__(256) void repack_kernel(const uint8_t* __restrict__ canon, uint4* __restrict__ out, int K, int N,
                                                     uint32_t flip, int groups_n, int64_t total, int64_t per_xcd) {
  constexpr int COLS = (MODE == REPACK_R32 || MODE == REPACK_R32_PLAIN) ? 2 : 4;     // adjacent columns of a lane
  constexpr int LANES = TILE_N / COLS;                                               // lanes per k-block
  constexpr uint32_t CODE = (1u << BITS) - 1u;
  // Rows in LDS: 8 * BITS dwords each, 16 more after every run that a k-block has of consecutive rows, so that the up to
  // 16 dwords that each k-block of a wavefront reads at a time lie in banks of their own
  constexpr int RUN = MODE == REPACK_I8 ? 16 : 8, ROW = 8 * BITS;
  auto row_at = [](int k) __attribute__((always_inline)) { return k * ROW + (k / RUN) * 16; };
  __shared__ __attribute__((aligned(16))) uint32_t rows[TILE_K * ROW + TILE_K / RUN * 16];
  const int64_t logical = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (logical >= total) return;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kc = (int)(logical / groups_n), nc0 = (int)(logical % groups_n) * 4, nc = nc0 + w;
  const int64_t row_bytes = (int64_t)(N / 8) * BITS;
  const uint8_t* src = canon + (int64_t)TILE_K * kc * row_bytes + (int64_t)nc0 * (8 * BITS);
  const int strips = min(4, N / TILE_N - nc0);
  if (strips == 4) {
    u4_any v[BITS];
#pragma unroll
    for (int q = 0; q < BITS; ++q) {                    // piece tid + 256 q; a row has 2 * BITS
      const int piece = tid + 256 * q, k = piece / (2 * BITS), at = piece % (2 * BITS);
      v[q] = *reinterpret_cast<const u4_any*>(src + k * row_bytes + 16 * at);
    }
#pragma unroll
    for (int q = 0; q < BITS; ++q) {
      const int piece = tid + 256 * q, k = piece / (2 * BITS), at = piece % (2 * BITS);
      *reinterpret_cast<uint4*>(rows + row_at(k) + 4 * at) = make_uint4(v[q].x, v[q].y, v[q].z, v[q].w);
    }
  } else {
    for (int piece = tid; piece < TILE_K * BITS * strips; piece += 256) {
      const int k = piece / (BITS * strips), at = piece % (BITS * strips);
      const u2_any v = *reinterpret_cast<const u2_any*>(src + k * row_bytes + 8 * at);
      *reinterpret_cast<uint2*>(rows + row_at(k) + 2 * at) = make_uint2(v.x, v.y);
    }
  }
  __syncthreads();
  if (w >= strips) return;
  const int i = l % LANES, b = l / LANES;
  // my field: bits sh .. sh + COLS * BITS - 1 of two dwords (the second one, where the first has all of it, is any dword
  // of `rows`: behind the last row lie 16 more)
  const int fbit = COLS * i * BITS, sh = fbit & 31;
  const uint32_t* mine = rows + 2 * BITS * w + (fbit >> 5);
  uint32_t flips = flip;
#pragma unroll
  for (int c = 1; c < COLS; ++c) flips |= flip << (c * BITS);
  const uint32_t* mine_b = mine + row_at(RUN * b);
  auto field = [&](int k) __attribute__((always_inline)) {        // row k + RUN * b
    const uint32_t* at = mine_b + row_at(k);
    return __builtin_amdgcn_alignbit(at[1], at[0], (uint32_t)sh) ^ flips;
  };
  uint32_t r[4 * BITS];
#pragma unroll
  for (int d = 0; d < 4 * BITS; ++d) r[d] = 0;
  if constexpr (MODE == REPACK_I8) {
    static_for<8>([&](auto Gc) __attribute__((always_inline)) {
      constexpr int J = decltype(Gc)::value / 4, V = decltype(Gc)::value % 4;
      uint32_t f[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = field(64 * J + 4 * V + e);
      static_for<4>([&](auto Nc) __attribute__((always_inline)) {
        constexpr int NT = decltype(Nc)::value, bit = ((J * 4 + NT) * 4 + V) * BITS, h = bit >> 3, p = bit & 7;
        uint32_t q = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) q |= ((f[e] >> (NT * BITS)) & CODE) << (8 * e);
        if constexpr (p + BITS <= 8) {
          r[h] |= q << p;
        } else {                          // the code straddles a byte of its stream
          constexpr int n1 = 8 - p;
          r[h] |= (q & (((1u << n1) - 1u) * 0x01010101u)) << p;
          r[h + 1] |= (q >> n1) & ((CODE >> n1) * 0x01010101u);
        }
      });
    });
  } else {
    static_for<64 / COLS>([&](auto Gc) __attribute__((always_inline)) {
      constexpr int J = decltype(Gc)::value / 4, V = decltype(Gc)::value % 4;
      constexpr int k = (COLS == 4 ? 32 : 16) * J + 2 * V;
      const uint32_t f0 = field(k), f1 = field(k + 1);
      static_for<COLS>([&](auto Nc) __attribute__((always_inline)) {
        constexpr int NT = decltype(Nc)::value, T = (J * COLS + NT) * 4 + V;
        const uint32_t lo = (f0 >> (NT * BITS)) & CODE, hi = (f1 >> (NT * BITS)) & CODE;
        if constexpr (MODE == REPACK_PLAIN || MODE == REPACK_R32_PLAIN) {
          constexpr int bit = 2 * T * BITS, h = bit >> 5, p = bit & 31;
          const uint32_t q = lo | (hi << BITS);
          r[h] |= q << p;
          if constexpr (p + 2 * BITS > 32) r[h + 1] |= q >> (32 - p);
        } else {
          constexpr int bit = T * BITS, h = bit >> 4, p = bit & 15;
          const uint32_t q = lo | (hi << 16);
          if constexpr (p + BITS <= 16) {
            r[h] |= q << p;
          } else {                        // the code straddles a register half of its stream
            constexpr int n1 = 16 - p;
            r[h] |= (q & (((1u << n1) - 1u) * 0x00010001u)) << p;
            r[h + 1] |= (q >> n1) & ((CODE >> n1) * 0x00010001u);
          }
        }
      });
    });
  }
  uint4* dst = out + ((int64_t)nc * (K / TILE_K) + kc) * (64 * BITS) + l;
#pragma unroll
  for (int d = 0; d < BITS; ++d) dst[64 * d] = make_uint4(r[4 * d], r[4 * d + 1], r[4 * d + 2], r[4 * d + 3]);
}

int launch_pack_codes(const uint8_t* codes, int bits, int64_t count, uint8_t* out, hipStream_t st) {
  if (count <= 0) return QG_OK;
  const int64_t out_bytes = (count * bits + 7) / 8;
  const dim3 grid((unsigned)((count + PACK_CODES - 1) / PACK_CODES));
  switch (bits) {
#define QG_PACK(B) case B: hipLaunchKernelGGL(pack_codes_kernel<B>, grid, dim3(256), 0, st, codes, count, out, out_bytes); break;
    QG_PACK(1) QG_PACK(2) QG_PACK(3) QG_PACK(4) QG_PACK(5) QG_PACK(6) QG_PACK(7) QG_PACK(8)
#undef QG_PACK
    default: return QG_EINVAL;
  }
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

template <int MODE>
static int launch_repack_mode(const uint8_t* canon, int bits, int K, int N, uint32_t flip, uint4* out, hipStream_t st) {
  const int groups_n = (N / TILE_N + 3) / 4;
  const int64_t total = (int64_t)(K / TILE_K) * groups_n, per_xcd = (total + 7) / 8;
  const dim3 grid((unsigned)(8 * per_xcd));
  switch (bits) {
#define QG_REPACK(B) case B: hipLaunchKernelGGL((repack_kernel<B, MODE>), grid, dim3(256), 0, st, canon, out, K, N, flip, groups_n, total, per_xcd); break;
    QG_REPACK(1) QG_REPACK(2) QG_REPACK(3) QG_REPACK(4) QG_REPACK(5) QG_REPACK(6) QG_REPACK(7) QG_REPACK(8)
#undef QG_REPACK
    default: return QG_EINVAL;
  }
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

int launch_repack(const uint8_t* canon, int bits, int K, int N, uint32_t flip, int natural, int layout, uint8_t* out, hipStream_t st) {
  uint4* o = reinterpret_cast<uint4*>(out);
  if (layout == QG_LAYOUT_TILE128x64_I8) return launch_repack_mode<REPACK_I8>(canon, bits, K, N, flip, o, st);
  if (layout == QG_LAYOUT_TILE128x64_R32)
    return natural ? launch_repack_mode<REPACK_R32_PLAIN>(canon, bits, K, N, flip, o, st)
                   : launch_repack_mode<REPACK_R32>(canon, bits, K, N, flip, o, st);
  return natural ? launch_repack_mode<REPACK_PLAIN>(canon, bits, K, N, flip, o, st)
                 : launch_repack_mode<REPACK_STREAMS>(canon, bits, K, N, flip, o, st);
}

}  // namespace qg
