// Prefill-sized matmul with int8 activations: LDS-staged A, register-resident W, the integer
// matrix instruction (see qg_a8_gemm.hip for what is computed and how the codes are laid out).
//
// A workgroup of 4 wavefronts computes a 128 x 256 tile of C; wavefront w owns 64 columns and
// all 128 rows, so a weight is unpacked once per 128 rows.  The 128 x 128-byte slab of A is shared
// through LDS, each wavefront's own codes and scales pass through LDS as well: everything is loaded
// straight into LDS by the memory pipe, which takes no registers -- 128 accumulators, the unpacked chunk
// and the sums in flight fill the 256 that leave two workgroups on a CU.
// What bounds the kernel is issue: per 16x16x64 instruction and scale group two vector operations
// per result value (two wavefronts per SIMD: an instruction every 17 clocks alone, every 25 with four
// vector operations beside it, every 33 with six).  So the rest is kept out of the loop:
//   * Codes enter the instruction as signed bytes in the TOP bits of each byte, (q - 2^(b-1)) * 2^(8-b):
//     one shift and one three-input logic operation per quad; the factor 2^(8-b) leaves at the end.  The
//     sums of a chunk stay within 2^21 and start from the bits of 1.5 * 2^23, so they are read as fp32
//     without a convert.
//   * What is left of the zero-points, z' = z - 2^(b-1) (0 for intk without an array), would cost a
//     third operation per value.  It is a product of rank K/group instead,
//     sum_g (s z')[g, n] * rowsum_g[m]: the row sums come from a small kernel ahead of this one, and
//     both factors, split into three bf16 terms each (the products kept are exact to 2^-32), go
//     through the bf16 matrix instruction into the same fp32 accumulators, four groups per instruction.
// Measured at M = 1000, K = 8192, N = 28672, 4 bits, group 128: 256 us = 1830 TOP/s without, 286 us with
// zero-points; in blocks of 64 rows through the streaming kernel (each block reads and unpacks
// all weights again) it was 750.  Without its loads the loop would take 15 % less, without its matrix instructions 22 %.
// Compiled once per code width (QG_BITS).
#include "qg_common.h"
#include "qg_static_for.h"

#ifndef QG_BITS
#error "compile with -DQG_BITS=<1..8>"
#endif

namespace qg {

typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
typedef int i4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));

constexpr int A8_BN = 256;
constexpr int A8_GROUP_M = 8;     // row tiles per L2 panel

// Quad T of the lane: every code in the top BITS bits of its byte with its top bit flipped, i.e. the
// signed byte (q - 2^(BITS-1)) * 2^(8-BITS) (the rest of the byte is zero).
template <int BITS, int T>
__device__ __forceinline__ uint32_t quad_top(const uint32_t (&r)[4 * BITS]) {
  constexpr int bit = T * BITS, h = bit >> 3, p = bit & 7;
  constexpr uint32_t ALL = 0x01010101u, CODE = (((1u << BITS) - 1u) << (8 - BITS)) & 0xffu, SIGN = 0x80808080u;
  if constexpr (BITS == 8) {
    return r[h] ^ SIGN;
  } else if constexpr (p + BITS <= 8) {
    return ((r[h] << (8 - BITS - p)) & (CODE * ALL)) ^ SIGN;
  } else {
    constexpr int n2 = p + BITS - 8;                               // bits of the code in register h + 1
    constexpr uint32_t HIGH = (CODE << (BITS - n2)) & 0xffu, LOW = CODE & ~HIGH;
    return (((r[h + 1] << (8 - n2)) & (HIGH * ALL)) ^ SIGN) | ((r[h] >> n2) & (LOW * ALL));
  }
}

// x as three bf16 terms, x = t0 + t1 + t2 up to 2^-24 |x|
__device__ __forceinline__ void split3(float x, float& t0, float& t1, float& t2) {
  t0 = (float)(__bf16)x;
  t1 = (float)(__bf16)(x - t0);
  t2 = (x - t0) - t1;
}
__device__ __forceinline__ uint32_t pk_bf16(float lo, float hi) {
  f2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t));
}

template <int BITS, int GPC, bool SBF16, bool SPLIT>
__global__ __launch_bounds__(256, 2) void a8_large_kernel(A8Params p, int tiles_m, int tiles_n, int per_xcd) {
  constexpr int RAW = 4 * BITS, BM = 128, MTS = BM / 16, BUF = BM * 128;
  // slabs of A in flight: two where LDS holds them for two workgroups per CU (160 KiB), else one
  constexpr int A_AHEAD = BITS <= 7 ? 2 : 1, ABUFS = A_AHEAD + 1;
  constexpr int W_AT = ABUFS * BUF, S_AT = W_AT + 4 * 1024 * BITS, LDS_BYTES = S_AT + 4 * 256;
  static_assert(2 * LDS_BYTES <= 160 * 1024, "two workgroups per CU");
  __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];   // A slabs, each wavefront's codes, each wavefront's scales

  const int tiles = tiles_m * tiles_n;
  const int logical = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (logical >= tiles * p.splitk) return;
  const int slab = SPLIT ? logical / tiles : 0, tile = SPLIT ? logical % tiles : logical;
  const int panel = A8_GROUP_M * tiles_n;
  const int first_m = (tile / panel) * A8_GROUP_M;
  const int gsize = min(tiles_m - first_m, A8_GROUP_M);
  const int tm = first_m + (tile % panel) % gsize;
  const int tn = (tile % panel) / gsize;

  const int tid = threadIdx.x, l = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = l >> 4, i16 = l & 15;
  const int KC = p.K / TILE_K, NCH = p.N / TILE_N;
  const int kbeg = slab * p.chunks_per_split, kend = min(KC, kbeg + p.chunks_per_split);
  const int m0 = tm * BM;
  const int ncw = tn * (A8_BN / TILE_N) + w;
  const bool active = ncw < NCH;
  const int nc = active ? ncw : NCH - 1;                 // idle wavefronts shadow a valid strip
  const int n16 = TILE_N * nc + 16 * b;                  // the 16 output columns this lane accumulates

  // ---- A slab of a chunk -> LDS: 16-byte slot s of row r holds piece s ^ swizzle(r) ------------
  // A load puts 64 x 16 bytes at consecutive LDS addresses, so the swizzle is applied to the
  // source: thread t fills slot t % 8 of row t / 8 + 32 i from piece (t % 8) ^ swizzle(row).  Rows at
  // or past M are out of the resource's range and read as zeros (the host keeps M * K below 2^31).
  // swizzle(r) = (r ^ r >> 3) & 7 makes the slots of one piece distinct in every aligned run of 8 rows,
  // and the bank groups of 16 rows distinct modulo 256 bytes.
  const int srow = tid >> 3;
  const uint32_t a_voff = (uint32_t)(m0 + srow) * (uint32_t)p.K + 16u * (uint32_t)((tid & 7) ^ ((srow ^ (srow >> 3)) & 7));
  // (rows srow + 32 i have the swizzle of srow for even i and swizzle ^ 4 for odd i: (r >> 3) & 7 changes by 4)
  const uint32_t a_vodd = (uint32_t)(m0 + srow) * (uint32_t)p.K + 16u * (uint32_t)((tid & 7) ^ (((srow ^ (srow >> 3)) & 7) ^ 4));
  const uint64_t a_base = reinterpret_cast<uint64_t>(p.A);
  const u4_t a_rsrc = {(uint32_t)a_base, (uint32_t)(a_base >> 32) & 0xffffu, (uint32_t)p.M * (uint32_t)p.K, 0x00020000u};
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
  const uint32_t lds_a = lds_base + 1024u * (uint32_t)w, lds_w = lds_base + W_AT + (uint32_t)(w * 1024 * BITS), lds_s = lds_base + S_AT + 256u * (uint32_t)w;
  auto a_fetch = [&](int buf, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t off = ((i & 1) ? a_vodd : a_voff) + (uint32_t)(32 * i) * (uint32_t)p.K;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(lds_a + (uint32_t)(buf * BUF + i * 4096)), "v"(off), "s"(a_rsrc), "s"(c * TILE_K) : "memory");
    }
  };

  // ---- W and its scales of the next chunk -> LDS too, for this wavefront alone ---------------------
  // (a register ring would not fit beside 128 accumulators).  One buffer is enough: the codes are
  // unpacked at the start of a chunk, and the load of the next ones starts right after that.
  const uint8_t* wstrip = p.W + (int64_t)nc * KC * (1024 * BITS) + 16 * l;
  // lanes 0..31 fetch two scales each of the chunk's (first) group, lanes 32..63 of its second group
  const uint16_t* sbase = p.S + (int64_t)(GPC == 2 ? l >> 5 : 0) * p.N + TILE_N * nc + 2 * (l & 31);
  auto w_fetch = [&](int c) __attribute__((always_inline)) {
    const uint8_t* src = wstrip + (int64_t)c * (1024 * BITS);
#pragma unroll
    for (int i = 0; i < BITS; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_w + (uint32_t)(i * 1024)), "v"(src + i * 1024) : "memory");
    const int g0 = (GPC > 1) ? GPC * c : ((c >> p.gshift) & p.gmask);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(lds_s), "v"(sbase + (int64_t)g0 * p.N) : "memory");
  };

  w_fetch(kbeg);
  a_fetch(0, kbeg);
  if constexpr (A_AHEAD == 2) a_fetch(1, min(kbeg + 1, kend - 1));

  f4_t acc[MTS][4];
#pragma unroll
  for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = (f4_t){0.f, 0.f, 0.f, 0.f};

  // ---- zero-points: acc -= sum_g (s z')[g, n] * rowsum_g[m], times 2^(8-b) like everything in acc ----
  // k slots of the instruction: lane block b takes group 4 q + b, its eight slots are the products
  // (r0, r1) x (t0, t0), (t1, t1), (t2, t2) and (r2, r2) x (t0, t1) of the terms of rowsum (r) and s z' (t).
  if (p.rowsum) {
    if (slab == 0) {
      const int G = p.K / p.group;
      const int n0 = TILE_N * nc + 4 * i16;
      const u2_t* rs = reinterpret_cast<const u2_t*>(p.rowsum);
      int64_t rrow[MTS];
#pragma unroll
      for (int mt = 0; mt < MTS; ++mt) rrow[mt] = min(m0 + mt * 16 + i16, p.M - 1);
      struct Low { u2_t s4; uint32_t z4; u2_t r[MTS]; };
      auto fetch = [&](Low& t, int q) __attribute__((always_inline)) {
        const int g = min(q + b, G - 1);
        t.s4 = *reinterpret_cast<const u2_t*>(p.S + (int64_t)g * p.N + n0);
        t.z4 = p.Z ? *reinterpret_cast<const uint32_t*>(p.Z + (int64_t)g * p.N + n0) : 0u;
#pragma unroll
        for (int mt = 0; mt < MTS; ++mt) t.r[mt] = rs[(int64_t)g * p.M + rrow[mt]];
      };
      auto add = [&](const Low& t, int q) __attribute__((always_inline)) {
        const float on = (q + b < G) ? -(float)(1 << (8 - BITS)) : 0.f;
        u4_t wz[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
          const uint32_t s16 = (t.s4[nt >> 1] >> (16 * (nt & 1))) & 0xffffu;
          const float s = SBF16 ? __builtin_bit_cast(float, s16 << 16) : (float)__builtin_bit_cast(_Float16, (uint16_t)s16);
          const float z = (float)((int)((t.z4 >> (8 * nt)) & 0xffu) + p.zbias - (1 << (BITS - 1)));
          float t0, t1, t2;
          split3(s * z * on, t0, t1, t2);
          wz[nt] = (u4_t){pk_bf16(t0, t0), pk_bf16(t1, t1), pk_bf16(t2, t2), pk_bf16(t0, t1)};
        }
#pragma unroll
        for (int mt = 0; mt < MTS; ++mt) {
          const u4_t ra = {t.r[mt].x, t.r[mt].x, t.r[mt].x, t.r[mt].y};
#pragma unroll
          for (int nt = 0; nt < 4; ++nt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8_t, wz[nt]), __builtin_bit_cast(b8_t, ra), acc[mt][nt], 0, 0, 0);
        }
      };
      Low even, odd;                    // four groups ahead of use
      fetch(even, 0);
      for (int q = 0; q < G; q += 8) {
        fetch(odd, q + 4);
        add(even, q);
        fetch(even, q + 8);
        add(odd, q + 4);
      }
    }
  }

  // my A fragment of row tile mt, k-step j: piece 4 j + b of row mt*16 + i16
  const int swz = (i16 ^ (i16 >> 3)) & 7;       // of row tile 0; row tile mt adds 2 mt to r >> 3
  __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0), in a form the compiler counts: nothing of its own is in flight in the loop
  __syncthreads();

  const i4_t magic = {0x4b400000, 0x4b400000, 0x4b400000, 0x4b400000};     // 1.5 * 2^23
  int abuf_i = 0;
  for (int c = kbeg; c < kend; ++c) {
    uint32_t raw[RAW];
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
      const u4_t q = *reinterpret_cast<const u4_t*>(lds + W_AT + (w * BITS + i) * 1024 + 16 * l);
      raw[4 * i + 0] = q.x; raw[4 * i + 1] = q.y; raw[4 * i + 2] = q.z; raw[4 * i + 3] = q.w;
    }
    float sf[GPC][16];                                  // the chunk's scales of my 16 columns
#pragma unroll
    for (int g = 0; g < GPC; ++g) {
      const u4_t* sp = reinterpret_cast<const u4_t*>(lds + S_AT + 256 * w + 128 * g + 32 * b);
      const u4_t s01[2] = {sp[0], sp[1]};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t two = s01[i >> 3][(i & 7) >> 1];
        if constexpr (SBF16) sf[g][i] = __builtin_bit_cast(float, (i & 1) ? (two & 0xffff0000u) : (two << 16));
        else sf[g][i] = (float)__builtin_bit_cast(h2_t, two)[i & 1];
        if constexpr (!SBF16) asm("" : "+v"(sf[g][i]));      // widened here and for good: the compiler would fold it into mixed multiply-adds, at half the rate
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // read: the buffers may be refilled
    const int abuf_n = abuf_i == 0 ? ABUFS - 1 : abuf_i - 1;        // the slab of the chunk before this one
    w_fetch(min(c + 1, kend - 1));
    a_fetch(abuf_n, min(c + A_AHEAD, kend - 1));
    u4_t wf[2][4];
    static_for<8>([&](auto Xc) __attribute__((always_inline)) {
      constexpr int X = decltype(Xc)::value, T0 = X * 4;
      wf[X / 4][X % 4] = (u4_t){quad_top<BITS, T0>(raw), quad_top<BITS, T0 + 1>(raw), quad_top<BITS, T0 + 2>(raw), quad_top<BITS, T0 + 3>(raw)};
    });

    const uint8_t* abuf = lds + abuf_i * BUF + i16 * 128;
    auto a_read = [&](int mt, int j) __attribute__((always_inline)) {
      return *reinterpret_cast<const i4_t*>(abuf + mt * 2048 + 16 * (((4 * j + b) ^ swz) ^ ((2 * mt) & 7)));
    };
    // value r of sub-tile nt: acc += scale * sum.  The sums start from the bits of 1.5 * 2^23, so that
    // read as fp32 they are 1.5 * 2^23 + sum exactly (|sum| < 2^22): a subtraction instead of a convert
    // (with several wavefronts on a SIMD fp32 add / multiply-add issue every 2 clocks, converts and
    // half-precision or mixed operations every 4).
    auto scale = [&](auto Gc, auto MTc, auto NTc, auto Rc, int bits) __attribute__((always_inline)) {
      constexpr int G = decltype(Gc)::value, MT = decltype(MTc)::value, NT = decltype(NTc)::value, R = decltype(Rc)::value;
      acc[MT][NT][R] = __builtin_fmaf(sf[G][4 * R + NT], __builtin_bit_cast(float, bits) - 12582912.0f, acc[MT][NT][R]);
    };
    // The chunk is a sequence of units: two sub-tiles of one row tile and one scale group, i.e. 4
    // (group 64: 2) matrix instructions.  Each instruction is followed by its share of the previous
    // unit's eight converts and multiply-adds (4, or 8), so vector and matrix work alternate
    // within one wavefront and the sums of two units (16 registers) are all that is in flight.
    constexpr int UPM = 2 * GPC, MPU = 4 / GPC, VPM = 8 / MPU;      // units per row tile, instructions per unit, values per instruction
    i4_t a[2][2], d[2][2];
    a[0][0] = a_read(0, 0);
    a[0][1] = a_read(0, 1);
    static_for<MTS * UPM + 1>([&](auto Uc) __attribute__((always_inline)) {
      constexpr int U = decltype(Uc)::value, MT = U / UPM, H = U % 2, J0 = (GPC == 2) ? (U / 2) % 2 : 0;
      constexpr int PU = U - 1, PMT = PU / UPM, PH = PU % 2, PG = (GPC == 2) ? (PU / 2) % 2 : 0;       // previous unit
      static_for<MPU>([&](auto Ic) __attribute__((always_inline)) {
        constexpr int I = decltype(Ic)::value, J = J0 + I / 2, N = I % 2, NT = 2 * H + N;
        if constexpr (U < MTS * UPM) {
          if constexpr (GPC == 2 || J == 0) d[U & 1][N] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i4_t, wf[J][NT]), a[MT & 1][J], magic, 0, 0, 0);
          else d[U & 1][N] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i4_t, wf[J][NT]), a[MT & 1][J], d[U & 1][N], 0, 0, 0);
          if constexpr (U % UPM == 0 && MT + 1 < MTS) {          // the next row tile's fragments
            if constexpr (I == 0) a[(MT + 1) & 1][0] = a_read(MT + 1, 0);
            if constexpr (I == 1) a[(MT + 1) & 1][1] = a_read(MT + 1, 1);
          }
        }
        if constexpr (U > 0) {
          static_for<VPM>([&](auto Vc) __attribute__((always_inline)) {
            constexpr int V = I * VPM + decltype(Vc)::value, PN = V / 4, R = V % 4;
            scale(std::integral_constant<int, PG>{}, std::integral_constant<int, PMT>{}, std::integral_constant<int, 2 * PH + PN>{},
                  std::integral_constant<int, R>{}, d[PU & 1][PN][R]);
          });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    // my part of the next chunk is in LDS (loads return in order: all but the newest slab)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(A_AHEAD == 2 ? 4 : 0) : "memory");
    __syncthreads();
    abuf_i = abuf_i == ABUFS - 1 ? 0 : abuf_i + 1;
  }

  if (!active) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the slab loaded past the end
  // ---- split-K: partial tiles meet in the workspace (the exchange of the 16-bit tiled kernel: stores that
  // write through and loads that bypass the caches, one arrival counter per 64-column strip of a tile,
  // the wavefront that arrives last sums the slabs in slab order) ---------------------------------
  if constexpr (SPLIT) {
    constexpr int SC1 = 16;                                   // cache policy: device coherence
    auto ws_rsrc = [&](int sp) __attribute__((always_inline)) {
      return __builtin_amdgcn_make_buffer_rsrc(p.ws + ((int64_t)tile * p.splitk + sp) * (BM * A8_BN), 0, BM * A8_BN * 4, 0x00020000);
    };
    {
      const __amdgpu_buffer_rsrc_t mine = ws_rsrc(slab);
#pragma unroll
      for (int mt = 0; mt < MTS; ++mt)
        if (m0 + mt * 16 + i16 < p.M) {
#pragma unroll
          for (int nt = 0; nt < 4; ++nt)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, acc[mt][nt]), mine, 16 * tid, (mt * 4 + nt) * 4096, SC1);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // my partial strip is out before my ticket is drawn
    unsigned* ticket = p.tickets + 4 * tile + w;
    unsigned drawn = 0;
    if (l == 0) drawn = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    drawn = __builtin_amdgcn_readfirstlane(drawn);
    if (drawn != (unsigned)(p.splitk - 1)) return;
#pragma unroll
    for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = (f4_t){0.f, 0.f, 0.f, 0.f};
    for (int sp = 0; sp < p.splitk; ++sp) {
      const __amdgpu_buffer_rsrc_t r = ws_rsrc(sp);
#pragma unroll
      for (int mt = 0; mt < MTS; ++mt) {
        if (m0 + mt * 16 + i16 < p.M) {                        // rows past M were not written
          u4_t v[4];
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) v[nt] = __builtin_amdgcn_raw_buffer_load_b128(r, 16 * tid, (mt * 4 + nt) * 4096, SC1);
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) acc[mt][nt] += __builtin_bit_cast(f4_t, v[nt]);
        }
      }
    }
    if (l == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
  }

  // ---- row scale, the factor 2^(b-8), one rounding to the output type, store ---------------------
#pragma unroll
  for (int mt = 0; mt < MTS; ++mt) {
    const int m = m0 + mt * 16 + i16;
    if (m < p.M) {
      const float as = (p.a_scale ? p.a_scale[m] : 1.0f) * (1.0f / (float)(1 << (8 - BITS)));
      uint32_t o[8];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f2_t f = {acc[mt][2 * h][r] * as, acc[mt][2 * h + 1][r] * as};
          o[2 * r + h] = p.out_bf16 ? __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t))
                                    : __builtin_bit_cast(uint32_t, __builtin_convertvector(f, h2_t));
        }
      u4_t* dst = reinterpret_cast<u4_t*>(p.C + (int64_t)m * p.N + n16);
      dst[0] = (u4_t){o[0], o[1], o[2], o[3]};
      dst[1] = (u4_t){o[4], o[5], o[6], o[7]};
    }
  }
}

#define QG_CAT2(a, b) a##b
#define QG_CAT(a, b) QG_CAT2(a, b)

template <int GPC, bool SBF16, bool SPLIT>
static int launch_one(const A8Params& p, hipStream_t st) {
  const int tiles_m = (p.M + 127) / 128, tiles_n = (p.N + A8_BN - 1) / A8_BN;
  const int per_xcd = (tiles_m * tiles_n * p.splitk + 7) / 8;
  hipLaunchKernelGGL((a8_large_kernel<QG_BITS, GPC, SBF16, SPLIT>), dim3((unsigned)(8 * per_xcd)), dim3(256), 0, st, p, tiles_m, tiles_n, per_xcd);
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

// p.rowsum: the row sums of a8_rowsum_kernel where a zero-point term is left, else null
int QG_CAT(a8_large_launch_bits, QG_BITS)(const A8Params& p, hipStream_t st) {
#define QG_A8L(GPC_, SB_, SP_) if (((p.group == 64) ? 2 : 1) == GPC_ && (p.scale_bf16 != 0) == SB_ && (p.splitk > 1) == SP_) return launch_one<GPC_, SB_, SP_>(p, st);
  QG_A8L(1, false, false) QG_A8L(1, false, true) QG_A8L(1, true, false) QG_A8L(1, true, true)
  QG_A8L(2, false, false) QG_A8L(2, false, true) QG_A8L(2, true, false) QG_A8L(2, true, true)
#undef QG_A8L
  return QG_EINVAL;
}

}  // namespace qg
