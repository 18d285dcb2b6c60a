// Prefill-sized matmul with int8 activations: LDS-staged A, register-resident W, the integer
// matrix instruction (see qg_a8_gemm.hip for what is computed and how the codes are laid out).
//
// A workgroup of 4 wavefronts computes a 128 x 256 tile of C -- or 64 x 256 where 128 rows would leave CUs idle,
// or (one launch, both heights) be more than the rows or the round that are left --;
// wavefront w owns 64 columns and all rows, so a weight is unpacked once per 128 rows.  The 128 x 128-byte slab of A is shared
// through LDS, each wavefront's own codes and scales pass through LDS as well: everything is loaded
// straight into LDS by the memory pipe, which takes no registers -- 128 accumulators, the unpacked chunk
// and the sums in flight fill the 256 that leave two workgroups on a CU.
// What bounds the kernel most is issue (counters: vector instructions take up to 0.67 of a busy CU's clocks, the
// matrix pipe 0.4 to 0.45): per 16x16x64 instruction and scale group two vector operations per result
// value (two wavefronts per SIMD: an instruction every 17 clocks alone, every 25 with four vector
// operations beside it, every 33 with six).  So the rest is kept out of the loop:
//   * Codes enter the instruction as signed bytes, times a power of two.  The sums of a chunk stay within 2^22 and
//     start from the bits of a float, so they are read as fp32 without a convert and without the factor.
//   * No zero-points (CORR = false): the byte is (q - 2^(b-1)) * 2^(8-b), one shift and one three-input
//     logic operation per quad.
//   * Zero-points, or uintk (CORR): the sum over a scale group has to stay an exact integer, because
//     q and z cancel in it.  Up to 7 bits a zero-point in the range of the codes is subtracted from the four
//     bytes of a quad at once, (q - z) * 2^(7-b), two more operations per quad and none per value.
//     A zero-point beyond the codes, and 8-bit codes, whose difference takes nine bits, go through the row
//     sums of A instead (one more matrix instruction per row tile and k-step, with ones for codes): one more
//     multiply-add per value, on the integer sum and therefore exact.  Which of the two is decided by each
//     wavefront from the zero-points it reads.
// Measured at M = 1000, K = 8192, N = 28672, group 128 (one box, us): int4 282, uint4 with zero-points 290, with
// zero-points beyond the codes 351, uint8 with zero-points 388 (group 64: 338, 364, -, 499); with the row sums of
// all groups taken off ahead of the loop, in fp32 and not exact, the second was 295, the last 345.
// In blocks of 64 rows through the streaming kernel (each block reads and unpacks all weights again) uint4 takes 750.
// Compiled once per code width (QG_BITS).
#include "qg_common.h"
#include "qg_static_for.h"
#include "qg_wait.h"

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

// Quad T of the lane, minus a zero-point: the signed bytes (q - z) * 2^(7-BITS), for BITS <= 7 and 0 <= z < 2^BITS.
// `up` has 128 - z * 2^(7-BITS) in every byte: with the code in bits 7-BITS .. 6 no byte carries into the next.
template <int BITS, int T>
__device__ __forceinline__ uint32_t quad_less(const uint32_t (&r)[4 * BITS], uint32_t up) {
  constexpr int bit = T * BITS, h = bit >> 3, p = bit & 7, TO = 7 - BITS;
  constexpr uint32_t ALL = 0x01010101u, CODE = ((1u << BITS) - 1u) << TO, SIGN = 0x80808080u;
  uint32_t x;
  if constexpr (p <= TO) {
    x = (r[h] & ((((1u << BITS) - 1u) << p) * ALL)) << (TO - p);
  } else if constexpr (p + BITS <= 8) {                            // the code ends its byte
    x = (r[h] >> 1) & (CODE * ALL);
  } else {
    constexpr int n1 = 8 - p;                                      // bits of the code in register h
    constexpr uint32_t LOW = ((1u << n1) - 1u) << TO, HIGH = CODE & ~LOW;
    x = ((r[h] >> (p - TO)) & (LOW * ALL)) | ((r[h + 1] << (n1 + TO)) & (HIGH * ALL));
  }
  return (x + up) ^ SIGN;
}

// LDS of a tile: A slabs, each wavefront's codes, scales, zero-points
template <int BITS, int BM, bool CORR>
struct A8Lds {
  static constexpr int BUF = BM * 128;
  // slabs of A in flight: two where LDS holds them for two workgroups per CU (160 KiB), else one
  static constexpr int A_AHEAD = BITS <= 7 ? 2 : 1, ABUFS = A_AHEAD + 1;
  static constexpr int W_AT = ABUFS * BUF, S_AT = W_AT + 4 * 1024 * BITS, Z_AT = S_AT + 4 * 256, BYTES = Z_AT + (CORR ? 4 * 256 : 0);
};

// Rows m0 .. m0 + BM - 1 of column tile tn over the chunks of a slab.  A split tile's partial sums are at number `tile` of
// the workspace, WS_BM rows each.
template <int BITS, int GPC, int BM, int WS_BM, bool SBF16, bool SPLIT, bool CORR>
__device__ __forceinline__ void a8_tile(const A8Params& p, uint8_t* lds, int tiles, int tile, int slab, int m0, int tn) {
  constexpr int RAW = 4 * BITS, MTS = BM / 16, A_LOADS = BM / 32;
  typedef A8Lds<BITS, BM, CORR> L;
  constexpr int BUF = L::BUF, A_AHEAD = L::A_AHEAD, ABUFS = L::ABUFS, W_AT = L::W_AT, S_AT = L::S_AT, Z_AT = L::Z_AT;

  const int tid = threadIdx.x, l = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = l >> 4, i16 = l & 15;
  const int KC = p.K / TILE_K, NCH = p.N / TILE_N;
  const int kbeg = slab * p.chunks_per_split, kend = min(KC, kbeg + p.chunks_per_split);
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
  const uint32_t lds_a = lds_base + 1024u * (uint32_t)w, lds_w = lds_base + W_AT + (uint32_t)(w * 1024 * BITS), lds_s = lds_base + S_AT + 256u * (uint32_t)w, lds_z = lds_base + Z_AT + 256u * (uint32_t)w;
  auto a_fetch = [&](int buf, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
      const uint32_t off = ((i & 1) ? a_vodd : a_voff) + (uint32_t)(32 * i) * (uint32_t)p.K;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(lds_a + (uint32_t)(buf * BUF + i * 4096)), "v"(off), "s"(a_rsrc), "s"(c * TILE_K) : "memory");
    }
  };

  // ---- W and its scales of the next chunk -> LDS too, for this wavefront alone ---------------------
  // (a register ring would not fit beside 128 accumulators).  One buffer is enough: the codes are
  // unpacked at the start of a chunk, and the load of the next ones starts right after that.
  // (scalar bases, 32-bit lane offsets)
  const uint8_t* wstrip = p.W + (int64_t)nc * KC * (1024 * BITS);
  // lanes 0..31 fetch two scales each of the chunk's (first) group, lanes 32..63 of its second group
  const uint8_t* sbase = reinterpret_cast<const uint8_t*>(p.S + TILE_N * nc);
  const uint32_t s_voff = 4u * (uint32_t)(l & 31) + (GPC == 2 ? 2u * (uint32_t)p.N * (uint32_t)(l >> 5) : 0u);
  // lanes 0..15 fetch four zero-points each of that group, lanes 16..31 of the second (no zero-points: valid
  // scale bytes instead, masked away)
  const uint8_t* zbase = (p.Z ? p.Z : reinterpret_cast<const uint8_t*>(p.S)) + TILE_N * nc;
  const uint32_t z_voff = 4u * (uint32_t)i16 + (GPC == 2 ? (uint32_t)p.N * (uint32_t)((l >> 4) & 1) : 0u);
  auto w_fetch = [&](int c) __attribute__((always_inline)) {
    const uint8_t* src = wstrip + (int64_t)c * (1024 * BITS);
#pragma unroll
    for (int i = 0; i < BITS; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(lds_w + (uint32_t)(i * 1024)), "v"(16u * (uint32_t)l), "s"(src + i * 1024) : "memory");
    const int g0 = (GPC > 1) ? GPC * c : ((c >> p.gshift) & p.gmask);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(lds_s), "v"(s_voff), "s"(sbase + 2 * (int64_t)g0 * p.N) : "memory");
    if constexpr (CORR)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(lds_z), "v"(z_voff), "s"(zbase + (int64_t)g0 * p.N) : "memory");
  };

  w_fetch(kbeg);
  a_fetch(0, kbeg);
  if constexpr (A_AHEAD == 2) a_fetch(1, min(kbeg + 1, kend - 1));

  f4_t acc[MTS][4];
#pragma unroll
  for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = (f4_t){0.f, 0.f, 0.f, 0.f};

  // ---- zero-points: z = zeros + zbias (zbias: intk codes are stored offset-binary) --------------------
  // What the unpack subtracts is z itself where z < 2^b (b <= 7), else nothing (8 bits: 128); `beyond` tells
  // a wavefront that its chunk has a zero-point of which something is left.
  const float left = (BITS == 8 ? 128.f : 0.f) - (float)p.zbias;
  constexpr uint32_t ALL = 0x01010101u, HALF = 1u << (BITS - 1);
  const uint32_t zmask = p.Z ? 0xffffffffu : 0u;
  const uint32_t zhalf = p.zbias ? HALF * ALL : 0u;
  const uint32_t zover = BITS == 8 ? 0u : ~((p.zbias ? HALF - 1u : 2u * HALF - 1u) * ALL);      // bits that zeros < 2^b - zbias do not have
  auto beyond = [&](uint32_t z4) __attribute__((always_inline)) { return BITS == 8 ? z4 ^ (zhalf ^ 0x80808080u) : z4 & zover; };
  // The sums are integers times the factor of the bytes, 2^SHIFT.  They are added to the bits of 1.5 * 2^(23 - SHIFT),
  // whose last bit is worth 2^-SHIFT, so the factor is gone when those are read as fp32.
  constexpr int SHIFT = CORR ? (BITS == 8 ? 0 : 7 - BITS) : 8 - BITS;
  constexpr int MAGIC = 0x4b400000 - (SHIFT << 23);
  constexpr float ORIGIN = 12582912.0f / (float)(1 << SHIFT);

  // my A fragment of row tile mt, k-step j: piece 4 j + b of row mt*16 + i16
  const int swz = (i16 ^ (i16 >> 3)) & 7;       // of row tile 0; row tile mt adds 2 mt to r >> 3
  __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0), in a form the compiler counts: nothing of its own is in flight in the loop
  __syncthreads();

  const i4_t magic = {MAGIC, MAGIC, MAGIC, MAGIC};
  int abuf_i = 0;
  auto zeros_of = [&](int g) __attribute__((always_inline)) {       // of my four columns as operand
    return *reinterpret_cast<const uint32_t*>(lds + Z_AT + 256 * w + 64 * g + 4 * i16) & zmask;
  };
  // One chunk.  ROWSUM: (what is left of) the zero-points goes through the row sums.
  auto chunk = [&](auto Rowsumc, int c) __attribute__((always_inline)) {
    constexpr bool ROWSUM = decltype(Rowsumc)::value;
    uint32_t raw[RAW];
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
      const u4_t q = *reinterpret_cast<const u4_t*>(lds + W_AT + (w * BITS + i) * 1024 + 16 * l);
      raw[4 * i + 0] = q.x; raw[4 * i + 1] = q.y; raw[4 * i + 2] = q.z; raw[4 * i + 3] = q.w;
    }
    u4_t s16[GPC][2], z16[GPC];                         // the chunk's scales (and zero-points) of my 16 columns
    uint32_t z4[GPC];
#pragma unroll
    for (int g = 0; g < GPC; ++g) {
      const u4_t* sp = reinterpret_cast<const u4_t*>(lds + S_AT + 256 * w + 128 * g + 32 * b);
      s16[g][0] = sp[0]; s16[g][1] = sp[1];
      if constexpr (ROWSUM) z16[g] = *reinterpret_cast<const u4_t*>(lds + Z_AT + 256 * w + 64 * g + 16 * b);
      else if constexpr (CORR && BITS <= 7) z4[g] = zeros_of(g);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // read: the buffers may be refilled
    const int abuf_n = abuf_i == 0 ? ABUFS - 1 : abuf_i - 1;        // the slab of the chunk before this one
    w_fetch(min(c + 1, kend - 1));
    a_fetch(abuf_n, min(c + A_AHEAD, kend - 1));
    u4_t wf[2][4];
    static_for<8>([&](auto Xc) __attribute__((always_inline)) {
      constexpr int X = decltype(Xc)::value, T0 = X * 4;
      if constexpr (CORR && BITS <= 7) {
        // byte NT of the zero-points, subtracted from 128, in every byte
        constexpr int G = (GPC == 2) ? X / 4 : 0, NT = X % 4;
        uint32_t up = 0x80808080u;
        if constexpr (!ROWSUM) up = __builtin_amdgcn_perm(0u, 0x80808080u - ((z4[G] | zhalf) << (7 - BITS)), NT * ALL);
        wf[X / 4][X % 4] = (u4_t){quad_less<BITS, T0>(raw, up), quad_less<BITS, T0 + 1>(raw, up), quad_less<BITS, T0 + 2>(raw, up), quad_less<BITS, T0 + 3>(raw, up)};
      } else {
        wf[X / 4][X % 4] = (u4_t){quad_top<BITS, T0>(raw), quad_top<BITS, T0 + 1>(raw), quad_top<BITS, T0 + 2>(raw), quad_top<BITS, T0 + 3>(raw)};
      }
    });

    const uint8_t* abuf = lds + abuf_i * BUF + i16 * 128;
    auto a_read = [&](int mt, int j) __attribute__((always_inline)) {
      return *reinterpret_cast<const i4_t*>(abuf + mt * 2048 + 16 * (((4 * j + b) ^ swz) ^ ((2 * mt) & 7)));
    };
    // The constants of a scale group: the scales, widened here and for good (the compiler would fold an fp16
    // one into mixed multiply-adds, at half the rate), and what is left to subtract: fp16 pairs (exact) where fp32
    // spills -- u8 on the shape above, group 128: 395 us against 452; group 64: 521 against 497.
    constexpr bool PAIRS = GPC == 1;
    float sf[16], nz[16];
    h2_t nz2[8];
    auto constants = [&](auto Gc) __attribute__((always_inline)) {
      constexpr int G = decltype(Gc)::value;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t two = s16[G][i >> 3][(i & 7) >> 1];
        if constexpr (SBF16) sf[i] = __builtin_bit_cast(float, (i & 1) ? (two & 0xffff0000u) : (two << 16));
        else sf[i] = (float)__builtin_bit_cast(h2_t, two)[i & 1];
        if constexpr (!SBF16) asm("" : "+v"(sf[i]));
      }
      if constexpr (ROWSUM) {
#pragma unroll
        for (int i = 0; i < (PAIRS ? 0 : 16); ++i) nz[i] = left - (float)((z16[G][i / 4] & zmask) >> (8 * (i % 4)) & 0xffu);
#pragma unroll
        for (int i = 0; i < (PAIRS ? 8 : 0); ++i) {     // from the bits of 1024 + z
          const _Float16 from = (_Float16)(1024.f + left);
          nz2[i] = (h2_t){from, from} - __builtin_bit_cast(h2_t, __builtin_amdgcn_perm(0x64646464u, z16[G][i / 2] & zmask, i % 2 ? 0x04030402u : 0x04010400u));
        }
      }
    };
    // value r of sub-tile nt: acc += scale * sum.  Below 2^22 the sum added to MAGIC is a change of the mantissa alone:
    // a subtraction instead of a convert (with several wavefronts on a SIMD fp32 add / multiply-add
    // issue every 2 clocks, converts and half-precision or mixed operations every 4).
    float rsum[2];                                      // ROWSUM: the row sums of two steps
    auto scale = [&](auto Fc, auto MTc, auto NTc, auto Rc, int bits) __attribute__((always_inline)) {
      constexpr int F = decltype(Fc)::value, MT = decltype(MTc)::value, NT = decltype(NTc)::value, R = decltype(Rc)::value;
      float t = __builtin_bit_cast(float, bits) - ORIGIN;
      if constexpr (ROWSUM) t = __builtin_fmaf(PAIRS ? (float)nz2[2 * R + NT / 2][NT % 2] : nz[4 * R + NT], rsum[F & 1], t);      // below 2^23: exact
      acc[MT][NT][R] = __builtin_fmaf(sf[4 * R + NT], t, acc[MT][NT][R]);
    };
    // The chunk is a sequence of steps -- a scale group and a row tile, group by group, so that one group's
    // constants are in registers -- of two units: two sub-tiles, i.e. 4 (group 64: 2) matrix
    // instructions.  Each instruction is followed by its share of the previous unit's eight
    // subtractions and multiply-adds (4, or 8), so vector and matrix work alternate within one
    // wavefront and the sums of two units (16 registers) are all that is in flight.
    constexpr int STEPS = GPC * MTS, JS = 2 / GPC, MPU = 2 * JS, VPM = 8 / MPU;      // steps, k-steps per step, instructions per unit, values per instruction
    i4_t a[2][JS], d[2][2], rs;
#pragma unroll
    for (int j = 0; j < JS; ++j) a[0][j] = a_read(0, j);
    static_for<2 * STEPS + 1>([&](auto Uc) __attribute__((always_inline)) {
      constexpr int U = decltype(Uc)::value, F = U / 2, G = F / MTS, H = U % 2;
      constexpr int PU = U - 1, PF = PU / 2, PMT = PF % MTS, PH = PU % 2;       // previous unit
      if constexpr (U % (2 * MTS) == 1) constants(std::integral_constant<int, G>{});
      if constexpr (ROWSUM && F < STEPS) {               // the row sums of this step, ready one unit later
        const i4_t ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
        if constexpr (H == 0) {
          rs = (i4_t){0, 0, 0, 0};
#pragma unroll
          for (int j = 0; j < JS; ++j) rs = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, a[F & 1][j], rs, 0, 0, 0);
        } else {
          rsum[F & 1] = (float)rs[0];
        }
      }
      static_for<MPU>([&](auto Ic) __attribute__((always_inline)) {
        constexpr int I = decltype(Ic)::value, J = I / 2, N = I % 2, NT = 2 * H + N;
        if constexpr (F < STEPS) {
          d[U & 1][N] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i4_t, wf[GPC == 2 ? G : J][NT]), a[F & 1][J], J == 0 ? magic : d[U & 1][N], 0, 0, 0);
          if constexpr (H == 0 && I < JS && F + 1 < STEPS)          // the next step's fragments
            a[(F + 1) & 1][I] = a_read((F + 1) % MTS, GPC == 2 ? (F + 1) / MTS : I);
        }
        if constexpr (U > 0) {
          static_for<VPM>([&](auto Vc) __attribute__((always_inline)) {
            constexpr int V = I * VPM + decltype(Vc)::value, PN = V / 4, R = V % 4;
            scale(std::integral_constant<int, PF>{}, std::integral_constant<int, PMT>{}, std::integral_constant<int, 2 * PH + PN>{},
                  std::integral_constant<int, R>{}, d[PU & 1][PN][R]);
          });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    // my part of the next chunk is in LDS (loads return in order: all but the newest slab)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(A_AHEAD == 2 ? A_LOADS : 0) : "memory");
    __syncthreads();
    abuf_i = abuf_i == ABUFS - 1 ? 0 : abuf_i + 1;
  };

  // From the first chunk on that has a zero-point beyond the codes, a wavefront uses the row sums.  (Two loops, one
  // after the other: two bodies in one loop cost 120 spilled registers.  Every wavefront meets one barrier per
  // chunk, whichever loop it is in.)
  int c = kbeg;
  for (; c < kend; ++c) {
    if constexpr (CORR) {
      uint32_t over = 0;
#pragma unroll
      for (int g = 0; g < GPC; ++g) over |= beyond(zeros_of(g));
      if (__builtin_amdgcn_ballot_w64(over != 0) != 0) break;
    }
    chunk(std::false_type{}, c);
  }
  if constexpr (CORR)
    for (; c < kend; ++c) chunk(std::true_type{}, c);

  if (!active) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the slab loaded past the end
  auto store_row = [&](int m, const f4_t (&v)[4]) __attribute__((always_inline)) {      // row scale, one rounding to the output type
    const float as = p.a_scale ? p.a_scale[m] : 1.0f;
    uint32_t o[8];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f2_t f = {v[2 * h][r] * as, v[2 * h + 1][r] * as};
        o[2 * r + h] = p.out_bf16 ? __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t))
                                  : __builtin_bit_cast(uint32_t, __builtin_convertvector(f, h2_t));
      }
    u4_t* dst = reinterpret_cast<u4_t*>(p.C + (int64_t)m * p.N + n16);
    dst[0] = (u4_t){o[0], o[1], o[2], o[3]};
    dst[1] = (u4_t){o[4], o[5], o[6], o[7]};
  };
  // ---- split-K: partial tiles meet in the workspace as in the 16-bit tiled kernel: a wavefront draws a ticket of its
  // 64-column strip; all but the last store their sums, count them as done and leave; the last keeps its own in
  // registers, waits for the count -- the others wait for nothing -- and adds the slabs in slab order (M = 200, K = N = 8192,
  // four slabs of 128-row tiles: 45.4 us when all stored and the last read one slab after the other, its own too, 43.0 now) ----
  if constexpr (SPLIT) {
    constexpr int SC1 = 16;                                   // cache policy: device coherence
    constexpr int AWAY = 0x40000000;                          // beyond the resource: loads give zeros, stores nothing
    auto ws_rsrc = [&](int sp) __attribute__((always_inline)) {
      return __builtin_amdgcn_make_buffer_rsrc(p.ws + ((int64_t)tile * p.splitk + sp) * (WS_BM * A8_BN), 0, BM * A8_BN * 4, 0x00020000);
    };
    auto ws_off = [&](int mt) __attribute__((always_inline)) { return m0 + mt * 16 + i16 < p.M ? 16 * tid : AWAY; };
    unsigned* ticket = p.tickets + ticket_stride(4 * tiles) * (4 * tile + w);
    unsigned drawn = 0;
    if (l == 0) drawn = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    drawn = __builtin_amdgcn_readfirstlane(drawn) & 0xffffu;
    if (drawn != (unsigned)(p.splitk - 1)) {
      const __amdgpu_buffer_rsrc_t mine = ws_rsrc(slab);
#pragma unroll
      for (int mt = 0; mt < MTS; ++mt) {
        const int off = ws_off(mt);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, acc[mt][nt]), mine, off, (mt * 4 + nt) * 4096, SC1);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // my partial strip is out before it counts as done
      if (l == 0) __hip_atomic_fetch_add(ticket, 0x10000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    (void)wait_for([&] { return __builtin_amdgcn_readfirstlane(__hip_atomic_load(ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 16; },
                   (unsigned)(p.splitk - 1), [] { __builtin_amdgcn_s_sleep(1); });
    asm volatile("" ::: "memory");                              // no slab is read ahead of the count
    if (l == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
    // R row tiles at a time, S slabs' loads in flight
    constexpr int R = 2, S = 4;
#pragma unroll
    for (int h = 0; h < MTS; h += R) {
      f4_t sum[R][4];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) sum[i][nt] = (f4_t){0.f, 0.f, 0.f, 0.f};
      for (int sp = 0; sp < p.splitk; sp += S) {
        u4_t x[S][R][4];
#pragma unroll
        for (int y = 0; y < S; ++y) {
          const __amdgpu_buffer_rsrc_t r = ws_rsrc(min(sp + y, p.splitk - 1));
#pragma unroll
          for (int i = 0; i < R; ++i) {
            const int off = sp + y < p.splitk && sp + y != slab ? ws_off(h + i) : AWAY;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) x[y][i][nt] = __builtin_amdgcn_raw_buffer_load_b128(r, off, ((h + i) * 4 + nt) * 4096, SC1);
          }
        }
#pragma unroll
        for (int y = 0; y < S; ++y)
          if (sp + y < p.splitk) {
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
              for (int nt = 0; nt < 4; ++nt) sum[i][nt] += sp + y == slab ? acc[h + i][nt] : __builtin_bit_cast(f4_t, x[y][i][nt]);
          }
      }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int m = m0 + (h + i) * 16 + i16;
        if (m < p.M) store_row(m, sum[i]);
      }
    }
    return;
  }

#pragma unroll
  for (int mt = 0; mt < MTS; ++mt) {
    const int m = m0 + mt * 16 + i16;
    if (m < p.M) store_row(m, acc[mt]);
  }
}

// Tiles of BM rows, or (BM = 128) `full` of 128 rows and `half` of 64.  The rows are cut into tiles_m row tiles of BM
// and, where at most 64 are left behind them, a last one of 64 (`half` tiles, one per column); of the former the last
// `cut` in panel order are computed as two halves (`half` tiles too: two each).  An XCD gets a run of either kind: `ahead` of the
// full ones, then its halves, then the rest.
template <int BITS, int GPC, int BM, bool SBF16, bool SPLIT, bool CORR>
__global__ __launch_bounds__(256, 2) void a8_large_kernel(A8Params p, int tiles_m, int tiles_n, int full, int half, int ahead) {
  typedef A8Lds<BITS, BM, CORR> L;
  static_assert(2 * L::BYTES <= 160 * 1024, "two workgroups per CU");
  __shared__ __attribute__((aligned(16))) uint8_t lds[L::BYTES];
  const int nfull = SPLIT ? full * p.splitk : full, nhalf = SPLIT ? half * p.splitk : half;
  const int xcd = (int)(blockIdx.x % 8), j = (int)(blockIdx.x / 8);
  const int fx = (nfull + 7) / 8, hx = (nhalf + 7) / 8, lead = min(fx, ahead);
  const int panel = A8_GROUP_M * tiles_n;
  auto position = [&](int tile, int* tm, int* tn) __attribute__((always_inline)) {
    const int first_m = (tile / panel) * A8_GROUP_M;
    const int gsize = min(tiles_m - first_m, A8_GROUP_M);
    *tm = first_m + (tile % panel) % gsize;
    *tn = (tile % panel) / gsize;
  };
  int tm, tn;
  if (BM == 64 || j < lead || j >= lead + hx) {
    const int at = j < lead ? j : j - hx, logical = xcd * fx + at;
    if (at >= fx || logical >= nfull) return;
    const int slab = SPLIT ? logical / full : 0, tile = SPLIT ? logical % full : logical;
    position(tile, &tm, &tn);
    a8_tile<BITS, GPC, BM, BM, SBF16, SPLIT, CORR>(p, lds, full + half, tile, slab, tm * BM, tn);
  } else if constexpr (BM == 128) {
    const int logical = xcd * hx + (j - lead);
    if (logical >= nhalf) return;
    const int slab = SPLIT ? logical / half : 0, i = SPLIT ? logical % half : logical;
    const int cut2 = 2 * (tiles_m * tiles_n - full);
    int m0;
    if (i < cut2) {
      position(full + i / 2, &tm, &tn);
      m0 = tm * 128 + 64 * (i & 1);
    } else {
      m0 = tiles_m * 128; tn = i - cut2;
    }
    a8_tile<BITS, GPC, 64, 128, SBF16, SPLIT, CORR>(p, lds, full + half, full + i, slab, m0, tn);
  }
}

#define QG_CAT2(a, b) a##b
#define QG_CAT(a, b) QG_CAT2(a, b)

template <int GPC, int BM, bool SBF16, bool SPLIT, bool CORR>
static int launch_one(const A8Params& p, int cut, hipStream_t st) {
  const bool last64 = BM == 128 && large_last64(p.M);
  const int tiles_m = last64 ? p.M / 128 : (p.M + BM - 1) / BM, tiles_n = (p.N + A8_BN - 1) / A8_BN;
  if (cut < 0 || cut > tiles_m * tiles_n || (cut && (BM != 128 || SPLIT))) return QG_EINVAL;
  const int full = tiles_m * tiles_n - cut, half = 2 * cut + (last64 ? tiles_n : 0);
  const int per_xcd = (full * p.splitk + 7) / 8 + (half * p.splitk + 7) / 8;
  hipLaunchKernelGGL((a8_large_kernel<QG_BITS, GPC, BM, SBF16, SPLIT, CORR>), dim3((unsigned)(8 * per_xcd)), dim3(256), 0, st, p, tiles_m, tiles_n, full, half, tiles_ahead(full));
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

template <int GPC, int BM, bool SBF16>
static int launch_scales(const A8Params& p, bool corr, int cut, hipStream_t st) {
  if (corr) return p.splitk > 1 ? launch_one<GPC, BM, SBF16, true, true>(p, cut, st) : launch_one<GPC, BM, SBF16, false, true>(p, cut, st);
  return p.splitk > 1 ? launch_one<GPC, BM, SBF16, true, false>(p, cut, st) : launch_one<GPC, BM, SBF16, false, false>(p, cut, st);
}

template <int BM>
static int launch_rows(const A8Params& p, bool corr, int cut, hipStream_t st) {
  if (p.group == 64) return p.scale_bf16 ? launch_scales<2, BM, true>(p, corr, cut, st) : launch_scales<2, BM, false>(p, corr, cut, st);
  return p.scale_bf16 ? launch_scales<1, BM, true>(p, corr, cut, st) : launch_scales<1, BM, false>(p, corr, cut, st);
}

// corr: zero-points, or uintk codes; bm: rows of a tile, 64 or 128; cut: so many of the latter as two halves
int QG_CAT(a8_large_launch_bits, QG_BITS)(const A8Params& p, bool corr, int bm, int cut, hipStream_t st) {
  if (bm == 64) return launch_rows<64>(p, corr, cut, st);
  if (bm == 128) return launch_rows<128>(p, corr, cut, st);
  return QG_EINVAL;
}

}  // namespace qg
