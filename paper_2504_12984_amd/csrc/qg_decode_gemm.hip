// Decode-sized matmul, M <= 64 (one to four tiles of 16 rows): the weights are streamed from HBM exactly once
// and the kernel is built to keep that stream saturated.
//
// One workgroup of NW wavefronts owns one 64-column strip of W and one slab of
// K; wavefront w takes every NW-th 128x64 chunk of the slab.  A wavefront keeps
// DEPTH chunks in flight at all times in a ring of registers (the software
// pipelining the paper calls essential, Sections "An Example of Tilus Program"
// and "End-to-End Performance"): per chunk BITS 16-byte loads of packed codes,
// four 16-byte loads of A per row tile (L2-resident), one load each of
// scales and zero-points.  The steady-state loop has no branches and refills a
// ring entry right after it has been consumed, so the compiler waits on exact
// outstanding-load counts instead of draining the queue.
// Codes are unpacked in registers and fed to the 16x16x32 matrix instruction
// with W as the row operand (the paper's load -> reinterpret -> cast -> mma
// pipeline, Section "Key Ideas", with no layout conversion and no trip through
// LDS).  From 13 or 16 rows on A passes through LDS where that pays (lds_rows, two_chunks_direct; two row tiles on four
// wavefronts load it directly), each wavefront's rows through a part of its own: the matrix
// instruction wants 16 rows in adjacent lanes, and loads in that order run at 16 bytes per clock and CU (a lane at a
// time), loads along the rows at 40 to 54.  M = 64, K = N = 8192, u4: 23.0 -> 19.7 us; M = 45 18.1 -> 16.8; M = 16, K = 8192,
// N = 28672, int4 27.6 -> 26.0, group 64 30.6 -> 27.7.  With fewer rows many lanes of a direct load share an address and the way
// through LDS costs more than it saves (M = 8 there 24.7 against 25.9).
// The K reduction runs inside the MFMA (across the four 8-wide k-blocks
// of lanes), then across the wavefronts through LDS, then -- when K is also
// split over workgroups -- through a binary tree of pairwise fp32 exchanges (the k-dimension parallelisation the paper names
// in Section "End-to-End Performance").
// Compiled once per weight type (QG_WT).
#include "qg_decode.h"
#include "qg_exchange.h"
#include "qg_static_for.h"

#ifndef QG_WT
#error "compile with -DQG_WT=<weight type index>"
#endif

namespace qg {

typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));

// Weights are used once: load them with the streaming (non-temporal) policy so that
// they do not push the re-used A rows out of the vector cache and L2 (measured:
// 5-10 % shorter kernels at 4..8 bits, M = 16).
__device__ __forceinline__ uint4 stream_load(const uint4* p) {
  u4_t v = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

template <int ROUTE>
__device__ __forceinline__ f4_t mfma16(u4_t w, u4_t a, f4_t c) {
  if constexpr (ROUTE == ROUTE_F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, w), __builtin_bit_cast(h8_t, a), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8_t, w), __builtin_bit_cast(b8_t, a), c, 0, 0, 0);
}

template <int ROUTE>
__device__ __forceinline__ uint32_t pack_out(float lo, float hi) {
  f2_t f = {lo, hi};
  if constexpr (ROUTE == ROUTE_F16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, h2_t));
  else return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t));
}

// MX: the scales are 8-bit exponents, one per 32 rows and column (GPC = 4), applied by the
// hardware converts of the e2m1 / e4m3 types; there are no zero-points.
// A_LDS: A through LDS; else loaded as the matrix instruction reads it.
template <int WT, int ROUTE, int GPC, int NW, int DEPTH, int MT, int NS, bool MX, bool A_LDS>
__global__ __launch_bounds__(NW * 64) void decode_kernel(GemmParams p) {
  // NS adjacent strips per workgroup, NK wavefronts along K for each: wavefront w
  // works on strip w % NS and takes every NK-th chunk of the slab starting at
  // w / NS, so the NS wavefronts with the same w / NS walk the same K range at the
  // same pace and find each other's A rows in the vector cache.
  constexpr int NK = NW / NS;
  static_assert(NW % NS == 0 && 16 % NK == 0, "wavefront grid");
  typedef Decoder<WT, ROUTE> D;
  constexpr int BITS = D::BITS, RAW = D::RAW;

  const int tid = threadIdx.x, l = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
  const int b = l >> 4, i16 = l & 15;
  const int ws = w % NS, wk = w / NS;                       // my strip and K position inside the workgroup
  const int KC = p.K / TILE_K, NCH = p.N / TILE_N;
  const int split = blockIdx.y;
  // Several strips per workgroup, K whole (so many strips that it is not split): adjacent strips on one XCD, whose L2 they
  // then share lines of scales and zero-points in.  Reading the weights alone, K = 8192, N = 28672, 4 bits, takes 18.3 us
  // this way and 19.9 dealt out in turn; the kernel, M = 1, u4 24.6 -> 23.8.  (One strip per workgroup, or split
  // K: up to 4 % longer; K <= 4096: u5, K = 2048, N = 30720 9.2 -> 9.5.)
  // (Chosen without a branch, and the workgroups counted from N: behind a branch, or with the grid's size from the launch, the
  // kernel's arguments come in two trips instead of one.  M = 1, u4, K = 1024, N = 32768 6.08 us with the branch, 5.93 now.)
  int group = blockIdx.x;
  if constexpr (NS > 1) {
    const int x = group & 7, groups = NCH / NS, run = x * (groups >> 3) + min(x, groups & 7) + (group >> 3);
    group = (p.splitk == 1 && KC > 32) ? run : group;
  }
  const int nc = group * NS + ws;
  const int c0 = split * p.chunks_per_split;
  const int c1 = min(KC, c0 + p.chunks_per_split);
  const int mine = (c1 - c0 > wk) ? (c1 - c0 - wk + NK - 1) / NK : 0;
  const int n0 = TILE_N * nc + 4 * i16;

  const uint4* wstrip = reinterpret_cast<const uint4*>(p.W + (int64_t)nc * KC * (1024 * BITS)) + l;
  // MT tiles of 16 rows; rows past M re-read row M-1, their results are never stored.
  // Through LDS: a load takes four rows x 256 bytes (buffer offsets below 2^31: 64 rows, K <= 2^24); eight lanes fill
  // 128 bytes of LDS.  A wavefront's slab is [k-step][row][4 pieces], piece q of row r at slot q ^ swizzle(r), so that
  // both the writes and the fragment reads find their banks apart.
  const uint16_t* arow[A_LDS ? 1 : MT];
#pragma unroll
  for (int mt = 0; mt < (A_LDS ? 1 : MT); ++mt) arow[mt] = p.A + (int64_t)min(mt * 16 + i16, p.M - 1) * p.K + 8 * b;
  const int apc = (l & 3) + 4 * ((l >> 3) & 3), ar4 = ((l >> 2) & 1) + 2 * (l >> 5);      // my piece of a row, my row of four
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.A), 0, (int)((uint32_t)p.M * (uint32_t)(2 * p.K)), 0x00020000);
  auto swizzle = [](int r) __attribute__((always_inline)) { return (((r >> 2) & 1) << 1) | (((r >> 1) ^ (r >> 3)) & 1); };
  constexpr int AQ = A_LDS ? 4 * MT : 1;                     // loads of a chunk's rows
  uint32_t a_off[AQ];
  int a_wr[4];
#pragma unroll
  for (int q = 0; q < AQ; ++q) a_off[q] = (uint32_t)min(4 * q + ar4, p.M - 1) * (uint32_t)(2 * p.K) + 16u * apc;
#pragma unroll
  for (int q = 0; q < 4; ++q) a_wr[q] = (apc >> 2) * (MT * 1024) + (4 * q + ar4) * 64 + 16 * ((apc & 3) ^ swizzle(4 * q + ar4));
  const int a_rd = i16 * 64 + 16 * (b ^ swizzle(i16));
  // no zero-points: read (valid) scale bytes instead and mask them away
  const uint8_t* zbase = p.Z ? p.Z : reinterpret_cast<const uint8_t*>(p.S);
  const uint32_t zmask = p.Z ? 0xffffffffu : 0u;

  // LDS: for codebook indices the replicated lookup table (built by all wavefronts while the first loads are in
  // flight), then a part for each wavefront: its rows of A during the main loop, its sums after it
  constexpr int LUT_BYTES = [] { if constexpr (D::IS_LUT) return D::TABLE_DWORDS * 4; else return 0; }();
  __shared__ __attribute__((aligned(16))) unsigned char lds_raw[LUT_BYTES + NW * MT * 4096];
  unsigned char* my_a = lds_raw + LUT_BYTES + w * (MT * 4096);

  // A in registers: as fragments two chunks like the weights; on its way to LDS two chunks with 16 wavefronts, else
  // one, loaded again as soon as it is in LDS (M = 16, K = 8192, N = 57344, u4, 16 wavefronts: 51.5 against 53.4 us;
  // eight with two chunks take more than the 128 registers that leave two workgroups on a CU: K = 8192,
  // N = 14336 19.6 against 16.6 us)
  constexpr int A_RING = !A_LDS || (NW == 16 && GPC == 1) ? DEPTH : 1;
  struct Stage {
    uint32_t r[RAW];
    uint2 s[GPC];          // GPC groups per chunk (group size 128 or more: 1; 64: 2; 32: 4)
    uint32_t z[GPC];
  };
  Stage st[DEPTH];
  u4_t ar[A_RING][4 * MT];

  auto issue_a = [&](auto Sc, int c) __attribute__((always_inline)) {
    constexpr int R = decltype(Sc)::value % A_RING;
    if constexpr (A_LDS) {
#pragma unroll
      for (int q = 0; q < AQ; ++q) ar[R][q] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (int)a_off[q], c * (2 * TILE_K), 0);
    } else {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) ar[R][4 * mt + j] = *reinterpret_cast<const u4_t*>(arow[mt] + c * TILE_K + 32 * j);
    }
  };
  auto issue = [&](auto Sc, int c) __attribute__((always_inline)) {
    constexpr int S = decltype(Sc)::value;
    Stage& s = st[S];
    __builtin_amdgcn_sched_barrier(0);         // stay below the last use of the entry being refilled,
                                               // so that the refill reuses the same registers
    if constexpr (A_RING == DEPTH) issue_a(Sc, c);
    const uint4* src = wstrip + (int64_t)c * (64 * BITS);
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
      uint4 q = stream_load(src + i * 64);
      s.r[4 * i + 0] = q.x; s.r[4 * i + 1] = q.y; s.r[4 * i + 2] = q.z; s.r[4 * i + 3] = q.w;
    }
    const int g0 = (GPC > 1) ? GPC * c : ((c >> p.gshift) & p.gmask);
    if constexpr (D::IS_LUT) {   // codebook indices: scales only
#pragma unroll
      for (int g = 0; g < GPC; ++g) s.s[g] = *reinterpret_cast<const uint2*>(p.S + (int64_t)(g0 + g) * p.N + n0);
      __builtin_amdgcn_sched_barrier(0);
      return;
    }
    if constexpr (MX) {          // four scale bytes (the lane's columns) per block of 32 rows, kept in the zero-point slot
#pragma unroll
      for (int g = 0; g < GPC; ++g)
        s.z[g] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(p.S) + (int64_t)(g0 + g) * p.N + n0);
      __builtin_amdgcn_sched_barrier(0);
      return;
    }
#pragma unroll
    for (int g = 0; g < GPC; ++g) {
      s.s[g] = *reinterpret_cast<const uint2*>(p.S + (int64_t)(g0 + g) * p.N + n0);
      s.z[g] = *reinterpret_cast<const uint32_t*>(zbase + (int64_t)(g0 + g) * p.N + n0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  f4_t acc[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = (f4_t){0.f, 0.f, 0.f, 0.f};

  typename D::Uniform u;
  u.init();
  // `next`: the chunk after this one, or none (-1)
  auto compute = [&](auto Sc, int next) __attribute__((always_inline)) {
    constexpr int S = decltype(Sc)::value;
    Stage& s = st[S];
    u4_t af[2][MT];                // fragments of this k-step and the next
    if constexpr (A_LDS) {
      // the lanes of a wavefront exchange rows: the last chunk's reads stay ahead of the writes, the writes ahead of the reads
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int q = 0; q < 4 * MT; ++q) *reinterpret_cast<u4_t*>(my_a + a_wr[q & 3] + (q >> 2) * 1024) = ar[S % A_RING][q];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if constexpr (A_RING == 1) {
        if (next >= 0) issue_a(Sc, next);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    auto fragments = [&](auto Jc) __attribute__((always_inline)) {
      constexpr int J = decltype(Jc)::value;
      if constexpr (J < 4)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          if constexpr (A_LDS) af[J & 1][mt] = *reinterpret_cast<const u4_t*>(my_a + a_rd + J * (MT * 1024) + mt * 1024);
          else af[J & 1][mt] = ar[S % A_RING][4 * mt + J];
        }
    };
    fragments(std::integral_constant<int, 0>{});
    if constexpr (MX) {
      static_assert(GPC == 4, "one scale block per k-step");
      static_for<4>([&](auto Jc) __attribute__((always_inline)) {
        constexpr int J = decltype(Jc)::value;
        fragments(std::integral_constant<int, J + 1>{});
        MxConsts mx;
        mx.make(s.z[J]);
        static_for<4>([&](auto NTc) __attribute__((always_inline)) {
          constexpr int NT = decltype(NTc)::value;
          uint32_t o[4];
          frag_mx<WT, ROUTE == ROUTE_BF16, J, NT>(s.r, mx, o);
          const u4_t wf = {o[0], o[1], o[2], o[3]};
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][NT] = mfma16<ROUTE>(wf, af[J & 1][mt], acc[mt][NT]);
        });
      });
      return;
    }
    typename D::Consts gc[GPC];
#pragma unroll
    for (int g = 0; g < GPC; ++g) D::make_consts(gc[g], s.s[g], D::IS_LUT ? 0u : (s.z[g] & zmask), p.zbias, p.scale_bf16);
    static_for<4>([&](auto Jc) __attribute__((always_inline)) {
      constexpr int J = decltype(Jc)::value;
      fragments(std::integral_constant<int, J + 1>{});
      static_for<4>([&](auto NTc) __attribute__((always_inline)) {
        constexpr int NT = decltype(NTc)::value;
        uint32_t o[4];
        D::template frag<J, NT>(s.r, gc[J * GPC / 4], u, o);          // k-step J lies in group J*GPC/4 of the chunk
        const u4_t wf = {o[0], o[1], o[2], o[3]};      // unpacked once, used by every row tile
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt][NT] = mfma16<ROUTE>(wf, af[J & 1][mt], acc[mt][NT]);
      });
    });
  };

  auto chunk_of = [&](int i) __attribute__((always_inline)) { return c0 + wk + min(i, mine - 1) * NK; };

  static_assert(!D::IS_LUT || NW * 64 >= 256, "one level per thread");
  uint32_t my_level = 0;
  if constexpr (D::IS_LUT) my_level = D::fetch(p.T, tid);
  // prologue: DEPTH chunks in flight (past-the-end stages re-load my last chunk)
  if (mine > 0) {
    if constexpr (A_RING == 1) issue_a(std::integral_constant<int, 0>{}, chunk_of(0));
    static_for<DEPTH>([&](auto Sc) __attribute__((always_inline)) { issue(Sc, chunk_of(decltype(Sc)::value)); });
  }
  if constexpr (D::IS_LUT) {      // (the levels are staged where nothing has been written yet)
    uint32_t* table = reinterpret_cast<uint32_t*>(lds_raw);
    D::build(table, reinterpret_cast<uint16_t*>(lds_raw + LUT_BYTES), my_level, tid, NW * 64);
    u.set_table(table, l);
  }
  if (mine > 0) {
    int i = 0;
    // steady state: no branches, so the compiler can wait on exact load counts
    for (; i + 2 * DEPTH <= mine; i += DEPTH)
      static_for<DEPTH>([&](auto Sc) __attribute__((always_inline)) {
        compute(Sc, chunk_of(i + decltype(Sc)::value + 1));
        issue(Sc, chunk_of(i + decltype(Sc)::value + DEPTH));
      });
    // drain
    auto after = [&](int n) __attribute__((always_inline)) { return n + 1 < mine ? chunk_of(n + 1) : -1; };
    static_for<DEPTH>([&](auto Sc) __attribute__((always_inline)) {
      constexpr int S = decltype(Sc)::value;
      if (i + S < mine) {
        compute(Sc, after(i + S));
        if (i + S + DEPTH < mine) issue(Sc, chunk_of(i + S + DEPTH));
      }
    });
    i += DEPTH;
    static_for<DEPTH>([&](auto Sc) __attribute__((always_inline)) {
      if (i + decltype(Sc)::value < mine) compute(Sc, after(i + decltype(Sc)::value));
    });
  }

  // ---- reduce over the NW wavefronts through LDS: all row tiles at once, each wavefront's sums where its A was -----
  float* red = reinterpret_cast<float*>(lds_raw + LUT_BYTES);      // [NW][MT][16 column offsets][64 lanes]
  constexpr int PER = 16 / NK;                             // column offsets per thread
  const int idx0 = PER * wk;
  float sum[MT][PER];
  if constexpr (A_LDS) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the last rows have been read
  // lanes whose row is past M carry nothing: they stay out of the LDS traffic, of the
  // split-K exchange and of the final store
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    if (mt * 16 + i16 < p.M) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((w * MT + mt) * 16 + 4 * r + nt) * 64 + l] = acc[mt][nt][r];   // column offset 4r + nt
    }
  __syncthreads();
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int e = 0; e < PER; ++e) sum[mt][e] = 0.f;
    if (mt * 16 + i16 < p.M) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        float t = 0.f;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) t += red[(((kk * NS + ws) * MT + mt) * 16 + idx0 + e) * 64 + l];
        sum[mt][e] = t;
      }
    }
  }

  // ---- split-K ------------------------------------------------------------------------------------
  if constexpr (MT <= 2) {
    if (p.splitk > 1) {
      constexpr int PAIR = PER >= 2 ? 2 : 1, NP = PER / PAIR;
      bool live[MT][NP];                                     // whose result is mine to store
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < NP; ++q) live[mt][q] = mt * 16 + i16 < p.M;
      if (!tree_exchange<MT, PER>(sum, live, p.slots, nc, NCH, split, p.splitk, idx0, l)) return;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < NP; ++q)
          if (live[mt][q]) {
            uint16_t* dst = p.C + (int64_t)(mt * 16 + i16) * p.N + TILE_N * nc + 16 * b + idx0;
            if constexpr (PAIR == 1) dst[q] = (uint16_t)(pack_out<ROUTE>(sum[mt][q], 0.f) & 0xffffu);
            else *reinterpret_cast<uint32_t*>(dst + 2 * q) = pack_out<ROUTE>(sum[mt][2 * q], sum[mt][2 * q + 1]);
          }
      return;
    }
  }
  if constexpr (MT > 2) if (p.splitk > 1) {
    int* last = reinterpret_cast<int*>(red);             // its sums are in registers by now
    // Three and four row tiles: too many sums for exchanges of 8 bytes (M = 64, K = N = 4096 in four slabs:
    // 13.1 us this way, 14.4 as a tree).  Partial tiles cross workgroups (and XCDs, whose L2s are not coherent with
    // each other) through device-scope relaxed atomics: such stores write
    // through and such loads bypass the local caches, so no cache-wide
    // write-back or invalidate is needed.  Order: my stores complete, barrier,
    // one arrival count per workgroup; the workgroup that counts splitk-1
    // earlier arrivals sums all tiles in split order, so the result does not
    // depend on arrival order.
    float* tile = p.ws + ((int64_t)split * NCH + nc) * (MT * 1024);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt * 16 + i16 < p.M) {
#pragma unroll
        for (int e = 0; e < PER; ++e)
          __hip_atomic_store(tile + mt * 1024 + (idx0 + e) * 64 + l, sum[mt][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // a workgroup barrier alone does not wait for global stores
    __syncthreads();
    if (tid == 0)
      *last = (__hip_atomic_fetch_add(&p.tickets[blockIdx.x], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(p.splitk - 1));
    __syncthreads();
    if (!*last) return;
    // all loads of a split are issued before the first add (independent accumulators)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < PER; ++e) sum[mt][e] = 0.f;
    for (int sp = 0; sp < p.splitk; ++sp) {
      const float* src = p.ws + ((int64_t)sp * NCH + nc) * (MT * 1024);
      float v[MT][PER];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          v[mt][e] = 0.f;
          if (mt * 16 + i16 < p.M)
            v[mt][e] = __hip_atomic_load(src + mt * 1024 + (idx0 + e) * 64 + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < PER; ++e) sum[mt][e] += v[mt][e];
    }
    if (tid == 0) __hip_atomic_store(&p.tickets[blockIdx.x], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = mt * 16 + i16;
    if (m < p.M) {
      uint16_t* dst = p.C + (int64_t)m * p.N + TILE_N * nc + 16 * b + idx0;
      if constexpr (PER == 1) {
        dst[0] = (uint16_t)(pack_out<ROUTE>(sum[mt][0], 0.f) & 0xffffu);
      } else {
#pragma unroll
        for (int e = 0; e + 1 < PER; e += 2) *reinterpret_cast<uint32_t*>(dst + e) = pack_out<ROUTE>(sum[mt][e], sum[mt][e + 1]);
      }
    }
  }
}

#define QG_CAT2(a, b) a##b
#define QG_CAT(a, b) QG_CAT2(a, b)

// One row tile: from how many rows on A goes through LDS (17: never).  u8 and i4 on K = 8192, N = 28672 (several strips)
// gain 2 to 5 % at 16 rows, 2 % at 13; one strip with 8 wavefronts 5 % at 16 rows (K = 8192, N = 14336, u4) and nothing
// below (K = N = 4096 3 % longer at 13), less unpacking nothing at all (e2m1, bf16 there 17.8 -> 18.3); with 4 wavefronts only group 32 gains (K = 4096, N = 28672 19.3 -> 17.2 us; u8 on
// K = N = 8192 13.3 -> 14.0).  16 wavefronts on one strip have half a chunk each at a time and nothing to hide the way behind
// (K = 4096, N = 14336, u3 8.6 -> 8.8); above 4 bits their registers do not hold it (f6, bf16, N = 28672 39 -> 49); and
// codebook lookups keep LDS busy already (4 bits, M = 16, N = 28672: two layers 59.5 -> 60.0).
// Four strips from 16 rows on (int4, M = 13, K = 2048, N = 57344 15.9 -> 17.1).
constexpr int lds_rows(int wt, int gpc, int nw, int ns) {
  if (wt_is_lut(wt) || (nw == 16 && (ns == 1 || wt_bits(wt) > 4)) || (ns == 1 && gpc < 4 && (nw == 4 || wt_natural(wt)))) return 17;
  return (ns > 1 && ns < 4) || gpc == 4 ? 13 : 16;
}

// Wavefronts with two chunks each have both in flight when A is loaded directly, and only the first one's rows on the way through LDS.
// Where the unpack is short enough for that to show they load it directly (16 rows: u4, K = 4096, N = 8192 6.9 us against 7.5, e2m2 8.1 against 8.9;
// u6, K = 2048, N = 16384 7.3 against 7.8; int3, K = 1024, N = 28672, two strips 6.1 against 6.7; u8, K = N = 4096 7.8 against 7.3, so not there).
constexpr bool two_chunks_direct(int wt, int nw, int ns, bool mx) {
  return !mx && (wt_bits(wt) <= 5 || (ns == 1 && nw == 8 && (wt_bits(wt) == 6 || wt >= 8)));
}

// DIRECT: A is loaded directly whatever lds_rows says.
template <int ROUTE, int GPC, int NW, int DEPTH, int MT, int NS = 1, bool MX = false, bool DIRECT = false>
static int launch_cfg(const GemmParams& p, hipStream_t st) {
  if ((p.N / TILE_N) % NS) return QG_EINVAL;
  constexpr int ROWS = DIRECT ? 17 : MT > 1 ? 0 : lds_rows(QG_WT, GPC, NW, NS);
  auto kern = decode_kernel<QG_WT, ROUTE, GPC, NW, DEPTH, MT, NS, MX, (ROWS <= 16)>;
  if constexpr (MT == 1 && ROWS <= 16)
    if (p.M < ROWS || (two_chunks_direct(QG_WT, NW, NS, MX) && p.chunks_per_split > NW / NS && p.chunks_per_split <= 2 * (NW / NS))) kern = decode_kernel<QG_WT, ROUTE, GPC, NW, DEPTH, MT, NS, MX, false>;
  dim3 grid((unsigned)(p.N / TILE_N / NS), (unsigned)p.splitk), block(NW * 64);
  hipLaunchKernelGGL(kern, grid, block, 0, st, p);
  return hipGetLastError() == hipSuccess ? QG_OK : QG_EHIP;
}

// variant = 10 * (row tiles: 1, 2, 3, 4) + arrangement.  One row tile: 0: 8 wavefronts on a strip, 1: 4, 2: 16, and
// those with several strips.  Several row tiles: 8 wavefronts, 1: on one strip, 6: 4 along K on each of two (two on a SIMD: one
// unpacks while the other's matrix instructions run; with 4 wavefronts M = 64, K = N = 8192 takes 20.5 us against 19.8, K = 8192,
// N = 28672 56.9 against 52.1, M = 32 there 42.5 against 38.4).  Also 4 wavefronts, 2: on one strip, 7: 2 along K on each of
// two, for the calls that four_wavefronts() in qg_api.hip names; two row tiles then load A directly.
template <int ROUTE, int GPC>
static int launch_variant(const GemmParams& p, int variant, hipStream_t st) {
  if constexpr (GPC == 4 && (QG_WT == 9 || QG_WT == 13)) {
    if (p.scale_e8m0) {              // block-scaled e2m1 / e4m3: every arrangement, scaled converts
      switch (variant) {
        case 10: return launch_cfg<ROUTE, 4, 8, 2, 1, 1, true>(p, st);
        case 11: return launch_cfg<ROUTE, 4, 4, 2, 1, 1, true>(p, st);
        case 12: return launch_cfg<ROUTE, 4, 16, 2, 1, 1, true>(p, st);
        case 14: return launch_cfg<ROUTE, 4, 8, 2, 1, 2, true>(p, st);
        case 15: return launch_cfg<ROUTE, 4, 16, 2, 1, 2, true>(p, st);
        case 16: return launch_cfg<ROUTE, 4, 16, 2, 1, 4, true>(p, st);
        case 21: return launch_cfg<ROUTE, 4, 8, 2, 2, 1, true>(p, st);
        case 22: return launch_cfg<ROUTE, 4, 4, 2, 2, 1, true, true>(p, st);
        case 27: return launch_cfg<ROUTE, 4, 4, 2, 2, 2, true, true>(p, st);
        case 26: return launch_cfg<ROUTE, 4, 8, 2, 2, 2, true>(p, st);
        case 31: return launch_cfg<ROUTE, 4, 8, 2, 3, 1, true>(p, st);
        case 32: return launch_cfg<ROUTE, 4, 4, 2, 3, 1, true>(p, st);
        case 36: return launch_cfg<ROUTE, 4, 8, 2, 3, 2, true>(p, st);
        case 37: return launch_cfg<ROUTE, 4, 4, 2, 3, 2, true>(p, st);
        case 46: return launch_cfg<ROUTE, 4, 8, 2, 4, 2, true>(p, st);
        case 47: return launch_cfg<ROUTE, 4, 4, 2, 4, 2, true>(p, st);
        case 41: return launch_cfg<ROUTE, 4, 8, 2, 4, 1, true>(p, st);
        case 42: return launch_cfg<ROUTE, 4, 4, 2, 4, 1, true>(p, st);
        default: return QG_EINVAL;
      }
    }
  }
  if (p.scale_e8m0) return QG_EUNSUPPORTED;
  if constexpr (GPC == 4) {          // group size 32: the one-strip arrangements only
    switch (variant) {
      case 11: return launch_cfg<ROUTE, 4, 4, 2, 1>(p, st);
      case 21: return launch_cfg<ROUTE, 4, 8, 2, 2>(p, st);
      case 22: return launch_cfg<ROUTE, 4, 4, 2, 2, 1, false, true>(p, st);
      case 32: return launch_cfg<ROUTE, 4, 4, 2, 3>(p, st);
      case 42: return launch_cfg<ROUTE, 4, 4, 2, 4>(p, st);
      case 31: if constexpr (wt_bits(QG_WT) <= 5) return launch_cfg<ROUTE, 4, 8, 2, 3>(p, st); else return QG_EINVAL;
      case 41: if constexpr (wt_bits(QG_WT) <= 5) return launch_cfg<ROUTE, 4, 8, 2, 4>(p, st); else return QG_EINVAL;
      default: return QG_EINVAL;
    }
  } else {
  switch (variant) {
    case 10: return launch_cfg<ROUTE, GPC, 8, 2, 1>(p, st);
    case 11: return launch_cfg<ROUTE, GPC, 4, 2, 1>(p, st);
    case 12: return launch_cfg<ROUTE, GPC, 16, 2, 1>(p, st);
    case 14: return launch_cfg<ROUTE, GPC, 8, 2, 1, 2>(p, st);     // 2 strips x 4
    case 15: return launch_cfg<ROUTE, GPC, 16, 2, 1, 2>(p, st);    // 2 strips x 8
    case 16: return launch_cfg<ROUTE, GPC, 16, 2, 1, 4>(p, st);    // 4 strips x 4
    case 21: return launch_cfg<ROUTE, GPC, 8, 2, 2>(p, st);
    case 22: return launch_cfg<ROUTE, GPC, 4, 2, 2, 1, false, true>(p, st);
    case 27: return launch_cfg<ROUTE, GPC, 4, 2, 2, 2, false, true>(p, st);     // 2 strips x 2
    case 26: return launch_cfg<ROUTE, GPC, 8, 2, 2, 2>(p, st);     // 2 row tiles, 2 strips x 4
    case 31: return launch_cfg<ROUTE, GPC, 8, 2, 3>(p, st);
    case 32: return launch_cfg<ROUTE, GPC, 4, 2, 3>(p, st);
    case 36: return launch_cfg<ROUTE, GPC, 8, 2, 3, 2>(p, st);     // 3 row tiles, 2 strips x 4
    case 37: return launch_cfg<ROUTE, GPC, 4, 2, 3, 2>(p, st);
    case 42: return launch_cfg<ROUTE, GPC, 4, 2, 4>(p, st);
    case 46: return launch_cfg<ROUTE, GPC, 8, 2, 4, 2>(p, st);     // 4 row tiles, 2 strips x 4
    case 47: return launch_cfg<ROUTE, GPC, 4, 2, 4, 2>(p, st);
    case 41: return launch_cfg<ROUTE, GPC, 8, 2, 4>(p, st);
    default: return QG_EINVAL;
  }
  }
}

// number of wavefronts along K per strip of a variant (the host sizes split-K with it)
int QG_CAT(decode_waves_wt, QG_WT)(int variant) {
  switch (variant) {
    case 10: case 15: case 21: case 31: case 41: return 8;
    case 12: return 16;
    case 27: case 37: case 47: return 2;
    default: return 4;
  }
}

int QG_CAT(decode_launch_wt, QG_WT)(const GemmParams& p, int route, int variant, hipStream_t st) {
  const int gpc = (p.group == 32) ? 4 : (p.group == 64) ? 2 : 1;       // groups per 128-row chunk
  if (route == ROUTE_F16)
    return gpc == 4 ? launch_variant<ROUTE_F16, 4>(p, variant, st)
         : gpc == 2 ? launch_variant<ROUTE_F16, 2>(p, variant, st) : launch_variant<ROUTE_F16, 1>(p, variant, st);
  return gpc == 4 ? launch_variant<ROUTE_BF16, 4>(p, variant, st)
       : gpc == 2 ? launch_variant<ROUTE_BF16, 2>(p, variant, st) : launch_variant<ROUTE_BF16, 1>(p, variant, st);
}

}  // namespace qg
