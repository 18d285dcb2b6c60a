// C ABI of the library: argument checks, kernel choice, workspace.  No compute
// happens on the host.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <string>

#include "qg_common.h"

namespace qg {

int launch_pack_codes(const uint8_t*, int, int64_t, uint8_t*, hipStream_t);
int launch_probe_stream(const void*, size_t, void*, hipStream_t);
int launch_probe_mfma(int, int, int, int, void*, hipStream_t);
int launch_repack(const uint8_t*, int, int, int, uint32_t, int, int, uint8_t*, hipStream_t);

#define QG_FOR_ALL_WT(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13)

#define QG_DECL(i)                                                            \
  int dequant_launch_wt##i(const DequantParams&, int, hipStream_t);           \
  int decode_launch_wt##i(const GemmParams&, int, int, hipStream_t);          \
  int decode_waves_wt##i(int);                                                \
  int large_launch_wt##i(const GemmParams&, int, int, hipStream_t);          \
  int large32_launch_wt##i(const GemmParams&, int, int, hipStream_t);        \
  int gemv_launch_wt##i(const GemmParams&, int, int, hipStream_t);
QG_FOR_ALL_WT(QG_DECL)
#undef QG_DECL
int large_launch_wt14(const GemmParams&, int, int, hipStream_t);
int launch_reduce_tiles(const GemmParams&, int, int, hipStream_t);
int launch_clear(void*, size_t, hipStream_t);
// codebook indices of 1..8 bits: kernel-side weight types WT_LUT0 .. WT_LUT0 + 7
#define QG_FOR_ALL_LUT(X) X(15) X(16) X(17) X(18) X(19) X(20) X(21) X(22)
#define QG_DECL(i)                                                            \
  int dequant_launch_wt##i(const DequantParams&, int, hipStream_t);           \
  int decode_launch_wt##i(const GemmParams&, int, int, hipStream_t);          \
  int large_launch_wt##i(const GemmParams&, int, int, hipStream_t);
QG_FOR_ALL_LUT(QG_DECL)
#undef QG_DECL
#define QG_DECL_A8(b) int a8_launch_bits##b(const A8Params&, int, int, hipStream_t);
QG_DECL_A8(1) QG_DECL_A8(2) QG_DECL_A8(3) QG_DECL_A8(4) QG_DECL_A8(5) QG_DECL_A8(6) QG_DECL_A8(7) QG_DECL_A8(8)
#undef QG_DECL_A8
#define QG_DECL_A8(b) int a8_large_launch_bits##b(const A8Params&, bool, int, int, hipStream_t);
QG_DECL_A8(1) QG_DECL_A8(2) QG_DECL_A8(3) QG_DECL_A8(4) QG_DECL_A8(5) QG_DECL_A8(6) QG_DECL_A8(7) QG_DECL_A8(8)
#undef QG_DECL_A8
typedef int (*a8_fn)(const A8Params&, int, int, hipStream_t);
typedef int (*a8_large_fn)(const A8Params&, bool, int, int, hipStream_t);
static const a8_large_fn kA8Large[8] = {a8_large_launch_bits1, a8_large_launch_bits2, a8_large_launch_bits3, a8_large_launch_bits4,
                                        a8_large_launch_bits5, a8_large_launch_bits6, a8_large_launch_bits7, a8_large_launch_bits8};
static const a8_fn kA8[8] = {a8_launch_bits1, a8_launch_bits2, a8_launch_bits3, a8_launch_bits4,
                             a8_launch_bits5, a8_launch_bits6, a8_launch_bits7, a8_launch_bits8};

typedef int (*dq_fn)(const DequantParams&, int, hipStream_t);
typedef int (*gm_fn)(const GemmParams&, int, int, hipStream_t);
#define QG_ENT(i) dequant_launch_wt##i,
static const dq_fn kDequant[NUM_WT] = {QG_FOR_ALL_WT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) large_launch_wt##i,
static const gm_fn kLarge[NUM_WT] = {QG_FOR_ALL_WT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) large32_launch_wt##i,
static const gm_fn kLarge32[NUM_WT] = {QG_FOR_ALL_WT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) decode_launch_wt##i,
static const gm_fn kDecode[NUM_WT] = {QG_FOR_ALL_WT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) gemv_launch_wt##i,
static const gm_fn kGemv[NUM_WT] = {QG_FOR_ALL_WT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) dequant_launch_wt##i,
static const dq_fn kDequantLut[NUM_LUT] = {QG_FOR_ALL_LUT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) decode_launch_wt##i,
static const gm_fn kDecodeLut[NUM_LUT] = {QG_FOR_ALL_LUT(QG_ENT)};
#undef QG_ENT
#define QG_ENT(i) large_launch_wt##i,
static const gm_fn kLargeLut[NUM_LUT] = {QG_FOR_ALL_LUT(QG_ENT)};
#undef QG_ENT
typedef int (*waves_fn)(int);
#define QG_ENT(i) decode_waves_wt##i,
static const waves_fn kDecodeWaves[NUM_WT] = {QG_FOR_ALL_WT(QG_ENT)};
#undef QG_ENT

static thread_local std::string g_last_error;
// Experiment overrides (qg_set_knob): process-wide, read once per call with relaxed loads.
static std::atomic<int> g_knob[4] = {{0}, {0}, {0}, {0}};
static int knob(int i) { return g_knob[i].load(std::memory_order_relaxed); }

// A failed call's error is reported by the status, so it is read away here: the runtime keeps it until
// hipGetLastError, and the check behind the next launch would take it for that launch's.
static int hip_fail(hipError_t e, const char* what) {
  (void)hipGetLastError();
  g_last_error = std::string(what) + ": " + hipGetErrorString(e);
  return QG_EHIP;
}

// ---- split-K workspace (partial sums + arrival counters) -----------------------------------
// What the automatic plans can ask for is bounded: the streaming kernel splits K only while
// strips x slabs stay below 512 (16 KiB of partial sums each at most), the tiled kernel only
// while tiles x slabs stay within 256 (at most 128 x 256 fp32 each), the int8 one within 512 and this size.  So every workspace has
// this one capacity; only forced split factors (the experiment knobs) can exceed it.
constexpr size_t WS_PARTIAL_BYTES = size_t(32) << 20;
// Behind them the slots in which the streaming kernel's slabs meet (up to two row tiles: 8 KiB per strip and
// slab), zero between calls, so that they cannot share memory with sums that stay behind.
constexpr size_t WS_SLOT_BYTES = size_t(4) << 20;
constexpr size_t WS_BYTES = WS_PARTIAL_BYTES + WS_TICKETS * sizeof(unsigned) + WS_SLOT_BYTES;

// qgemm: one workspace per device and stream.  Kernels of one stream run in order, so they
// can share a workspace; kernels of different streams may overlap, so each stream gets its
// own.  It is allocated once, on the first call of that (device, stream) that splits K, at
// the fixed capacity, and never freed or moved, so a HIP graph captured later keeps valid
// pointers.  (A forced split beyond the capacity gets a larger block; the old one is kept
// allocated for the same reason.)  The counters and slots are zeroed by a memset enqueued on the
// stream ahead of the first kernel; nothing synchronises.
struct Workspace {
  int dev = -1;
  hipStream_t stream = nullptr;
  unsigned char* base = nullptr;
  size_t partial_bytes = 0;
  size_t ticket_count = 0;
};
static std::mutex g_ws_mutex;
static Workspace g_ws[32];
static int g_ws_used = 0;

static int get_workspace(size_t partial_bytes, size_t ticket_count, hipStream_t st, float** partial, unsigned** tickets, void** slots = nullptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  Workspace* found = nullptr;
  for (int i = 0; i < g_ws_used; ++i)
    if (g_ws[i].dev == dev && g_ws[i].stream == st) { found = &g_ws[i]; break; }
  if (!found) {
    if (g_ws_used == 32) { g_last_error = "split-K workspaces for more than 32 (device, stream) pairs"; return QG_EUNSUPPORTED; }
    found = &g_ws[g_ws_used++];
    found->dev = dev; found->stream = st;
  }
  Workspace& w = *found;
  if (w.partial_bytes < partial_bytes || w.ticket_count < ticket_count) {
    // Never under capture, not even where the capture mode allows hipMalloc: the memset would become a node of the
    // graph, and the counters would count as cleared for calls that run before it.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) { (void)hipGetLastError(); cap = hipStreamCaptureStatusNone; }      // hipMalloc will tell
    if (cap != hipStreamCaptureStatusNone) { g_last_error = "split-K workspace: none yet on a stream that is being captured"; return QG_EHIP; }
    const size_t pb = partial_bytes < WS_PARTIAL_BYTES ? WS_PARTIAL_BYTES : ((partial_bytes + 255) & ~size_t(255));
    const size_t tc = ticket_count < WS_TICKETS ? WS_TICKETS : ticket_count;
    unsigned char* block = nullptr;
    const size_t cleared = ((tc * sizeof(unsigned) + 255) & ~size_t(255)) + WS_SLOT_BYTES;
    e = hipMalloc(&block, pb + cleared);
    if (e != hipSuccess) return hip_fail(e, "hipMalloc(workspace)");
    // counters and slots start at zero; every kernel that uses them leaves them at zero
    e = hipMemsetAsync(block + pb, 0, cleared, st);
    if (e != hipSuccess) { (void)hipFree(block); return hip_fail(e, "hipMemsetAsync(tickets)"); }
    w.base = block; w.partial_bytes = pb; w.ticket_count = tc;      // an earlier, smaller block stays allocated
  }
  *partial = reinterpret_cast<float*>(w.base);
  *tickets = reinterpret_cast<unsigned*>(w.base + w.partial_bytes);
  if (slots) *slots = w.base + w.partial_bytes + ((w.ticket_count * sizeof(unsigned) + 255) & ~size_t(255));
  return QG_OK;
}

// qgemm_noalloc: the same workspace as one fixed array in device memory, part of the code
// object (zero when it is loaded), one copy per GPU.  Its address on a device is looked up
// once, with that device current, and kept; host code never uses the array's name otherwise.
// Partial sums need no clearing (a call reads back only what it has written itself);
// every arrival counter and exchange slot is returned to zero by the kernel that used it.
static __device__ __align__(256) unsigned char scratch[WS_BYTES];
static std::mutex g_scratch_mutex;
static unsigned char* g_scratch_ptr[64] = {};

// Looks the array's address up on the current device (first call there) and keeps it.
static int static_scratch_base(unsigned char** base) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= 64) { g_last_error = "qgemm_noalloc: device index beyond 63"; return QG_EUNSUPPORTED; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
  }
  *base = g_scratch_ptr[dev];
  return QG_OK;
}

static int get_static_scratch(size_t partial_bytes, size_t ticket_count, float** partial, unsigned** tickets, void** slots) {
  if (partial_bytes > WS_PARTIAL_BYTES || ticket_count > WS_TICKETS) {
    g_last_error = "qgemm_noalloc: this call needs " + std::to_string(partial_bytes) + " bytes of split-K partial sums and " +
                   std::to_string(ticket_count) + " arrival counters; the fixed scratch holds " +
                   std::to_string(WS_PARTIAL_BYTES) + " bytes and " + std::to_string(WS_TICKETS) + " counters";
    return QG_EUNSUPPORTED;
  }
  unsigned char* base = nullptr;
  int rc = static_scratch_base(&base);
  if (rc != QG_OK) return rc;
  *partial = reinterpret_cast<float*>(base);
  *tickets = reinterpret_cast<unsigned*>(base + WS_PARTIAL_BYTES);
  *slots = base + WS_PARTIAL_BYTES + WS_TICKETS * sizeof(unsigned);
  return QG_OK;
}

// Counters of the tiled kernels, one per 64-column strip of a tile.
static size_t tile_tickets(int64_t tiles) { return (size_t)(4 * tiles * ticket_stride(4 * tiles)); }

enum WsMode { WS_PER_STREAM = 0, WS_STATIC = 1 };
static int acquire_ws(int mode, size_t partial_bytes, size_t ticket_count, hipStream_t st, GemmParams& p) {
  return mode == WS_STATIC ? get_static_scratch(partial_bytes, ticket_count, &p.ws, &p.tickets, &p.slots)
                           : get_workspace(partial_bytes, ticket_count, st, &p.ws, &p.tickets, &p.slots);
}

// Slots for a streaming kernel's exchange, in a workspace acquired for the partial sums of all its slabs.  More
// than the workspace has (a forced split factor) lie where the partial sums would, cleared ahead of the kernel.
static int exchange_slots(int splitk, int strips, int row_tiles, float* partial, hipStream_t st, void** slots) {
  const size_t bytes = (size_t)(splitk - 1) * strips * (size_t)(row_tiles * 16 * TILE_N) * sizeof(float);
  if (row_tiles > 2 || bytes <= WS_SLOT_BYTES) return QG_OK;
  *slots = partial;
  return launch_clear(partial, bytes, st);
}

// ---- buffer of the de-quantise-first path (forced path 4) -------------------------------------
// The whole weight in 16 bits, K*N*2 bytes, rewritten by every call: one buffer per (device,
// stream), allocated on first use and replaced (after the stream has drained) when a larger
// weight arrives.  Only this explicitly selected path allocates beyond the fixed workspace.
struct DenseBuffer { int dev = -1; hipStream_t stream = nullptr; void* ptr = nullptr; size_t bytes = 0; };
static DenseBuffer g_dense[32];
static int g_dense_used = 0;

static int get_dense_buffer(size_t bytes, hipStream_t st, void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  DenseBuffer* found = nullptr;
  for (int i = 0; i < g_dense_used; ++i)
    if (g_dense[i].dev == dev && g_dense[i].stream == st) { found = &g_dense[i]; break; }
  if (!found) {
    if (g_dense_used == 32) { g_last_error = "de-quantised weight buffers for more than 32 (device, stream) pairs"; return QG_EUNSUPPORTED; }
    found = &g_dense[g_dense_used++];
    found->dev = dev; found->stream = st;
  }
  if (found->bytes < bytes) {
    if (found->ptr) {
      e = hipStreamSynchronize(st);                    // earlier calls on the stream may still read the old buffer
      if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
      (void)hipFree(found->ptr);
      found->ptr = nullptr; found->bytes = 0;
    }
    e = hipMalloc(&found->ptr, bytes);
    if (e != hipSuccess) return hip_fail(e, "hipMalloc(de-quantised weight)");
    found->bytes = bytes;
  }
  *out = found->ptr;
  return QG_OK;
}

static bool layout_ok(int layout) { return layout == QG_LAYOUT_TILE128x64 || layout == QG_LAYOUT_TILE128x64_R32; }
static bool pack_layout_ok(int layout) { return layout_ok(layout) || layout == QG_LAYOUT_TILE128x64_I8; }
static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// `codebook`: the call brought a table of levels (the *_codebook entry points); a codebook weight
// type needs one and no other type takes one.
static int check_common(qg_wtype t, int layout, int act, int scale_dtype, int64_t group, int64_t K, int64_t N,
                        int* wt_out, int* route_out, bool codebook = false) {
  if (!layout_ok(layout)) return QG_EINVAL;
  int wt = wt_index(t);
  if (wt == -2) return QG_EUNSUPPORTED;
  if (wt < 0) return QG_EINVAL;
  if (wt_is_lut(wt) != codebook) return QG_EINVAL;
  if (codebook && (layout != QG_LAYOUT_TILE128x64 || scale_dtype == QG_E8M0)) return QG_EUNSUPPORTED;
  if (K <= 0 || N <= 0 || K % TILE_K || N % TILE_N || K > (1 << 24) || N > (1 << 24)) return QG_EINVAL;
  if (group <= 0 || K % group) return QG_EINVAL;
  if (!((group % TILE_K) == 0 || group == 64 || group == 32)) return QG_EINVAL;
  if ((act != QG_F16 && act != QG_BF16) || (scale_dtype != QG_F16 && scale_dtype != QG_BF16 && scale_dtype != QG_E8M0)) return QG_EINVAL;
  if (act == QG_F16 && scale_dtype == QG_BF16) return QG_EUNSUPPORTED;
  // power-of-two block scales: 32 rows per scale, e2m1 / e4m3 codes (the scaled hardware converts), first layout
  if (scale_dtype == QG_E8M0 && (group != 32 || !(wt == 9 || wt == 13) || layout != QG_LAYOUT_TILE128x64)) return QG_EUNSUPPORTED;
  *wt_out = wt;
  *route_out = (act == QG_F16) ? ROUTE_F16 : ROUTE_BF16;
  return QG_OK;
}

// tiles of 16 rows a wavefront of the streaming kernel carries for M rows (M <= 64)
static int row_tiles(int64_t M) { return M <= 16 ? 1 : (M <= 32 ? 2 : 4); }

// Whether an arrangement (its tens are its row tiles) serves M rows: it has the row tiles they need, and not
// twice as many or more.
static bool covers_rows(int variant, int64_t M) {
  return variant / 10 == row_tiles(M) || (variant / 10 == 3 && M > 32 && M <= 48);
}

// Three and four row tiles, both with A through LDS (770 calls, M = 33 .. 64; times: eight wavefronts against four).
static bool four_wavefronts_many(bool four_tiles, int NCH, int KC, int group, int wt, bool one_strip, bool mx) {
  const int bits = wt_bits(wt);
  const bool lut = wt_is_lut(wt), narrow_lut = lut && bits <= 4;
  // four groups' constants, or four row tiles, beside wide codes do not fit the registers of eight (spilled bytes a lane, two groups a chunk, f16 / bf16
  // activations: u8 60 / 60, u7 36 / 92, e4m3 36 / 28, with one 24 / 68, e3m2 16 / 36, u6 12 / 16, which is too little to matter with one.  M = 64:
  // u8, K = 2048, N = 16384 15.1 us against 13.5, group 64, K = 1024, N = 14336 11.6 against 8.7; bf16, K = N = 8192: u7, group 64 29.7 against 24.7, e4m3 27.9
  // against 23.3, e3m2 24.8 against 23.3; group 32, u8 39.2 against 29.4)
  if (group == 32 && !mx && bits > 5) return true;
  if (four_tiles && !lut && ((wt < 8 && bits + (group == 64 ? 1 : 0) >= 7) || wt == 11 || wt == 13)) return true;
  if (one_strip) {
    if (narrow_lut) return !four_tiles && NCH > 256;      // (building the table costs what four leave: M = 40, K = 512, N = 24640 12.4 against 9.6)
    // one chunk for each of eight, two for each of four (M = 33, u8, K = 1024, N = 16384 8.5 against 7.6); a round and a fraction, or all CUs just
    // full (M = 33, u8, K = 1024, N = 24640 14.3 against 10.2; M = 40, u4, K = 2048, N = 16384 10.2 against 9.5)
    return (KC <= 8 && (four_tiles || KC <= 4 || KC >= 7)) || (!four_tiles && (NCH > 256 || (NCH > 224 && !lut)));
  }
  // pairs of strips: short K (M = 52, 8-bit codebook, K = 1024, N = 32768 19.6 against 17.7; M = 40, e3m2, K = 512, N = 28672 8.2 against 7.3), several rounds
  if (narrow_lut) return !four_tiles && NCH > 512;
  return (NCH >= 384 && KC <= 4) || (four_tiles && lut && KC <= 8) || (!four_tiles && NCH > 512);
}

// Several row tiles: four wavefronts instead of eight?  Two row tiles: they load A directly (22, 27), eight through LDS (21, 26).  Both sides timed over 1372
// calls (M = 17 .. 32, K = 512 .. 16384, N = 512 .. 57344, all widths, kinds and groups): what this picks takes 0.2 % longer than the better
// of the two on average, 1 call in 35 more than 3 %.  Eight (158 registers each, u4) have a CU to themselves, of four two or three workgroups share one.
static bool four_wavefronts(int M, int NCH, int KC, int splitk, int group, int wt, bool one_strip, bool mx) {
  const int bits = wt_bits(wt);
  if (M > 32) return four_wavefronts_many(M > 48, NCH, KC, group, wt, one_strip, mx);
  const bool lut = wt_is_lut(wt), codes_float = !lut && !mx && wt >= 8, few = M <= 24;
  // several rounds of the 256 CUs (M = 20, u4, K = 1024, N = 57344: 12.1 us against 14.8; codebook of 6 bits, K = 2048, N = 41024 24.2 against 32.7)
  if (NCH > 512) return few || KC <= 16 || lut;
  // a round and a fraction, where strips have no partner or K is split (M = 20, u4, K = 8192: N = 24640 34.0 us against 35.0, N = 12160
  // 20.7 against 22.0; the codebook's 35.6 against 39.8); with more rows A through LDS is worth the round (M = 32, N = 24640 39.9 against 36.2)
  if (one_strip && NCH * splitk > 256) return lut || (few && !(mx && KC > 32)) || (NCH > 256 && KC <= 16);
  // one chunk for each of eight wavefronts, two for each of four, both in flight (M = 20, K = 1024, N = 16384: u4 5.0 us against 5.5, u8 6.3 against 7.5)
  if ((KC == 7 || KC == 8) && !lut) return NCH <= 256 ? few || bits > 5 || mx : NCH < 384 ? few && bits <= 5 : !codes_float;
  if (NCH >= 384 && KC <= 4) return !lut || bits > 4;      // (M = 20, u4, K = 512, N = 28672: 5.3 us against 5.9)
  if (NCH >= 384 && KC <= 16) return mx || (!lut && !codes_float && bits > 6 && few);      // (M = 20, u8, K = 1408, N = 28672: 11.0 against 12.7)
  return NCH > 224 && NCH <= 256 && few && KC >= 16 && KC <= 32 && !lut && !codes_float && (mx || group != 32);      // (M = 17, u4, K = 4096, N = 16384: 11.9 against 13.0)
}

// Streaming kernel: strips that a workgroup of an arrangement computes.
static int strips_of(int variant) {
  const int e = variant % 10;
  return variant / 10 == 1 ? (e == 6 ? 4 : e == 4 || e == 5 ? 2 : 1) : (e == 6 || e == 7 ? 2 : 1);
}

// Streaming kernel: what a call takes, in microseconds, up to a factor that a weight type has for itself: chunks of K after each
// other in the workgroups of a CU, more for every further round of them, and the exchange -- a trip to memory for every level of the
// tree, with three and four row tiles a slab after the other -- and its traffic.
static double streaming_cost(int M, int N, int K, int bits, int variant, int splitk) {
  const int KC = K / TILE_K, strips = strips_of(variant), mt = variant / 10, cps = (KC + splitk - 1) / splitk;
  const int64_t rounds = ((int64_t)((N / TILE_N + strips - 1) / strips) * splitk + 255) / 256;
  const double chunk = (0.095 + 0.049 * mt) * (1.0 + 0.09 * (bits > 4 ? bits - 4 : 0)) * strips;
  double exchange = 0.0;
  if (splitk > 1) {
    exchange = 2.4e-6 * splitk * (double)M * (double)N;
    if (mt > 2) exchange += 0.3 + 0.6 * (splitk - 1);
    else for (int s = 1; s < splitk; s *= 2) exchange += 1.0;
  }
  return 5.0 + chunk * (double)(rounds * cps) + 2.5 * (double)(rounds - 1) + exchange;
}

// The slabs that doubling came to, or a number that is better by 7 % or more: doubling leaves CUs idle, or a second round with few
// workgroups, where the strips are no power of two, 80 in four slabs for instance (us, M = 16 and 64: K = 13824, N = 5120, u4 15.0 and 29.3, in
// three slabs 11.7 and 20.8; K = 4096, N = 10240 whole instead of in two, M = 64 21.0 and 15.2).
// 1056 calls (22 shapes, M = 1 .. 64, u4, u8, int2, e2m2, e3m2, 4-bit codebook): 180 get other slabs and are 1.04 to 1.57 times as fast, 1.29 on average.
// The int8 kernel by the same estimate (285 calls, 19 shapes, u4, i8, int2, each in 1 to 8 slabs): 0.2 % longer than the best on average, by doubling 19.6 %;
// K = 4096, N = 14336, u4, M = 16 11.0 us in two slabs, whole 8.2; K = 13824, N = 5120 15.1 in four, 10.3 in three.
// A call that needs no workspace keeps doing without.  Looked at are up to four slabs, or as many as doubling came to
// (eight at most: K = 16384, N = 3072, 48 strips, u8, M = 8 15.2 us, in five 13.0; e4m3, M = 16 15.0 and 12.9).
static int better_split(int M, int N, int K, int bits, int variant, int splitk) {
  if (splitk == 1) return 1;
  const int KC = K / TILE_K, NCH = N / TILE_N, mt = variant / 10;
  double least = 0.93 * streaming_cost(M, N, K, bits, variant, splitk);
  int best = splitk;
  for (int sk = 1; sk <= std::max(4, splitk); ++sk) {
    if (sk > 1 && ((KC + sk - 1) / sk < 4 || NCH * sk >= 512 || (size_t)(sk - 1) * NCH * (size_t)(mt * 16 * TILE_N) * sizeof(float) > WS_SLOT_BYTES)) continue;
    const double cost = streaming_cost(M, N, K, bits, variant, sk);
    if (cost < least) { least = cost; best = sk; }
  }
  return best;
}

// Streaming kernel (M <= 64): wavefront arrangement and split-K by shape.  Host arithmetic only.
// (mx: block-scaled weights -- group 32, but only four scale bytes per block and lane, so every
// arrangement has the registers for them)
static void plan_streaming(int M, int N, int K, int group, int wt, int* variant_out, int* splitk_out, int* cps_out,
                           bool mx = false) {
  const int KC = K / TILE_K, NCH = N / TILE_N;
  const int mt = row_tiles(M);
  // 33 .. 48 rows carry three row tiles: a quarter less of A to load and of matrix instructions than four
  // (K = N = 8192, M = 40, u4: 17.8 us against 19.8; K = 4096, N = 28672: 25.4 against 28.2)
  const int tens = (M > 32 && M <= 48) ? 30 : 10 * mt;
  int variant = tens + 1;                     // one strip: 4 wavefronts, with several row tiles 8 (or 4: four_wavefronts)
  // One row tile, short K (at most 32 chunks): as many wavefronts per strip as leaves each
  // two chunks -- 16 (every load of the strip in flight at once) up to 4-bit codes, whose
  // ring fits the 128 registers 16 wavefronts leave each; 8 from 16 chunks on; else 4.
  // With enough strips for pairs of them, two strips per workgroup as for long K below
  // (measured on K = 1024 .. 4096, N = 8192 .. 57344, 3, 4 and 8 bits: within 10 % of the
  // best arrangement everywhere; 16 wavefronts on wide codes or one-chunk shares cost 2-3x).
  if (mt == 1 && KC <= 32) {
    const int bits = wt_bits(wt);
    if (NCH % 2 == 0 && NCH / 2 >= 192) {
      variant = 14;
      if (bits <= 6 && group != 64 && KC >= 16) variant = 15;
      if (variant == 15 && NCH % 4 == 0 && NCH / 4 >= 192) variant = 16;
    } else if (KC >= 32 && bits <= 4 && NCH >= 192) {      // enough strips to occupy most CUs unsplit
      variant = 12;
    } else if (KC >= 16) {
      variant = 10;
    }
  }
  // long K and enough strips to fill the chip with pairs of them: 8 wavefronts on 2
  // adjacent strips, 4 along K each -- wavefronts at the same K position share
  // their A rows in the vector cache (measured 2-4 % shorter at K = 8192, N = 28672;
  // with several row tiles 2 strips x 4 wavefronts along K, 10-15 % shorter, also for short K: K = 4096,
  // N = 28672, M = 24: 20.8 us against 22.4)
  // (several row tiles from 257 strips on: eight wavefronts of theirs fill a CU, and 257 .. 383 strips, one each, would be a
  // round and a fraction: K = 8192, N = 20480, M = 20 35.6 us)
  if ((KC > 32 || mt > 1) && NCH % 2 == 0 && (NCH / 2 >= 192 || (mt > 1 && NCH > 256))) variant = (mt == 1) ? 14 : tens + 6;
  // up to 6 bits per code a wavefront needs few enough registers for 16 of them per
  // workgroup (2 strips x 8 along K): twice the wavefronts in flight, 1-6 % shorter
  if (KC > 32 && variant == 14 && wt_bits(wt) <= 6 && group != 64) variant = 15;
  // and with enough strips for groups of four: 4 strips x 4 along K, half as many, twice as
  // long-lived workgroups (measured 5-9 % shorter at K = 8192, N = 57344, 2 to 6 bits)
  if (KC > 32 && variant == 15 && NCH % 4 == 0 && NCH / 4 >= 192) variant = 16;
  // long K but too few strips to fill the chip (K is split over workgroups below): more
  // wavefronts per strip for narrow codes -- 16 up to 4 bits, 8 up to 6 (measured on
  // K = N = 8192: 11 % and 7 % shorter at 4 bits, no gain at 8)
  if (variant == 11 && KC > 32 && NCH <= 128) variant = wt_bits(wt) <= 4 ? 12 : (wt_bits(wt) <= 6 ? 10 : 11);
  // between 128 and 256 strips a split in two gives more workgroups than CUs: 8-wavefront
  // workgroups, two of which share a CU (K = 8192, N = 14336: 16.3 us against 19.3 with 16
  // wavefronts at 3 bits; 8-bit codes: two strips x 4 wavefronts, 23.5 against 27.3)
  if (variant == 11 && KC > 32 && NCH > 128 && NCH < 256) variant = wt_bits(wt) <= 6 ? 10 : (NCH % 2 == 0 ? 14 : 11);
  if (knob(3) > 0) variant = knob(3);
  if (group == 32 && !mx) variant = tens + 1;   // four groups per chunk: one strip
  const int waves = kDecodeWaves[wt_is_lut(wt) ? 0 : wt](variant);      // the same map for every type
  // Split K over workgroups only when the column strips alone cannot fill the
  // 256 CUs, and never below 4 chunks per wavefront (2 with 16 wavefronts per strip, or with a
  // short K on at most 128 strips: K = 4096, N = 4096 .. 8192 is 15-25 % shorter with 8
  // wavefronts and K in two; half as many with several row tiles: M = 45, K = N = 4096 10.1 us with one
  // chunk per wavefront, 10.5 with two).
  int splitk = knob(1);
  if (splitk <= 0) {
    splitk = 1;
    const bool eight = mt > 1 && (variant % 10 == 1 || variant % 10 == 6);
    const int min_chunks = ((waves >= 16 || (KC <= 32 && NCH <= 128)) ? 2 : 4) / (eight ? 2 : 1);      // per wavefront
    // (several row tiles: 192 workgroups are enough -- K = 4096, N = 14336, M = 24 takes 12.1 us
    // unsplit against 14.7 in two; N = 6144, M = 40: 11.9 in two, 17.2 in four)
    while (NCH * splitk < 256 && !(mt > 1 && NCH * splitk >= 192) && KC / (splitk * 2) >= min_chunks * waves) splitk *= 2;
    // long K and still at most half of the CUs busy: K in four, down to one chunk per wavefront
    // (K = 14336, N = 4096: 11.0 us against 16.2 with K in two; deeper splits lose to the exchange)
    while (KC > 32 && splitk < 4 && NCH * splitk <= 128 && KC / (splitk * 2) >= waves) splitk *= 2;
    // (not 17 .. 24 rows, mostly on four wavefronts, and one row tile of some types on eight: two workgroups to a CU -- e3m2, M = 1, K = 8192,
    // N = 7168 went from 9.8 to 13.5 us --; the two slabs that two row tiles have on long K stay)
    if (!(M > 16 && M <= 24) && variant != 10 && !(mt == 2 && KC > 32 && splitk == 2)) splitk = better_split(M, N, K, wt_bits(wt), variant, splitk);
  }
  if (splitk > KC) splitk = KC;
  const int cps = (KC + splitk - 1) / splitk;
  // (the slabs stay: half as many wavefronts, twice the chunks for each)
  if (mt > 1 && (knob(3) <= 0 || (group == 32 && !mx)) && four_wavefronts(M, NCH, KC, splitk, group, wt, variant == tens + 1, mx))
    variant = variant == tens + 6 && (mt > 2 || NCH >= 384) ? tens + 7 : tens + 2;
  *variant_out = variant;
  *splitk_out = (KC + cps - 1) / cps;
  *cps_out = cps;
}

// Matrix-vector kernel (forced path 5, M <= 4): wavefronts per strip and split-K.  Host arithmetic only.
static void plan_gemv(int M, int N, int K, int group, int wt, int* waves_out, int* splitk_out, int* cps_out) {
  const int KC = K / TILE_K, NCH = N / TILE_N;
  // as many wavefronts per strip as leaves each two chunks: 16 on long K for one row of A, codes of up to 4 bits and one
  // scale group per chunk (beyond that the ring does not fit the 128 registers 16 wavefronts leave each), 8 from 16 chunks on, else 4
  // (measured: 16 pay on short slabs only -- K = 4096, or long K on at most 128 strips, where K is split;
  // K = 8192 on 448 or 896 strips is 6-13 % shorter with 8)
  const bool short_slabs = KC == 32 || (KC > 32 && NCH <= 128);
  int waves = (short_slabs && wt_bits(wt) <= 4 && M == 1 && group >= TILE_K) ? 16 : (KC >= 16 ? 8 : 4);
  if (knob(3) == 4 || knob(3) == 8 || (knob(3) == 16 && M == 1)) waves = knob(3);      // 16 wavefronts: one row only
  int splitk = knob(1);
  if (splitk <= 0) {
    splitk = 1;
    // K over workgroups while the strips alone leave CUs idle and every wavefront keeps two chunks
    while (NCH * splitk < 256 && KC / (splitk * 2) >= 2 * waves) splitk *= 2;
  }
  if (splitk > KC) splitk = KC;
  const int cps = (KC + splitk - 1) / splitk;
  *waves_out = waves; *splitk_out = (KC + cps - 1) / cps; *cps_out = cps;
}

// One launch of the streaming kernel.
static int launch_streaming(GemmParams& p, int wt, int route, int ws_mode, hipStream_t st) {
  int variant;
  plan_streaming(p.M, p.N, p.K, p.group, wt, &variant, &p.splitk, &p.chunks_per_split, p.scale_e8m0 != 0);
  const int mt = row_tiles(p.M);
  if (!covers_rows(variant, p.M)) { g_last_error = "wavefront arrangement does not cover M rows"; return QG_EINVAL; }
  if (p.splitk > 1) {
    const int NCH = p.N / TILE_N;
    size_t pbytes = (size_t)p.splitk * NCH * (size_t)(mt * 16 * TILE_N) * sizeof(float);
    int rc = acquire_ws(ws_mode, pbytes, (size_t)NCH, st, p);
    if (rc == QG_OK) rc = exchange_slots(p.splitk, NCH, mt, p.ws, st, &p.slots);
    if (rc != QG_OK) return rc;
  }
  return wt_is_lut(wt) ? kDecodeLut[wt - WT_LUT0](p, route, variant, st) : kDecode[wt](p, route, variant, st);
}

// Tiled kernel of the first layout: row-tile height (0 = the kernel's own choice: tiles of 256 rows, or of 128 and 64 in one
// launch, or both) and split-K.  Host arithmetic only.
//
// Split-K serves the lower row tiles when they would leave CUs idle.  Candidates: 64- or
// 128-row tiles, K cut into 1 to 8 slabs of an even number of chunks (the kernel
// works in pairs of chunks), at most one workgroup per CU when split.  tiled_cost estimates the
// time in microseconds; the shape of the estimate and the widths' factors are a fit to 2000 measurements at K = 1024 .. 28672,
// N = 2048 .. 28672, M = 24 .. 1000 at 3, 4, 6 and 8 bits, its constants to the exchange as it is now: u4, K = 2048 .. 14336,
// N = 4096 .. 28672, M = 65 .. 768 (70 cases): what it picks takes 0.4 % longer than the best candidate on average and 5 % at most; with
// the constants from before the counters had lines of their own 2.2 % and 15 % (M = 200, K = 5120, N = 13824 44.1 -> 38.3 us,
// M = 300, K = N = 4096 23.3 -> 21.5).  Three slabs that meet in the kernel cost 0.8 us more for every 64 rows of a tile, which its last wavefronts
// read twice: without that they were picked too often on short K, which those cases lack (829 calls of all kinds and widths, K = 512 .. 16384, N = 512 .. 28672,
// M = 65 .. 1000, every candidate timed: 1.05 % longer than the best on average, 1.27 without; M = 112, K = 3072, N = 11008, u4 24.9 us in three
// slabs of 128 rows, 20.4 in two of 64; M = 929, K = 2304, N = 2112 24.4 against 20.4 whole; M = 93, K = 2944, N = 11072, int2, group 32 26.6 against 20.9).
// Codebooks of more than 4 bits are looked up code by code, a chunk takes 1.9 of what u4 takes (98 calls: 0.2 % longer than the best on average, 1.5 with
// the integer type's factor; 8 bits, M = 128, K = 4096, N = 14336 41.3 us in two slabs, 38.6 in four).
// Up to 64 rows (one 64-row tile per column tile) a fit of its own, to K = 4096 .. 28672,
// N = 4096 .. 28672 at 4, 6 and 8 bits: 6 + chunks per workgroup x (1.41 + 0.11 per bit
// above 4; float codes, whose unpack is longer: 1.6 + 0.41 per bit above 4, + 0.4 without a
// hardware convert) + 1.2 per slab.  That fit is older than the kernel's present exchange: the 1.2 is what reading
// the slabs back one pair after the other cost, where up to LARGE_MEET slabs now meet and more have a second kernel.
struct TiledFit { double start, alone64, pair64, alone128, pair128, meet, meet_mb, many, many_mb, third, lookup; };
static constexpr TiledFit TILED_FIT = {3.9, 0.99, 1.66, 1.32, 2.86, 3.6, 0.26, 2.6, 0.42, 0.8, 1.9};
// The first fit.  It settles which calls can do without a workspace (under capture, or without memory): one that it leaves whole
// has always been served there, and is served whole there still if the fit of today splits it.
static constexpr TiledFit TILED_FIT_WHOLE = {4.0, 0.95, 1.65, 1.30, 2.6, 4.0, 0.385, 3.0, 0.335, 0.0, 0.0};

static double tiled_cost(const TiledFit& f, int bm, int sk, int cps, int64_t M, int64_t N, int64_t K, qg_wtype t) {
  const int over = t.bits > 4 ? t.bits - 4 : 0;
  const bool hw_convert = (t.bits == 4 || t.bits == 6 || t.bits == 8);      // e2m1, e3m2, e4m3
  const double unpack = t.kind == QG_CODEBOOK && t.bits > 4 && f.lookup > 0.0 ? f.lookup : t.kind == QG_FLOAT ? (hw_convert ? 1.0 + 0.04 * over : 1.5) : 1.0 + 0.085 * over;
  // a chunk alone on a CU, and with a second workgroup there
  const double alone = unpack * (bm == 64 ? f.alone64 : f.alone128), pair = unpack * (bm == 64 ? f.pair64 : f.pair128);
  const int64_t n = ((M + bm - 1) / bm) * ((N + 255) / 256) * sk, full = n / 512, rest = n % 512;
  const double loop = cps * (full * pair + (rest == 0 ? 0.0 : rest <= 256 ? alone : pair));
  const double read = 0.19e-6 * (double)K * (double)N * t.bits / 8.0;       // the weights from memory
  const double mb = (double)sk * (double)M * (double)N * 4.0e-6;            // partial sums
  const double third = sk == 3 ? f.third * (double)M / (64.0 * (double)((M + bm - 1) / bm)) : 0.0;
  return f.start + std::max(loop, read) + third + (sk == 1 ? 0.0 : sk <= LARGE_MEET ? f.meet + f.meet_mb * mb : f.many + f.many_mb * mb);
}

// The cheapest tile height and split-K under a fit (more than 64 rows whose 128-row tiles leave half of the CUs idle); its cost.
static double best_tiled(const TiledFit& f, int64_t M, int64_t N, int64_t K, qg_wtype t, int* bm_out, int* splitk_out) {
  const int KC = (int)(K / TILE_K);
  const int64_t tiles_n = (N + 255) / 256;
  double best = 1e30;
  for (int bm = 64; bm <= 128; bm *= 2)
    for (int sk = 1; sk <= 8; ++sk) {
      const int64_t tiles_m = (M + bm - 1) / bm;
      int cps = (KC + sk - 1) / sk;
      if (sk > 1 && (cps & 1)) ++cps;
      if (sk > 1 && (cps < 4 || (KC + cps - 1) / cps != sk || tiles_m * tiles_n * sk > 256)) continue;
      const double cost = tiled_cost(f, bm, sk, cps, M, N, K, t);
      if (cost < best) { best = cost; *bm_out = bm; *splitk_out = sk; }
    }
  return best;
}

static void plan_tiled(int64_t M, int64_t N, int64_t K, qg_wtype t, int* bm_out, int* splitk_out, int* cps_out,
                       double* cost_out = nullptr) {
  const int bits = t.bits;
  int bm = knob(2), splitk = knob(1);
  const int KC = (int)(K / TILE_K);
  const int64_t tiles_n = (N + 255) / 256;
  if (bm == 0 && (M <= 64 || large_prefers_64_rows(M, N))) {
    bm = 64;
    if (splitk <= 0 && M <= 64) {
      const int over = bits > 4 ? bits - 4 : 0;
      const bool hw_convert = (bits == 4 || bits == 6 || bits == 8);      // e2m1, e3m2, e4m3
      const double tc = (t.kind == QG_FLOAT) ? 1.6 + 0.41 * over + (hw_convert ? 0.0 : 0.4) : 1.41 + 0.11 * over;
      double best = 1e30;
      for (int sk = 1; sk <= 8; sk *= 2) {
        int cps = (KC + sk - 1) / sk;
        if (sk > 1 && (cps & 1)) ++cps;
        if (sk > 1 && (cps < 8 || tiles_n * sk > 256)) continue;       // short slabs do not pay for the exchange
        const double rounds = (double)((tiles_n * sk + 255) / 256);
        const double cost = 6.0 + rounds * cps * tc + (sk > 1 ? 1.2 * sk : 0.0);
        if (cost < best) { best = cost; splitk = sk; }
      }
      if (cost_out) *cost_out = best;
    } else if (splitk <= 0) {
      const double best = best_tiled(TILED_FIT, M, N, K, t, &bm, &splitk);
      if (cost_out) *cost_out = best;
    }
  }
  if (splitk <= 0 || (bm != 64 && bm != 128)) splitk = 1;
  if (splitk > KC) splitk = KC;
  int cps = (KC + splitk - 1) / splitk;
  if (splitk > 1 && (cps & 1)) ++cps;
  *bm_out = bm;
  *splitk_out = (KC + cps - 1) / cps;
  *cps_out = cps;
}

// No workspace is to be had for a planned split: whether the call is one that runs whole then, and its tile height: those that the
// first fit leaves whole (see TILED_FIT_WHOLE), and codebooks where the integer type of the width is left whole.
static bool tiled_runs_whole(int64_t M, int64_t N, int64_t K, qg_wtype t, int* bm) {
  if (knob(1) > 0 || knob(2) > 0 || M <= 64 || !large_prefers_64_rows(M, N)) return false;
  int splitk = 0;
  (void)best_tiled(TILED_FIT_WHOLE, M, N, K, t, bm, &splitk);
  if (splitk > 1 && t.kind == QG_CODEBOOK) (void)best_tiled(TILED_FIT, M, N, K, qg_wtype{QG_UINT, t.bits, 0, 0}, bm, &splitk);
  return splitk == 1;
}

// The tiled kernels' 32-bit byte offsets: A, the packed weight and the scale array each below 2 GiB.
static bool tiled_operands_fit(int64_t M, int64_t N, int64_t K, int64_t group, int bits) {
  const uint64_t lim = 1ull << 31;
  return (uint64_t)M * (uint64_t)K * 2u < lim && (uint64_t)K * (uint64_t)N / 8u * (uint64_t)bits < lim &&
         (uint64_t)(K / group) * (uint64_t)N * 2u < lim;
}

// path of the first layout: 1 = streaming kernel, 2 = tiled kernel, 3 = streaming kernel
// over blocks of 64 rows (forced only), 4 = de-quantise first (forced, or wide codebooks on many rows)
static int plan_path(int64_t M, int64_t N, int64_t K, int64_t group, qg_wtype t) {
  const int bits = t.bits;
  if (knob(0)) return knob(0);
  // Codebooks of more than 4 bits are looked up code by code (six vector instructions and two LDS
  // reads per pair), which no longer hides between the matrix instructions of the tiled kernel: from
  // about 1024 rows on the paper's prefill variant -- de-quantise once, then the 16-bit matmul -- is
  // faster (6 bits on K = 8192, N = 57344: 1.04 ms against 1.09 at M = 1024, 3.22 against 4.11 at 4096,
  // 9.22 against 12.33 at 12288).  It needs K*N*2 bytes of library-owned buffer below 2 GiB.
  if (t.kind == QG_CODEBOOK && bits > 4 && M >= 1024 && tiled_operands_fit(M, N, K, group, bits) &&
      (uint64_t)K * (uint64_t)N * 2u < (1ull << 31)) return 4;
  if (M > 64) return 2;
  // 33 .. 64 rows: the streaming kernel (4 row tiles per wavefront) re-reads A from L2 for
  // every 64-column strip -- measured 10 us + 2.2 us (+ 0.09 per bit above 4) per 1024 of K
  // at N = 8192 -- while the tiled kernel shares A through LDS among four strips and splits K
  // instead; it wins on all but the small problems (K = 8192, N = 28672, M = 64, 6 bits:
  // 59 us against 75; K = N = 8192: a tie; K = 14336, N = 4096: 32 against 26).  Up to 48 rows the
  // streaming kernel carries three row tiles (0.92 of that).  Both fits are older than the kernels: the streaming estimate is 25.4 us
  // at M = 45, K = N = 8192, u4, where 16.8 are measured.  What they choose (u4, M = 64): K = N = 8192 streaming, 18.4 us against 19.3 tiled in
  // eight slabs; K = 8192, N = 28672 tiled, 43.7 against 50.0.  Between the two the line has not been fitted again.
  if (M > 32 && (double)K * (double)N >= 16.0e6 && knob(1) == 0 &&
      knob(2) == 0 && knob(3) == 0) {
    double tiled = 1e30;
    int bm, sk, cps;
    plan_tiled(M, N, K, t, &bm, &sk, &cps, &tiled);
    const double streaming = (M <= 48 ? 0.92 : 1.0) * (10.0 + (2.2 + 0.09 * (bits > 4 ? bits - 4 : 0)) * ((double)K / 1024.0) * ((double)N / 8192.0));
    if (tiled < 0.9 * streaming) return 2;          // both fits are good to about 10 %
  }
  return 1;
}

}  // namespace qg

using namespace qg;

extern "C" {

const char* qg_status_string(int status) {
  switch (status) {
    case QG_OK: return "ok";
    case QG_EINVAL: return "invalid argument";
    case QG_EUNSUPPORTED: return "valid request with no kernel";
    case QG_EHIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

const char* qg_last_error(void) { return g_last_error.c_str(); }

size_t qg_canonical_bytes(int bits, int64_t count) {
  if (bits < 1 || bits > 8 || count < 0) return 0;
  return (size_t)((count * bits + 7) / 8);
}

size_t qgemm_packed_bytes(qg_wtype t, int layout, int64_t K, int64_t N) {
  if (!pack_layout_ok(layout) || wt_index(t) == -1) return 0;
  if (layout == QG_LAYOUT_TILE128x64_I8 && t.kind == QG_FLOAT) return 0;
  if (t.kind == QG_CODEBOOK && layout != QG_LAYOUT_TILE128x64) return 0;
  if (K <= 0 || N <= 0 || K % TILE_K || N % TILE_N) return 0;
  return (size_t)(K * N * t.bits / 8);
}

int qg_pack_codes(const uint8_t* codes, int bits, int64_t count, uint8_t* stream_out, void* stream) {
  if (bits < 1 || bits > 8 || count < 0) return QG_EINVAL;
  if (count == 0) return QG_OK;
  if (!codes || !stream_out) return QG_EINVAL;
  return launch_pack_codes(codes, bits, count, stream_out, static_cast<hipStream_t>(stream));
}

int repack(const void* canonical, qg_wtype t, int layout, int64_t K, int64_t N, void* packed_out, void* stream) {
  if (!pack_layout_ok(layout)) return QG_EINVAL;
  int wt = wt_index(t);
  if (wt == -1) return QG_EINVAL;   // any float split can be re-laid out; only the type must be well formed
  if (layout == QG_LAYOUT_TILE128x64_I8 && t.kind == QG_FLOAT) return QG_EUNSUPPORTED;   // integer weights only
  if (t.kind == QG_CODEBOOK && layout != QG_LAYOUT_TILE128x64) return QG_EUNSUPPORTED;   // the lookup kernels read the first layout
  if (!canonical || !packed_out || canonical == packed_out) return QG_EINVAL;
  if (K <= 0 || N <= 0 || K % TILE_K || N % TILE_N || K > (1 << 24) || N > (1 << 24)) return QG_EINVAL;
  if (!aligned16(packed_out)) return QG_EINVAL;
  uint32_t flip = (t.kind == QG_INT) ? (1u << (t.bits - 1)) : 0u;
  const int natural = (wt >= 0 && wt_natural(wt) && layout != QG_LAYOUT_TILE128x64_I8) ? 1 : 0;   // types decoded by the hardware converts
  return launch_repack(static_cast<const uint8_t*>(canonical), t.bits, (int)K, (int)N, flip, natural, layout,
                       static_cast<uint8_t*>(packed_out), static_cast<hipStream_t>(stream));
}

static int qdequant_run(const void* packed_W, const void* scales, const uint8_t* zeros, const void* codebook, bool with_codebook,
                        qg_wtype t, int layout, int act, int scale_dtype, int64_t group, int64_t K, int64_t N, void* W_out,
                        void* stream) {
  if (group == 0) group = K;               // 0 = one scale per output column
  int wt, route;
  int rc = check_common(t, layout, act, scale_dtype, group, K, N, &wt, &route, with_codebook);
  if (rc != QG_OK) return rc;
  if (!packed_W || !scales || !W_out || (with_codebook && !codebook)) return QG_EINVAL;
  if (!aligned16(packed_W) || !aligned16(scales) || !aligned16(W_out) || (zeros && !aligned16(zeros)) ||
      (codebook && (reinterpret_cast<uintptr_t>(codebook) & 1u))) return QG_EINVAL;
  DequantParams p;
  p.W = static_cast<const uint8_t*>(packed_W);
  p.S = static_cast<const uint16_t*>(scales);
  p.Z = zeros;
  p.T = static_cast<const uint16_t*>(codebook);
  p.out = static_cast<uint16_t*>(W_out);
  p.layout = layout;
  p.K = (int)K; p.N = (int)N; p.group = (int)group;
  p.zbias = (t.kind == QG_INT) ? (1 << (t.bits - 1)) : 0;
  p.scale_bf16 = (scale_dtype == QG_BF16);
  p.scale_e8m0 = (scale_dtype == QG_E8M0);
  if (p.scale_e8m0 && zeros) return QG_EINVAL;       // block scales come without zero-points
  p.frag_out = 0;
  if (wt_is_lut(wt)) return kDequantLut[wt - WT_LUT0](p, route, static_cast<hipStream_t>(stream));
  return kDequant[wt](p, route, static_cast<hipStream_t>(stream));
}

int qdequant(const void* packed_W, const void* scales, const uint8_t* zeros, qg_wtype t, int layout, int act,
             int scale_dtype, int64_t group, int64_t K, int64_t N, void* W_out, void* stream) {
  return qdequant_run(packed_W, scales, zeros, nullptr, false, t, layout, act, scale_dtype, group, K, N, W_out, stream);
}

int qdequant_codebook(const void* packed_W, const void* codebook, const void* scales, int bits, int act, int scale_dtype,
                      int64_t group, int64_t K, int64_t N, void* W_out, void* stream) {
  const qg_wtype t = {QG_CODEBOOK, bits, 0, 0};
  return qdequant_run(packed_W, scales, nullptr, codebook, true, t, QG_LAYOUT_TILE128x64, act, scale_dtype, group, K, N, W_out, stream);
}

static int qgemm_run(const void* A, const void* packed_W, const void* scales, const uint8_t* zeros, qg_wtype t, int layout,
                     int act, int scale_dtype, int64_t group, int64_t M, int64_t N, int64_t K, void* C, void* stream,
                     int ws_mode, const void* codebook = nullptr, bool with_codebook = false) {
  if (group == 0) group = K;               // 0 = one scale per output column
  int wt, route;
  int rc = check_common(t, layout, act, scale_dtype, group, K, N, &wt, &route, with_codebook);
  if (rc != QG_OK) return rc;
  if (M < 0 || M > (1 << 24)) return QG_EINVAL;
  if (ws_mode == WS_STATIC) {
    // every call with valid shapes, also one with M = 0 or one that will not split K, makes sure
    // the scratch array's address on this device is known: the first such call on a device is the
    // set-up (the runtime loads this library's device code then, if nothing of it has run yet),
    // which a caller that must not allocate later can do once with M = 0
    unsigned char* base = nullptr;
    rc = static_scratch_base(&base);
    if (rc != QG_OK) return rc;
  }
  if (M == 0) return QG_OK;
  if (!A || !packed_W || !scales || !C || (with_codebook && !codebook)) return QG_EINVAL;
  if (!aligned16(A) || !aligned16(packed_W) || !aligned16(scales) || !aligned16(C) || (zeros && !aligned16(zeros)) ||
      (codebook && (reinterpret_cast<uintptr_t>(codebook) & 1u))) return QG_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // one handle value that names a different stream in every thread: the per-stream
  // workspaces (and the stream order the shared scratch relies on) cannot be keyed by it
  if (st == hipStreamPerThread) { g_last_error = "hipStreamPerThread is not accepted: pass a stream of your own"; return QG_EINVAL; }

  GemmParams p;
  p.A = static_cast<const uint16_t*>(A);
  p.W = static_cast<const uint8_t*>(packed_W);
  p.S = static_cast<const uint16_t*>(scales);
  p.Z = zeros;
  p.T = static_cast<const uint16_t*>(codebook);
  p.C = static_cast<uint16_t*>(C);
  p.ws = nullptr; p.tickets = nullptr; p.slots = nullptr;
  p.M = (int)M; p.N = (int)N; p.K = (int)K; p.group = (int)group;
  p.zbias = (t.kind == QG_INT) ? (1 << (t.bits - 1)) : 0;
  p.scale_bf16 = (scale_dtype == QG_BF16);
  p.scale_e8m0 = (scale_dtype == QG_E8M0);
  if (p.scale_e8m0 && zeros) return QG_EINVAL;       // block scales come without zero-points
  p.splitk = 1; p.chunks_per_split = (int)(K / TILE_K);
  if (!set_group_index(p)) return QG_EUNSUPPORTED;

  // The tiled kernels address A, the packed weight and the scales through buffer
  // resources with 32-bit byte offsets, some of them formed in signed arithmetic and A's
  // with the top bit used to push padding rows out of range: each operand stays below 2 GiB.
  const bool fits32 = tiled_operands_fit(M, N, K, group, t.bits);
  if (layout == QG_LAYOUT_TILE128x64_R32) {      // one kernel for every M
    if (!fits32 || group == 32) return QG_EUNSUPPORTED;      // the second layout's kernel has no variant for four groups per chunk
    return kLarge32[wt](p, route, knob(2), st);
  }

  int path = plan_path(M, N, K, group, t);
  if (p.scale_e8m0 && path == 4) return QG_EUNSUPPORTED;      // the de-quantise-first path has no block-scaled variant
  if (path == 1 && M > 64) return QG_EINVAL;
  if (path < 1 || path > 5) return QG_EINVAL;
  if (path == 5) {
    // The decode-sized product as matrix-vector products on the vector ALU (two-element dot
    // products, partial sums added across lanes with permutes): the measured alternative to
    // the matrix-core streaming kernel for M <= 4.  Forced only.
    if (M > 4 || wt_is_lut(wt)) return QG_EINVAL;
    if (p.scale_e8m0) return QG_EUNSUPPORTED;
    int waves;
    plan_gemv(p.M, p.N, p.K, p.group, wt, &waves, &p.splitk, &p.chunks_per_split);
    if (p.splitk > 1) {
      const int NCH = p.N / TILE_N;
      const int mr = M <= 1 ? 1 : 4;
      rc = acquire_ws(ws_mode, (size_t)p.splitk * NCH * (size_t)(mr * TILE_N) * sizeof(float), (size_t)NCH, st, p);
      if (rc != QG_OK) return rc;
    }
    return kGemv[wt](p, route, waves, st);
  }

  void* dense = nullptr;
  if (path == 4) {
    // The paper's prefill variant (Section "End-to-End Performance"): de-quantise the whole
    // weight to 16 bits once, then a plain 16-bit matmul -- here the same tiled kernel reading
    // ready-made operand registers instead of unpacking codes.
    const uint64_t dense_bytes = (uint64_t)K * (uint64_t)N * 2u;
    if (!fits32 || dense_bytes >= (1ull << 31)) return QG_EUNSUPPORTED;
    if (ws_mode == WS_STATIC) { g_last_error = "qgemm_noalloc: the de-quantise-first path needs a K*N*2-byte buffer"; return QG_EUNSUPPORTED; }
    rc = get_dense_buffer((size_t)dense_bytes, st, &dense);
    if (rc != QG_OK && knob(0) == 4) return rc;
    if (rc != QG_OK) path = 2;       // chosen by the library, no memory for the buffer: the fused kernel instead
  }
  if (path == 4) {
    DequantParams d;
    d.W = p.W; d.S = p.S; d.Z = p.Z; d.out = static_cast<uint16_t*>(dense);
    d.layout = QG_LAYOUT_TILE128x64; d.K = p.K; d.N = p.N; d.group = p.group; d.zbias = p.zbias; d.scale_bf16 = p.scale_bf16;
    d.scale_e8m0 = 0;
    d.frag_out = 1;
    d.T = p.T;
    rc = wt_is_lut(wt) ? kDequantLut[wt - WT_LUT0](d, route, st) : kDequant[wt](d, route, st);
    if (rc != QG_OK) return rc;
    GemmParams q = p;
    q.W = static_cast<const uint8_t*>(dense);
    q.Z = nullptr; q.group = p.K; q.zbias = 0;
    if (!set_group_index(q)) return QG_EINVAL;
    qg_wtype t16 = {QG_UINT, 4, 0, 0};               // cost model of the tiled kernel: nothing to unpack, as for a narrow code
    int bm;
    plan_tiled(M, N, K, t16, &bm, &q.splitk, &q.chunks_per_split);
    if (q.splitk > 1) {
      const int64_t tiles = ((M + bm - 1) / bm) * ((N + 255) / 256);
      rc = acquire_ws(ws_mode, (size_t)q.splitk * (size_t)tiles * (size_t)(bm * 256) * sizeof(float), tile_tickets(tiles), st, q);
      if (rc != QG_OK && !tiled_runs_whole(M, N, K, t16, &bm)) return rc;
      if (rc != QG_OK) { q.splitk = 1; q.chunks_per_split = (int)(K / TILE_K); }
    }
    rc = large_launch_wt14(q, route, bm, st);
    return rc == QG_OK && q.splitk > LARGE_MEET ? launch_reduce_tiles(q, route, bm, st) : rc;
  }

  if (path == 1 || path == 3) {
    // a forced arrangement must have the row tiles every block of rows needs, or rows would stay unwritten
    if (knob(3) > 0 && (group != 32 || p.scale_e8m0))
      for (int64_t r0 = 0; r0 < M; r0 += 64)
        if (!covers_rows(knob(3), M - r0 < 64 ? M - r0 : 64)) { g_last_error = "forced wavefront arrangement does not cover the rows of M"; return QG_EINVAL; }
    for (int64_t r0 = 0; r0 < M; r0 += 64) {
      GemmParams q = p;
      q.A = p.A + r0 * K;
      q.C = p.C + r0 * N;
      q.M = (int)((M - r0 < 64) ? (M - r0) : 64);
      rc = launch_streaming(q, wt, route, ws_mode, st);
      if (rc != QG_OK) return rc;
    }
    return QG_OK;
  }
  if (!fits32) return QG_EUNSUPPORTED;
  int bm;
  plan_tiled(M, N, K, t, &bm, &p.splitk, &p.chunks_per_split);
  if (p.splitk > 1) {
    const int64_t tiles = ((M + bm - 1) / bm) * ((N + 255) / 256);
    rc = acquire_ws(ws_mode, (size_t)p.splitk * (size_t)tiles * (size_t)(bm * 256) * sizeof(float), tile_tickets(tiles), st, p);   // a ticket per 64-column strip
    if (rc != QG_OK && !tiled_runs_whole(M, N, K, t, &bm)) return rc;
    if (rc != QG_OK) { p.splitk = 1; p.chunks_per_split = (int)(K / TILE_K); }
  }
  rc = wt_is_lut(wt) ? kLargeLut[wt - WT_LUT0](p, route, bm, st) : kLarge[wt](p, route, bm, st);
  return rc == QG_OK && p.splitk > LARGE_MEET ? launch_reduce_tiles(p, route, bm, st) : rc;
}

int qgemm(const void* A, const void* packed_W, const void* scales, const uint8_t* zeros, qg_wtype t, int layout,
          int act, int scale_dtype, int64_t group, int64_t M, int64_t N, int64_t K, void* C, void* stream) {
  return qgemm_run(A, packed_W, scales, zeros, t, layout, act, scale_dtype, group, M, N, K, C, stream, WS_PER_STREAM);
}

int qgemm_noalloc(const void* A, const void* packed_W, const void* scales, const uint8_t* zeros, qg_wtype t, int layout,
                  int act, int scale_dtype, int64_t group, int64_t M, int64_t N, int64_t K, void* C, void* stream) {
  return qgemm_run(A, packed_W, scales, zeros, t, layout, act, scale_dtype, group, M, N, K, C, stream, WS_STATIC);
}

int qgemm_codebook(const void* A, const void* packed_W, const void* codebook, const void* scales, int bits, int act,
                   int scale_dtype, int64_t group, int64_t M, int64_t N, int64_t K, void* C, void* stream) {
  const qg_wtype t = {QG_CODEBOOK, bits, 0, 0};
  return qgemm_run(A, packed_W, scales, nullptr, t, QG_LAYOUT_TILE128x64, act, scale_dtype, group, M, N, K, C, stream,
                   WS_PER_STREAM, codebook, true);
}

// int8 activations: row tiles of up to 64 rows -- 33 to 48 rows carry three, as in the 16-bit kernel (M = 45, u4: K = N = 8192
// 17.4 -> 15.3 us, N = 28672 46.7 -> 39.0)
static int a8_row_tiles(int64_t M) { return M > 32 && M <= 48 ? 3 : row_tiles(M); }

// int8 activations: wavefronts per strip and split-K of one block of at most 64 rows
static void plan_a8(int M, int N, int K, int bits, int* waves_out, int* splitk_out, int* cps_out) {
  const int KC = K / TILE_K, NCH = N / TILE_N, mt = a8_row_tiles(M);
  // eight wavefronts per strip on long K; four with three or four row tiles (their accumulators and
  // the ring do not fit the registers eight wavefronts leave each) and on short K
  int waves = (KC >= 16 && mt < 3) ? 8 : 4;
  int splitk = knob(1);
  if (splitk <= 0) {
    splitk = 1;
    // K over workgroups while the strips alone leave CUs idle and every wavefront keeps two chunks
    while (NCH * splitk < 256 && KC / (splitk * 2) >= 2 * waves) splitk *= 2;
    splitk = better_split(M, N, K, bits, 10 * mt + 1, splitk);
  }
  if (splitk > KC) splitk = KC;
  const int cps = (KC + splitk - 1) / splitk;
  *waves_out = waves; *splitk_out = (KC + cps - 1) / cps; *cps_out = cps;
}

// Tiled int8 kernel: tile height and split-K of `rows` rows, and the estimated time in microseconds.  Host arithmetic only.
// Workgroups (64 or 128 x 256 tiles times K-slabs) sit two to a CU.  A chunk of K takes a 128-row tile 1.45 us alone
// on a CU and 2.3 with a neighbour, a 64-row tile 1.0 and 1.5 (2 % more per bit above 4, group 64 30 %); a launch 6 us; the
// exchange of partial sums 4 + 0.12 per MB + 1.2 per slab of 64 rows that the last one of a tile reads.  Fitted to M = 65 .. 1000,
// K = 2048 .. 14336, N = 4096 .. 28672, u4, i8, groups 64 and 128 (640 points, 7 % rms) when a launch had tiles of one height; what it
// picked took 3.6 % longer than the best of all heights and splits on average (252 calls with both heights, M = 100 .. 1100: 4 % shorter than
// then on average, none longer).  64-row tiles: M = 300, K = N = 8192, u4 60.6 -> 44.4 us in three slabs, M = 128
// 36.9 -> 29.2, K = N = 4096, M = 200 36.1 -> 23.2; 128-row tiles stay where they fill the chip.
// A chunk of K on the fullest CU.  One launch of both heights (a8_large_kernel): a last row tile of at most 64 rows costs that and no
// more, and 128-row tiles beyond whole rounds of 256 are computed as halves where that is shorter.  us, before and now: K = 8192, N = 28672,
// u4, M = 300 139.4 and 110.2, M = 600 218.2 and 194.1, M = 1000 284.9 and 272.3; u8 in groups of 64, M = 300 190.8 and 132.9, M = 600
// 296.5 and 241.8; K = 4096, N = 14336, u4, M = 600 74.1 and 59.0.  No such tile and no better cut: as before (M = 512 146.7 and 148).
static double a8_round(int64_t high, int64_t low) { return tiles_level(high, low, 1.15, 0.75, low == 0 ? 0.3 : 0.25); }

static double plan_a8_tiled(int64_t rows, int64_t N, int64_t K, int64_t group, int bits, int* bm_out, int* splitk_out, int* cps_out, int* cut_out) {
  const int KC = (int)(K / TILE_K);
  const double f = (group == 64 ? 1.3 : 1.0) * (1.0 + 0.02 * (bits > 4 ? bits - 4 : 0));
  double best = 1e30;
  int splitk = 1, bm = 128, cut = 0;
  for (int cand = 64; cand <= 128; cand *= 2)
    for (int sk : {1, 2, 3, 4, 6, 8}) {
      if ((knob(2) == 64 || knob(2) == 128) && cand != knob(2)) continue;      // (no other height here: chosen as without)
      const int64_t tiles_m = (rows + cand - 1) / cand, tiles = tiles_m * ((N + 255) / 256);
      const int cps = (KC + sk - 1) / sk;
      const size_t part = (size_t)sk * tiles * (cand * 256 * sizeof(float));
      if (sk > 1 && (cps < 4 || tiles * sk > 512 || part > WS_PARTIAL_BYTES)) continue;
      // workgroups of 128 rows and of 64: what is over whole rounds of the former may be cut in halves (not under a forced split).  Split tiles
      // count as 128-row ones all, also a last row tile of 64: its workgroups end early, but the others' last one waits for
      // neither (counted as what they are, K = N = 8192, M = 150 went from 34.3 to 40.4 us, K = 14336, N = 4096, M = 400 from 52.3 to 58.7).
      const int64_t low = cand == 64 ? tiles : sk == 1 && large_last64(rows) ? (N + 255) / 256 : 0, high = tiles - low;
      const int64_t over = cand == 128 && sk == 1 && knob(1) <= 0 ? high % 256 : 0;
      const double whole = a8_round(high * sk, low * sk), mixed = over ? a8_round(high - over, low + 2 * over) : whole;
      const int c = mixed < whole ? (int)over : 0;
      const double loop = f * cps * std::min(whole, mixed);
      const double mb = (double)sk * (double)rows * (double)N * 4.0e-6;
      const double cost = 6.0 + loop + (sk == 1 ? 0.0 : 4.0 + 0.12 * mb + 1.2 * (sk - 1) * (double)rows / (64.0 * tiles_m));
      if (cost < best) { best = cost; splitk = sk; bm = cand; cut = c; }
    }
  if (knob(1) > 0) splitk = std::min(knob(1), 4096);      // (a strip's counter has 16 bits for its slabs)
  if (splitk > KC) splitk = KC;
  const int cps = (KC + splitk - 1) / splitk;
  *cut_out = cut;
  *bm_out = bm;
  *splitk_out = (KC + cps - 1) / cps;
  *cps_out = cps;
  return best;
}

// int8 activations on more than 64 rows: the tiled kernel, or blocks of 64 rows through the streaming kernel?
// The latter take 8 us + 0.16 per million weights (6 % more per bit above 4) each (a last block of up to 16 rows 0.48 of that, of
// up to 32 rows 0.65, 48 0.85), and win while the tiled kernel's chip is nearly empty (an estimate from before the streaming kernel's slabs were chosen by theirs): M = 65 on K = N = 8192 26.9 us against 28.5,
// M = 128 36.7 against 29.1; M = 96 on K = N = 4096 a tie (19.7); M = 1000 on N = 28672 750 against 287.
static bool plan_a8_path(int64_t M, int64_t N, int64_t K, int64_t group, int bits) {
  if (knob(0) == 2 || knob(0) == 3) return knob(0) == 2;
  if (M <= 64) return false;
  if (M > 1024) return true;
  const double block = 8.0 + 0.16e-6 * (1.0 + 0.06 * (bits > 4 ? bits - 4 : 0)) * (double)K * (double)N;
  const int rem = (int)(M % 64);
  const double blocks = block * ((double)(M / 64) + (rem == 0 ? 0.0 : rem <= 16 ? 0.48 : rem <= 32 ? 0.65 : rem <= 48 ? 0.85 : 1.0));
  int bm, sk, cps, cut;
  const double tiled = plan_a8_tiled(M, N, K, group, bits, &bm, &sk, &cps, &cut);
  return tiled < blocks;
}

// The tiled int8 kernel over all rows; `corr`: zero-points, or uintk codes.  K stays whole where it would be split but
// no workspace is to be had.  QG_EUNSUPPORTED, with nothing enqueued: not even 128 rows of A fit its offsets.
static int run_a8_tiled(const A8Params& p, int64_t M, bool corr, int bits, hipStream_t st) {
  const int64_t most = ((int64_t(1) << 31) - 1) / p.K / 128 * 128;      // rows per launch: A's byte offsets stay below 2^31
  if (most < 128) return QG_EUNSUPPORTED;
  for (int64_t r0 = 0; r0 < M; r0 += most) {
    A8Params q = p;
    q.A = p.A + r0 * p.K;
    q.a_scale = p.a_scale ? p.a_scale + r0 : nullptr;
    q.C = p.C + r0 * p.N;
    q.M = (int)std::min(most, M - r0);
    int bm, cut;
    plan_a8_tiled(q.M, q.N, q.K, q.group, bits, &bm, &q.splitk, &q.chunks_per_split, &cut);
    const int64_t tiles = (int64_t)((q.M + bm - 1) / bm) * ((q.N + 255) / 256);
    if (q.splitk > 1 && get_workspace((size_t)q.splitk * tiles * (size_t)(bm * 256) * sizeof(float), tile_tickets(tiles), st, &q.ws, &q.tickets) != QG_OK) {
      q.splitk = 1; q.chunks_per_split = q.K / TILE_K;
    }
    const int rc = kA8Large[bits - 1](q, corr, bm, cut, st);
    if (rc != QG_OK) return rc;
  }
  return QG_OK;
}

int qgemm_a8(const int8_t* A8, const float* a_scale, const void* packed_W, const void* scales, const uint8_t* zeros,
             qg_wtype t, int out_dtype, int scale_dtype, int64_t group, int64_t M, int64_t N, int64_t K, void* C,
             void* stream) {
  if (group == 0) group = K;
  int wt = wt_index(t);
  if (wt == -1) return QG_EINVAL;
  if (t.kind == QG_CODEBOOK) return QG_EINVAL;                    // no table in this call
  if (t.kind == QG_FLOAT) return QG_EUNSUPPORTED;                 // the integer instruction multiplies integers
  if (K <= 0 || N <= 0 || K % TILE_K || N % TILE_N || K > (1 << 24) || N > (1 << 24)) return QG_EINVAL;
  if (group <= 0 || K % group) return QG_EINVAL;
  if (group == 32) return QG_EUNSUPPORTED;                         // the instruction sums 64 values of k
  if (!((group % TILE_K) == 0 || group == 64)) return QG_EINVAL;
  if ((out_dtype != QG_F16 && out_dtype != QG_BF16) || (scale_dtype != QG_F16 && scale_dtype != QG_BF16)) return QG_EINVAL;
  if (M < 0 || M > (1 << 24)) return QG_EINVAL;
  if (M == 0) return QG_OK;
  if (!A8 || !packed_W || !scales || !C) return QG_EINVAL;
  if (!aligned16(A8) || !aligned16(packed_W) || !aligned16(scales) || !aligned16(C) || (zeros && !aligned16(zeros)) ||
      (a_scale && (reinterpret_cast<uintptr_t>(a_scale) & 3u))) return QG_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (st == hipStreamPerThread) { g_last_error = "hipStreamPerThread is not accepted: pass a stream of your own"; return QG_EINVAL; }

  A8Params p;
  p.A = A8; p.a_scale = a_scale;
  p.W = static_cast<const uint8_t*>(packed_W);
  p.S = static_cast<const uint16_t*>(scales);
  p.Z = zeros;
  p.C = static_cast<uint16_t*>(C);
  p.ws = nullptr; p.tickets = nullptr; p.slots = nullptr;
  p.N = (int)N; p.K = (int)K; p.group = (int)group;
  p.zbias = (t.kind == QG_INT) ? (1 << (t.bits - 1)) : 0;
  p.scale_bf16 = (scale_dtype == QG_BF16);
  p.out_bf16 = (out_dtype == QG_BF16);
  p.M = 0;
  if (!set_group_index(p)) return QG_EUNSUPPORTED;
  if (plan_a8_path(M, N, K, group, t.bits)) {
    const int rc = run_a8_tiled(p, M, zeros || t.kind == QG_UINT, t.bits, st);
    if (rc != QG_EUNSUPPORTED) return rc;
  }
  for (int64_t r0 = 0; r0 < M; r0 += 64) {
    A8Params q = p;
    q.A = p.A + r0 * K;
    q.a_scale = a_scale ? a_scale + r0 : nullptr;
    q.C = p.C + r0 * N;
    q.M = (int)((M - r0 < 64) ? (M - r0) : 64);
    int waves;
    plan_a8(q.M, q.N, q.K, t.bits, &waves, &q.splitk, &q.chunks_per_split);
    const int mt = a8_row_tiles(q.M);
    if (q.splitk > 1) {
      const int NCH = q.N / TILE_N;
      float* ws = nullptr; unsigned* tk = nullptr;
      int rc = get_workspace((size_t)q.splitk * NCH * (size_t)(mt * 16 * TILE_N) * sizeof(float), (size_t)NCH, st, &ws, &tk, &q.slots);
      if (rc == QG_OK) rc = exchange_slots(q.splitk, NCH, mt, ws, st, &q.slots);
      if (rc != QG_OK && M > 64 && r0 == 0) return run_a8_tiled(p, M, zeros || t.kind == QG_UINT, t.bits, st);      // no workspace: the tiled kernel does without
      if (rc != QG_OK) return rc;
      q.ws = ws; q.tickets = tk;
    }
    int rc = kA8[t.bits - 1](q, waves, mt, st);
    if (rc != QG_OK) return rc;
  }
  return QG_OK;
}

int qg_probe_stream_read(const void* buf, size_t bytes, void* sink, void* stream) {
  if (!buf || !sink || bytes < 16 || !aligned16(buf)) return QG_EINVAL;
  return launch_probe_stream(buf, bytes, sink, static_cast<hipStream_t>(stream));
}

int qg_probe_mfma(int bf16, int random_data, int iters, int waves_per_simd, void* sink, double* flops_out, void* stream) {
  if (!sink || iters < 1 || waves_per_simd < 1 || waves_per_simd > 8) return QG_EINVAL;
  // 8 instructions of 32*32*16*2 flop per iteration and wavefront, 4 wavefronts per block
  if (flops_out) *flops_out = 8.0 * 32768.0 * (double)iters * 4.0 * 256.0 * waves_per_simd;
  return launch_probe_mfma(bf16 != 0, random_data != 0, iters, waves_per_simd, sink, static_cast<hipStream_t>(stream));
}

int qg_plan(qg_wtype t, int layout, int act, int scale_dtype, int64_t group, int64_t M, int64_t N, int64_t K, int plan[5]) {
  if (group == 0) group = K;               // 0 = one scale per output column
  int wt, route;
  int rc = check_common(t, layout, act, scale_dtype, group, K, N, &wt, &route, t.kind == QG_CODEBOOK);
  if (rc != QG_OK) return rc;
  if (M < 1 || M > (1 << 24) || !plan) return QG_EINVAL;
  plan[0] = plan[1] = plan[2] = 0; plan[3] = 1; plan[4] = (int)(K / TILE_K);
  if (layout == QG_LAYOUT_TILE128x64_R32) {
    plan[0] = 2; plan[2] = knob(2);
    return (group == 32 || !tiled_operands_fit(M, N, K, group, t.bits)) ? QG_EUNSUPPORTED : QG_OK;
  }
  plan[0] = plan_path(M, N, K, group, t);
  if (scale_dtype == QG_E8M0 && plan[0] == 4) return QG_EUNSUPPORTED;   // the de-quantise-first path has no block-scaled variant
  if (plan[0] == 1 && M > 64) return QG_EINVAL;
  if (plan[0] == 1 || plan[0] == 3) {
    plan_streaming((int)(M < 64 ? M : 64), (int)N, (int)K, (int)group, wt, &plan[1], &plan[3], &plan[4], scale_dtype == QG_E8M0);
    if (knob(3) > 0 && (group != 32 || scale_dtype == QG_E8M0))
      for (int64_t r0 = 0; r0 < M; r0 += 64)
        if (!covers_rows(knob(3), M - r0 < 64 ? M - r0 : 64)) return QG_EINVAL;
  } else {
    if (plan[0] < 1 || plan[0] > 5) return QG_EINVAL;
    if (plan[0] == 5) {
      if (M > 4 || wt_is_lut(wt)) return QG_EINVAL;
      if (scale_dtype == QG_E8M0) return QG_EUNSUPPORTED;
      plan_gemv((int)M, (int)N, (int)K, (int)group, wt, &plan[1], &plan[3], &plan[4]);
      return QG_OK;
    }
    if (!tiled_operands_fit(M, N, K, group, t.bits)) return QG_EUNSUPPORTED;
    qg_wtype tt = t;
    if (plan[0] == 4) {
      if ((uint64_t)K * (uint64_t)N * 2u >= (1ull << 31)) return QG_EUNSUPPORTED;
      tt = qg_wtype{QG_UINT, 4, 0, 0};
    }
    plan_tiled(M, N, K, tt, &plan[2], &plan[3], &plan[4]);
  }
  return QG_OK;
}

int qg_set_knob(int knob, int value) {
  if (knob < 0 || knob >= 4) return 0;
  return g_knob[knob].exchange(value, std::memory_order_relaxed);
}

}  // extern "C"
