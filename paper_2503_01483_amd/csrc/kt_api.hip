// kt_api.hip -- host side of libkurtail: argument checks, workspace layout, launch
// sequences, and the extern "C" boundary declared in include/kt.h.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/kt.h"
#include "kt_aux.h"
#include "kt_cayley_d128.h"
#include "kt_fused_d128.h"
#include "kt_hadamard.h"
#include "kt_rows.h"
#include "kt_rowsync.h"
#include "kt_skinny.h"

namespace kt {

// ------------------------------------------------------------------ errors --------
static thread_local char g_err[512] = "";

static kt_status fail(kt_status code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

static bool launch_ok() { return hipGetLastError() == hipSuccess; }

// Kernels that use more than 64 KiB of dynamic LDS need the limit raised once per kernel AND per
// device (the attribute belongs to the device's copy of the code).  Remembers what has been set;
// safe to call from several host threads.
static bool ensure_dynamic_lds(const void* kernel, size_t bytes) {
  struct Entry { const void* kernel; int device; size_t bytes; };
  static std::mutex mu;
  static std::vector<Entry> done;
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return false;
  std::lock_guard<std::mutex> lock(mu);
  Entry* hit = nullptr;
  for (Entry& e : done)
    if (e.kernel == kernel && e.device == device) hit = &e;
  if (hit && hit->bytes >= bytes) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
  if (hit) hit->bytes = bytes;
  else done.push_back({kernel, device, bytes});
  return true;
}

// ------------------------------------------------------------------ static scratch
// Device memory owned by the library image itself, for the one entry point that must not allocate
// (kt_cayley_step_static).  Every GPU the library runs on holds its own copy of the array at its own
// address until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress: the address a kernel can use is looked up once per device, with that device
// current, and kept in g_scratch_ptr; nothing else in this file may pass `scratch` itself anywhere.
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mu;

// Address of this device's copy of the scratch array (null on failure; text in kt_last_error()).
static void* static_scratch_of_current_device() {
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) {
    fail(KT_ERR_DEVICE, "no current HIP device (or device index beyond %d)", kMaxDevices - 1);
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* ptr = nullptr;
    const hipError_t rc = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (rc != hipSuccess || !ptr) {
      fail(KT_ERR_DEVICE, "hipGetSymbolAddress(scratch) failed on device %d: %s", device, hipGetErrorString(rc));
      return nullptr;
    }
    g_scratch_ptr[device] = ptr;
  }
  return g_scratch_ptr[device];
}

// ------------------------------------------------------------------ profiling -----
// Optional event brackets around the large launches (see kt_profile_enable).
// Entry points running on several host threads may take records at the same time: the slot counter is
// atomic (a slot belongs to the scope that drew it); enabling, reading and resetting are not, as the header says.
struct ProfRecord { hipEvent_t start, stop; int id; };
static ProfRecord* g_prof = nullptr;
static int g_prof_cap = 0;
static std::atomic<int> g_prof_used{0};

struct ProfScope {
  ProfRecord* rec = nullptr;
  hipStream_t st;
  ProfScope(int id, hipStream_t s) : st(s) {
    if (g_prof && g_prof_used.load(std::memory_order_relaxed) < g_prof_cap) {
      const int slot = g_prof_used.fetch_add(1, std::memory_order_relaxed);
      if (slot >= g_prof_cap) return;  // another thread drew the last slot meanwhile
      rec = &g_prof[slot];
      rec->id = id;
      (void)hipEventRecord(rec->start, st);
    }
  }
  ~ProfScope() {
    if (rec) (void)hipEventRecord(rec->stop, st);
  }
};

// ------------------------------------------------------------------ tiles ---------
using bf16 = __bf16;
using TB_BIG = Tile<bf16, 256, 256, 2, 2>;
using TB_M128 = Tile<bf16, 128, 256, 1, 4>;  // features on m, d % 256 != 0
using TB_N128 = Tile<bf16, 256, 128, 4, 1>;  // features on n, d % 256 != 0
using TB_128 = Tile<bf16, 128, 128, 2, 2>;   // few tiles
using TB_64 = Tile<bf16, 64, 64, 2, 2>;      // fewer
using TF = Tile<float, 128, 128, 2, 2>;      // fp32 path, every contraction
using TH_BIG = Tile<_Float16, 256, 256, 2, 2>;  // retraction, d >= 1024 (split3_kernel)
using TH_128 = Tile<_Float16, 128, 128, 2, 2>;
using TH_64 = Tile<_Float16, 64, 64, 2, 2>;
using TF_64 = Tile<float, 64, 64, 2, 2>;     // fp32 path, d x d outputs of few tiles

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

constexpr int kNumCUs = 256;

// fp32 products: 64 x 64 tiles when `tiles` 128 x 128 ones would leave CUs idle, in all of the launch or in its last
// round.  A 128 x 128 tile takes a CU about 4100 cycles per 32 of K, a 64 x 64 one a little over a quarter of that, four
// of them share a CU, and the bits are the same (so are the order of K and its splits).
// kt_fuse_rotation, us, large / small tiles: 48 tiles 26 / 14, 256 tiles 143 / 139 (d = 2048), 704 tiles 378 / 354, 1024
// tiles 976 / 989, 3584 tiles 3377 / 3448.
static inline bool use_small_f32(int64_t tiles) {
  return tiles <= kNumCUs || 33 * tiles < 32 * round_up(tiles, kNumCUs);
}
// go(tile) with the tile of an M x N product.  32 x 32 ones (kt_gemm32.h) up to two a CU.  us, 64 x 64 / 32 x 32 tiles: fp32
// fake-quant, d = 1024: 16 tokens 25.4 / 14.7, 200 tokens (224 tiles of 32) 26.1 / 15.1; metrics, 600 tokens (608) 40.7 / 49.1; fp32
// steps, d = 256 (64) 99.3 / 93.0, 512 (256) 188.7 / 172.3, 640 (400) 161.7 / 155.5, bf16 step, d = 768 (576) 215 / 229.
template <class Go>
static auto with_f32_tile(int64_t M, int64_t N, int64_t batch, Go go) {
  if (ceil_div(M, 32) * ceil_div(N, 32) * batch <= 2 * kNumCUs) return go(TF_32{});
  return use_small_f32(ceil_div(M, TF::BM) * ceil_div(N, TF::BN) * batch) ? go(TF_64{}) : go(TF{});
}
static inline bool small_f32_tiles(int64_t d, int64_t batch) { return use_small_f32(ceil_div(d, 128) * ceil_div(d, 128) * batch); }
// Token-minor operands (dL/dY, Y kept for it) are stored in blocks of this many tokens: within a block a
// feature row is contiguous, blocks follow each other feature-row-set by feature-row-set, so
// the 256 rows a tile streams together span 2 MiB per block instead of one page per row.
constexpr int64_t kTokenBlock = 4096;
constexpr int kHadMfmaFrom = 12;  // bf16 Hadamard factors of at least this order run on the matrix cores (measured: the vector kernel wins for 4 and 8)
constexpr int kSensBlocks = 1024;  // workgroups of the sensitivity sweeps
constexpr int kCayleyMaxIters = 32;
// Iterations that are a launch each; those behind them share one launch (cayley_iterate_kernel; `tiles` of it per problem, `edge` wide).
// A launch that finds the iteration converged costs 2 to 3 us.  An iteration inside the kernel costs more than one by itself, by 3 to 10 us
// up to 128 tiles, by up to 40 us at 1000 (each tile drops an L2 that others work from).  A step of usual size takes two or
// three iterations, (lr / 2) ||A|| = 0.1, 0.3, 0.5 takes 5, 11, 25: no more than the first three while 11 iterations are no slower for it than with
// 32 launches of the former kind (d = 768 163 / 348 / 649, 640, 2 problems 151 / 306 / 595, 896, 2 237 / 548 / 1103), a few more above.  us, 3 / 8 / 16 / 32 by themselves:
//   fp32  d = 512 (64 tiles)             3 its 53 / 62 / 77 / 107        11 its 184 / 160 / 153 / 183        25 its 408 / 371 / 332 / 268
//         d = 768 (144)                        95 / 103 / 118 / 147             288 / 268 / 267 / 296              609 / 589 / 556 / 541
//         d = 640, 2 problems (200)            87 / 96 / 110 / 139              277 / 251 / 244 / 273              625 / 600 / 560 / 520
//         d = 256, 16 problems (256)           59 / 68 / 83 / 113               179 / 170 / 169 / 199              361 / 353 / 340 / 333
//         d = 896, 2 problems (392)           162 / 165 / 177 / 207             569 / 485 / 438 / 469             1308 / 1218 / 1076 / 926
//         d = 512, 8 problems (512)           125 / 133 / 147 / 175             394 / 363 / 345 / 377              831 / 803 / 762 / 716
//         d = 896, 4 problems (784)           285 / 277 / 293 / 329            1000 / 846 / 763 / 799             2255 / 2098 / 1862 / 1610
//         d = 256, 64 problems (1024)         148 / 160 / 175 / 210             467 / 430 / 411 / 449              919 / 889 / 838 / 807
//         d = 512, 32 problems (512 of 128 x 128; only the 16 of a problem wait for each other)
//                                             372 / - / 402 / 438              1135 / - / 1115 / 1152             2276 / - / 2295 / 2269
//   fp16  d = 1024 (256)                      129 / 138 / 152 / 182             396 / 361 / 351 / 381              863 / 830 / 777 / 725
//         d = 2048 (256)                      307 / 317 / 332 / 362             958 / 875 / 837 / 865             2008 / 1928 / 1799 / 1676
//         d = 4096 (256)                     1580 / 1586 / 1601 / 1632         4128 / 4041 / 4023 / 4042          9237 / 9153 / 9015 / 8911
static int cayley_own_launches(int64_t tiles, int64_t batch, int edge, bool split) {
  if (!split && edge == TF::BM) return tiles <= 16 ? 3 : kCayleyMaxIters;
  if (tiles * batch < (split && edge > 64 ? kNumCUs / 2 : 200) || (split && edge == 64)) return 3;
  if (split) return 8;
  return tiles * batch <= 400 ? 6 : 16;
}
constexpr float kCayleyTol = 3e-7f;

#ifdef KT_PHASE_STAMPS
static int g_stamp_next = -1;  // developer build: slot the next GEMM launch records its phase stamps in (-1: none)
#endif

// A tile is addressed with 32-bit byte offsets from its first row (K along the rows: the tile's rows) or from the first row of a slab (K as the
// row index: the slab's).  Whether `rows` rows of ld elements can be.
static bool tile_offsets_fit(int64_t rows, int64_t ld, int64_t esz) { return (rows - 1) * ld * esz + 512 <= (int64_t)UINT32_MAX; }

template <class TL, class Epi, bool ATN = false, bool BTN = false, bool TWO = false>
static bool launch_gemm(const void* A, int64_t lda, int64_t bsa, int M, const void* B, int64_t ldb,
                        int64_t bsb, int N, int64_t K, int slabs_per_split, int batch,
                        const Epi& epi, hipStream_t stream, int64_t k_block = 0,
                        int64_t block_stride_b = 0, int k_valid = 0) {
  // ATN: A is [K][lda] with the M index along its rows (see gemm_mainloop); BTN: B [K][ldb].
  constexpr auto kern = [] {
    if constexpr (std::is_same_v<TL, TF_32>) return &gemm32_kernel<Epi, ATN, BTN>;
    else if constexpr (TWO) return &gemm_two_kernel<TL, Epi>;
    else return &gemm_nt_kernel<TL, Epi, ATN, BTN>;
  }();
  constexpr int lds_bytes = (TWO ? 2 : 1) * TL::LDS_BYTES;
  static_assert(!TWO || (!ATN && !BTN && lds_bytes <= 160 * 1024), "two groups: both operands along K");
  const int64_t esz = (int64_t)sizeof(typename TL::T);
  if (!tile_offsets_fit(ATN ? TL::BK : TL::BM, lda, esz) || !tile_offsets_fit(BTN ? TL::BK : TL::BN, ldb, esz)) return false;
  if (ATN && (k_valid < 1 || k_valid > K)) return false;
  if (esz == 4 && ((ATN && M % 4 != 0) || (BTN && N % 4 != 0))) return false;
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes)) return false;
  GemmShape g;
  g.A = A; g.B = B; g.lda = lda; g.ldb = ldb;
  g.batch_stride_a = bsa; g.batch_stride_b = bsb;
  g.M = M; g.N = N;
  g.tiles_m = (int)ceil_div(M, TL::BM);
  g.tiles_n = (int)ceil_div(N, TL::BN);
  g.slabs_total = (int)(K / TL::BK);
  g.slabs_per_split = slabs_per_split > 0 ? slabs_per_split : g.slabs_total;
  g.split_k = (int)ceil_div(g.slabs_total, g.slabs_per_split);  // every split non-empty
  g.tiles_total = g.tiles_m * g.tiles_n * g.split_k;
  g.grid_padded = (int)round_up(g.tiles_total, 8);
  // K blocking of B: rows hold K in blocks of k_block elements, block b of a row starts
  // block_stride_b elements after block b-1 (k_block = 0: ordinary contiguous rows)
  g.slabs_per_block = k_block > 0 ? (int)(k_block / TL::BK) : (g.slabs_total > 0 ? g.slabs_total : 1);
  g.block_bytes_b = block_stride_b * (int64_t)sizeof(typename TL::T);
  g.k_valid = k_valid;
#ifdef KT_PHASE_STAMPS
  g.stamp_slot = g_stamp_next >= 0 && g_stamp_next < kStampSlots ? g_stamp_next++ : -1;
#endif
  if (TWO && (g.split_k != 1 || g.slabs_total % 2 != 0)) return false;
  hipLaunchKernelGGL(kern, dim3(g.grid_padded, batch), dim3((TWO ? 2 : 1) * TL::NT), lds_bytes, stream, g, epi);
  return launch_ok();
}

// A product of a retraction of 22 slabs or more (before that the second prologue and the sum cost what it gives) whose tiles leave a CU to one workgroup
// (128 x 128) or two (64 x 64) takes gemm_two_kernel.  Retractions of two iterations, us, one group of waves / two: d = 1024 79.8 / 72.2, 1152 90.8 / 86.7, 1408
// 112.8 / 103.6, 1664 155.6 / 144.8, 2048 196.6 / 190.1.  Not the rotated rows of few tokens, whose y has to come in the order of a larger call's and of
// one with given scales (kt.h), although fake-quant of 65 tokens of 4096 takes 49.4 us instead of 41.9 for it.
template <class TL, class Epi>
static bool launch_gemm_few(const void* A, int64_t lda, int64_t bsa, int M, const void* B, int64_t ldb, int64_t bsb, int N, int64_t K, int slabs_per_split,
                            int batch, const Epi& epi, hipStream_t stream, int64_t k_block = 0) {
  if constexpr (TL::BM == TL::BN && TL::BM <= 128) {
    const bool few = ceil_div(M, TL::BM) * ceil_div(N, TL::BN) * batch <= (TL::BM == 64 ? 2 : 1) * kNumCUs;
    if (few && K / TL::BK >= 22 && slabs_per_split == 0) return launch_gemm<TL, Epi, false, false, true>(A, lda, bsa, M, B, ldb, bsb, N, K, slabs_per_split, batch, epi, stream, k_block);
  }
  return launch_gemm<TL>(A, lda, bsa, M, B, ldb, bsb, N, K, slabs_per_split, batch, epi, stream, k_block);
}

// Whether a row-major fp32 operand can be read in place, K as its row index (16-byte loads).  Otherwise a launch copies it first.
static bool f32_in_place(const void* p, int64_t ld) {
  return ((reinterpret_cast<uintptr_t>(p) | (uintptr_t)(ld * 4)) & 15) == 0 && tile_offsets_fit(TF::BK, ld, 4);
}

static bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + b_bytes && y < x + a_bytes;
}

// C = R^T X^T with the features on the rows of the GEMM: R is either R^T in the GEMM dtype (in_place false, rows of d) or, fp32,
// the rotation as the caller laid it out.
template <class TL, class Epi>
static bool launch_features_gemm(const typename TL::T* R, int64_t ldr, bool in_place, const typename TL::T* X, int64_t ldx, int64_t batch,
                                 int64_t n, int64_t d, const Epi& e, hipStream_t st) {
  if constexpr (sizeof(typename TL::T) == 4) {
    if (in_place) return launch_gemm<TL, Epi, true>(R, ldr, d * ldr, (int)d, X, ldx, n * ldx, (int)n, d, 0, (int)batch, e, st, 0, 0, (int)d);
  }
  return launch_gemm<TL>(R, d, d * d, (int)d, X, ldx, n * ldx, (int)n, d, 0, (int)batch, e, st);
}

// ---- row_sync_kernel: features on the rows of the GEMM, one launch for all token tiles of all problems.
// The tiles of as many whole row blocks as the chip holds are in flight; a block wider than that cannot wait for itself.
template <class TL>
static bool row_sync_shape(int64_t batch, int64_t n, int64_t d, RowSync* rs) {
  const int64_t fit = kNumCUs * (160 * 1024 / TL::LDS_BYTES), cols = ceil_div(d, TL::BM), rows = ceil_div(n, TL::BN) * batch;
  int64_t at_once = fit / cols;
  if (at_once > rows) at_once = rows;
  if (at_once < 1 || cols > 64 || rows * cols > INT32_MAX / 2) return false;  // (RowSync::order)
  rs->rows = (int)rows;
  rs->cols = (int)cols;
  rs->at_once = (int)at_once;
  rs->per_queue = (int)ceil_div(at_once * cols, 8);
  rs->items = (int)(ceil_div(rows, at_once) * rs->per_queue);
  return true;
}
template <class TL, class Op>
static bool launch_row_sync(RowSync& rs, const typename TL::T* RT, const typename TL::T* X, int64_t ldx, int64_t n, int64_t d, const Op& op,
                            hipStream_t stream) {
  auto kern = &row_sync_kernel<TL, Op>;
  static_assert(kNumCUs * (160 * 1024 / TL::LDS_BYTES) <= kRowSyncMost, "all tiles in flight have an entry");
  rs.arrange();
  if (!tile_offsets_fit(TL::BM, d, (int64_t)sizeof(typename TL::T)) || !tile_offsets_fit(TL::BN, ldx, (int64_t)sizeof(typename TL::T))) return false;
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), TL::LDS_BYTES)) return false;
  GemmShape g = {};
  g.A = RT; g.B = X; g.lda = d; g.ldb = ldx;
  g.batch_stride_a = d * d; g.batch_stride_b = n * ldx;
  g.M = (int)d; g.N = (int)n;
  g.tiles_m = rs.cols;
  g.tiles_n = (int)ceil_div(n, TL::BN);
  g.slabs_total = g.slabs_per_block = (int)(d / TL::BK);
#ifdef KT_PHASE_STAMPS
  g.stamp_slot = -1;
#endif
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * rs.per_queue)), dim3(TL::NT), TL::LDS_BYTES, stream, RowSyncArgs<Op>{g, rs, op});
  return launch_ok();
}

// Iterations it0, ... of `batch` retractions (cayley_iterate_kernel): U and B have rows of ld in the GEMM dtype.  As many workgroups per
// problem as the chip holds, at most one per tile.
template <class TL>
static int64_t cayley_control_words(int64_t d) {
  return kCayleyControlWords + ceil_div(d, TL::BM) * ceil_div(d, TL::BN);
}
template <class TL>
static bool launch_cayley_iterations(const typename TL::T* U0, const typename TL::T* U1, const typename TL::T* B, int64_t K, int64_t d,
                                     int64_t ld, int64_t batch, const EpiCayleyIter<TL>& epi, unsigned* control, int it0, hipStream_t stream) {
  auto kern = &cayley_iterate_kernel<TL, false>;
  if constexpr (TL::BM == 64)
    if (ceil_div(d, TL::BM) * ceil_div(d, TL::BN) * batch >= 200) kern = &cayley_iterate_kernel<TL, true>;
  if (!tile_offsets_fit(TL::BM, ld, (int64_t)sizeof(typename TL::T))) return false;
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), TL::LDS_BYTES)) return false;
  GemmShape g = {};
  g.B = B; g.lda = g.ldb = ld; g.batch_stride_a = g.batch_stride_b = d * ld;
  g.M = g.N = (int)d;
  g.tiles_m = (int)ceil_div(d, TL::BM);
  g.tiles_n = (int)ceil_div(d, TL::BN);
  g.tiles_total = g.tiles_m * g.tiles_n;
  g.slabs_total = (int)(K / TL::BK);
  g.slabs_per_block = (int)(d / TL::BK);
  const int64_t fit = kNumCUs * (160 * 1024 / TL::LDS_BYTES);
  const unsigned wgs = (unsigned)(g.tiles_total < fit ? g.tiles_total : fit);
  hipLaunchKernelGGL(kern, dim3(wgs, (unsigned)batch), dim3(TL::NT), TL::LDS_BYTES, stream, g, epi, U0, U1, control,
                     cayley_control_words<TL>(d), it0);
  return launch_ok();
}

// K slabs per split so that `tiles` output tiles give about `target_wgs` workgroups
// (one per CU for 256 x 256 tiles, several for the small tiles that share a CU), with at
// least 8 slabs of work in each split.
static int choose_slabs_per_split(int64_t tiles, int64_t slabs_total, int64_t target_wgs) {
  int64_t s = ceil_div(target_wgs, tiles);
  const int64_t cap = slabs_total / 8 > 0 ? slabs_total / 8 : 1;
  if (s > cap) s = cap;
  if (s < 1) s = 1;
  return (int)ceil_div(slabs_total, s);
}

// ------------------------------------------------------------------ workspace -----
struct Carver {
  size_t off = 0;
  size_t take(size_t bytes) {
    const size_t o = off;
    off = (size_t)round_up((int64_t)(off + bytes), 256);
    return o;
  }
};

struct LossGradPlan {
  bool fused;      // d = 128 bf16: single-pass kernel, no token-minor copies
  int fused_wgs;   // workgroups per problem on the fused path
  bool fp32;
  size_t esz;
  int64_t ldt;     // padded token count of the token-minor copies (multiple of 128)
  int64_t tb;      // tokens per block of the token-minor copies (row length inside a block)
  int64_t nblk;    // blocks per feature row
  int P;           // moment partials per token
  bool small_fwd, small_dr;  // bf16: 128 x 128 tiles in the forward product, in dR
  int slabs_per_split, split_k;
  size_t o_rt, o_part, o_coef, o_losspart, o_gt, o_splitk, o_gstat, o_yt, total;
  int loss_blocks;
  bool keep_y;     // the forward pass writes Y (fp32, token-minor) and the backward pass reads it instead of recomputing it
};

// Up to this many bytes of kept Y, kt_workspace_bytes(KT_OP_LOSS_GRAD / KT_OP_POOLED_LOSS_GRAD) asks for the
// room to keep it (4 n d bytes per problem); beyond, for the recompute form.
constexpr int64_t kKeepYMaxBytes = (int64_t)64 << 30;

// Workgroups per problem of fused_d128_kernel (a CU holds one at a time): the number that finishes first when they start
// in rounds of 256, a round taking its longest workgroup's tiles and about three more (R^T, the first tile, dR), and every
// partial dR beyond one per problem about a hundredth of a tile (written and read again).
static int fused_d128_wgs(int64_t batch, int64_t n) {
  const int64_t tiles = ceil_div(n, kF128Tile);
  int64_t best = 1;
  double least = -1.0;
  for (int64_t k = 1; k <= tiles && k <= 4 * ceil_div(kNumCUs, batch); ++k) {
    const double cost = (double)(ceil_div(k * batch, kNumCUs) * (ceil_div(tiles, k) + 3)) + (k > 1 ? 0.01 * (double)(k * batch) : 0.0);
    if (least < 0.0 || cost < least) { best = k; least = cost; }
  }
  return (int)best;
}

// ---- tiles of the bf16 loss + gradient pass: 256 x 256, alone on a CU, or 128 x 128, two to a CU.
// Time in units of one slab of K of a 256 x 256 tile (about 1 us).  Such a tile has a prologue and an epilogue of 10 slabs' time
// with nothing beside them (8 without row moments); two 128 x 128 tiles cover each other's, but take 0.7 (dR: 0.8) of the unit for
// half the work, one alone on its CU 0.55.  Loss + gradient, us, 256 / 128: forward d = 512, n = 6000 56.4 / 46.0; 1152, 40000 324 / 301;
// 1408, 20000 219 / 213; 2048, 2000 95 / 73; 2048, 8000 168 / 173; 2688, 20000 567 / 598; 3712, 8000 411 / 437; dR 512, 30000 98 / 86; 1024, 16384
// 124 / 116; 1152, 10007 111 / 102; 1152, 40000 309 / 320; 2432, 5000 164 / 159; 2688, 20000 570 / 624; 3712, 8000 410 / 457.
static double bf16_tile_time(bool small, int64_t tiles, int64_t slabs, double ends, double pair) {
  if (!small) return (double)ceil_div(tiles, kNumCUs) * ((double)slabs + ends);
  const int64_t rest = tiles % (2 * kNumCUs);
  return (pair * (double)(tiles / (2 * kNumCUs)) + (rest == 0 ? 0.0 : rest <= kNumCUs ? 0.55 : pair)) * (double)(slabs + 4);
}
// From four rounds over the chip on two 128 x 128 tiles take 0.76: the workgroups have drifted apart and the row moments (and kept Y) of
// twice the tiles meet the loads of others.  Loss alone, us, 256 / 128: d = 512, 2 problems of 131072 tokens (16 rounds) 160 / 176, 64 of 4096 184 / 204, loss +
// gradient 561 / 585, 712 / 717; 896, 131072 (14) 226 / 210; 1152, 131072 (18), with gradient, 867 / 969.
static bool small_forward_tiles(int64_t batch, int64_t n, int64_t d) {
  const int64_t slabs = d / TB_BIG::BK, tiles = d / 128 * ceil_div(n, 128) * batch;
  return bf16_tile_time(true, tiles, slabs, 0, tiles < 8 * kNumCUs ? 0.7 : 0.76) <
         bf16_tile_time(false, ceil_div(d, 256) * ceil_div(n, 256) * batch, slabs, 10, 0);
}
// dR = X^T G over `slabs` slabs of 64 tokens: tile and slabs per range of tokens, at least eight.  Every range beyond the first
// writes and reads another d x d partial.
static bool small_dr_tiles(int64_t batch, int64_t slabs, int64_t d, int* slabs_per_split) {
  double least = -1.0;
  bool best = false;
  for (const bool small : {false, true}) {
    const int64_t edge = small ? 128 : 256, tiles = ceil_div(d, edge) * ceil_div(d, edge) * batch;
    const int64_t most = ceil_div(small ? 4 * kNumCUs : kNumCUs, tiles);
    for (int64_t s = 1; s <= most && (s == 1 || slabs / s >= 8); ++s) {
      const int64_t per = ceil_div(slabs, s);
      if (ceil_div(slabs, per) != s) continue;
      const double cost = bf16_tile_time(small, tiles * s, per, 8, 0.8) + (s > 1 ? 3.0 + 1.0e-6 * (double)((s + 1) * d * d * batch) : 0.0);
      if (least < 0.0 || cost < least) { least = cost; best = small; *slabs_per_split = (int)per; }
    }
  }
  return best;
}

// ---- rows in one launch (kt_rowsync.h): with which tile, or not at all.
// Time in the unit of bf16_tile_time.  Whole row blocks are in flight, so that the rounds are those of the row blocks; a large tile's ends take 9
// slabs' time, a pair of small ones 0.82 of the unit (0.63 alone on their CUs) with ends of 4, fitted to 168 calls of d = 256 .. 4096, 1 .. 131072
// tokens (off by more than 2 % at three of them).
enum class RowSyncTile { none, small, large };
template <class TL>
static double row_sync_time(const RowSync& rs, int64_t slabs) {
  if (TL::BM == 256) return (double)ceil_div(rs.rows, rs.at_once) * (double)(slabs + 9);
  const int64_t rest = rs.rows % rs.at_once;
  auto round = [&](int64_t r) { return r == 0 ? 0.0 : r * rs.cols <= kNumCUs ? 0.63 : 0.82; };
  return ((double)(rs.rows / rs.at_once) * round(rs.at_once) + round(rest)) * ((double)slabs + 4.0);
}
// Loss + gradient, us, three launches (forward product that keeps Y, row statistics, dL/dY) and their better tile / this: d = 256, 16384 tokens 37.7 / 34.9, 131072
// 136 / 92; 512, 16384 50.7 / 46.0, 131072 279 / 195; 1152, 40000 289 / 262; 2048, 4096 94.6 / 90.8, 16384 285 / 240, 131072 1954 / 1700; 4096, 7000 409 / 392, 131072 6550 / 6070.
//  - wide rows and up to 256 tokens, or a few of any width, where the launches saved cost less than the wait: d = 2688, 100 55.4 / 56.5, 4096, 256 83.0 /
//    84.1; but 2048, 256 46.1 / 45.5; 4096, 700 95.0 / 93.9.  One token: 23.7 / 23.6 (256) to 79.1 / 81.2 (4096)
//  - a second round of large tiles for the last quarter of the row blocks, d > 1408: small ones that drift apart share the CUs better: 1920, 10007 183 / 192,
//    2048, 10007 192 / 202, 2688, 7000 232 / 241; but 1152, 16384 135 / 133, 1408, 10007 (one round) 116 / 104
static RowSyncTile loss_row_sync_tile(int64_t batch, int64_t n, int64_t d) {
  RowSync small, large;
  if (!row_sync_shape<TB_128>(batch, n, d, &small) || !row_sync_shape<TB_BIG>(batch, n, d, &large)) return RowSyncTile::none;
  if (batch * n < 64 || (d > 2048 && batch * n <= 256)) return RowSyncTile::none;
  if (d > 1408 && large.rows > large.at_once && 4 * (int64_t)large.rows <= 5 * (int64_t)large.at_once) return RowSyncTile::none;
  const int64_t slabs = d / TB_BIG::BK;
  return row_sync_time<TB_128>(small, slabs) < row_sync_time<TB_BIG>(large, slabs) ? RowSyncTile::small : RowSyncTile::large;
}
// Fake-quant, us, staged rows and their best tile / this: d = 256, 16384 tokens 23.6 / 18.3, 131072 80 / 52; 512, 10007 26.6 / 21.4, 131072 166 / 111; 1024, 16384
// 52.2 / 45.6, 131072 418 / 291; 1920, 16384 151 / 120; 2048, 131072 1174 / 908; 4096, 4096 129 / 125, 16384 468 / 429, 40000 1153 / 1023.
//  - d <= 640: from about a third of the chip's pairs of small tiles on: 256, 10007 (0.31) 18.2 / 17.6; 512, 4096 (0.25) 16.8 / 18.5; 640, 4096 (0.31) 20.5 / 20.4
//  - wider rows with large tiles only, where they fill 0.7 of one or two rounds (1024, 7000, 0.44: 32.1 / 40.8; 2048, 10007, 0.62: 118 / 125; 1152, 10007, 0.70: 49.0 /
//    46.4), or take no round more than the staged product (3072, 16384, four instead of three: 285 / 296)
static RowSyncTile quant_row_sync_tile(int64_t batch, int64_t n, int64_t d) {
  RowSync small, large;
  if (!row_sync_shape<TB_128>(batch, n, d, &small) || !row_sync_shape<TB_BIG>(batch, n, d, &large)) return RowSyncTile::none;
  const int64_t slabs = d / TB_BIG::BK, rounds = ceil_div(large.rows, large.at_once);
  if (d <= 640) {
    if (100 * (int64_t)small.rows * small.cols < 36 * 2 * kNumCUs) return RowSyncTile::none;
    return row_sync_time<TB_128>(small, slabs) < row_sync_time<TB_BIG>(large, slabs) ? RowSyncTile::small : RowSyncTile::large;
  }
  const bool pays = rounds <= 2 ? 10 * (int64_t)large.rows * (d / 128) >= 7 * 2 * kNumCUs * rounds
                                : rounds > 4 || rounds == ceil_div((int64_t)large.rows * large.cols, kNumCUs);
  return pays ? RowSyncTile::large : RowSyncTile::none;
}

// max_fused_wgs: no more workgroups per problem than this on the d = 128 path (a caller's smaller workspace)
static LossGradPlan plan_loss_grad(int64_t batch, int64_t n, int64_t d, kt_dtype xdt, bool pooled = false,
                                   bool keep_y = false, int64_t max_fused_wgs = INT32_MAX) {
  LossGradPlan p;
  p.keep_y = false;
  p.o_yt = 0;
  p.small_fwd = p.small_dr = false;
  p.fp32 = (xdt == KT_F32);
  p.esz = p.fp32 ? 4 : 2;
  p.fused = !p.fp32 && d == 128 && !pooled;  // the pooled loss needs its global statistics before the gradient
  p.fused_wgs = 0;
  if (p.fused) {
    p.fused_wgs = fused_d128_wgs(batch, n);
    if (p.fused_wgs > max_fused_wgs) p.fused_wgs = (int)max_fused_wgs;
    p.ldt = p.tb = p.nblk = 0;
    p.P = p.slabs_per_split = p.split_k = p.loss_blocks = 0;
    Carver c;
    p.o_rt = 0;
    p.o_losspart = c.take((size_t)batch * p.fused_wgs * 8);
    p.o_splitk = c.take(p.fused_wgs > 1 ? (size_t)p.fused_wgs * batch * d * d * 4 : 0);  // one: straight into dR
    p.o_part = p.o_coef = p.o_gt = p.o_gstat = 0;
    p.total = c.off;
    return p;
  }
  p.ldt = round_up(n, 128);
  p.tb = p.ldt < kTokenBlock ? p.ldt : kTokenBlock;
  p.nblk = ceil_div(p.ldt, p.tb);
  Carver c;
  if (p.fp32) {
    // token ranges as for 128 x 128 tiles (also with smaller ones: a quarter of the ranges would be sums four times as long, in
    // fp32; d = 1024, 16384 tokens: dR off by 8.8e-7 of its norm instead of 6.9e-7).  Whole blocks of 128 tokens where 32 x 32 tiles take
    // them (with_f32_tile on the ranges): four waves share each, so that no sum is longer for it.
    const int64_t slabs = p.ldt / TF::BK;
    p.slabs_per_split = choose_slabs_per_split(ceil_div(d, TF::BM) * ceil_div(d, TF::BN) * batch, slabs, 4 * kNumCUs);
    if (d / 32 * (d / 32) * batch * ceil_div(slabs, p.slabs_per_split) <= 2 * kNumCUs) p.slabs_per_split = (int)round_up(p.slabs_per_split, 4);
    p.split_k = (int)ceil_div(slabs, p.slabs_per_split);
    p.P = 1;
    p.loss_blocks = (int)(p.ldt / 4 < 2048 ? p.ldt / 4 : 2048);  // workgroups of loss_rows_kernel per problem
    p.o_rt = c.take((size_t)batch * d * d * 4);
    p.o_part = c.take(pooled ? (size_t)batch * n * 16 : 0);
    p.o_losspart = c.take((size_t)batch * p.loss_blocks * 8 * (pooled ? 4 : 1));
    p.o_gstat = c.take(pooled ? (size_t)batch * 4 * 8 : 0);
    p.o_gt = c.take((size_t)batch * p.ldt * d * 4);  // Y, then dL/dY
    p.o_splitk = c.take(p.split_k > 1 ? (size_t)p.split_k * batch * d * d * 4 : 0);
    p.o_coef = 0;
    p.total = c.off;
    return p;
  }
  p.P = (int)(d / 128);
  p.small_fwd = small_forward_tiles(batch, n, d);
  p.small_dr = small_dr_tiles(batch, p.ldt / TB_BIG::BK, d, &p.slabs_per_split);
  p.split_k = (int)ceil_div(p.ldt / TB_BIG::BK, p.slabs_per_split);
  p.loss_blocks = (int)ceil_div(n, 256);
  p.o_rt = c.take((size_t)batch * d * d * p.esz);
  p.o_part = c.take((size_t)batch * p.P * n * 16);
  p.o_coef = c.take((size_t)batch * n * 16);
  p.o_losspart = c.take((size_t)batch * p.loss_blocks * 8 * (pooled ? 4 : 1));
  p.o_gstat = c.take(pooled ? (size_t)batch * 4 * 8 : 0);
  p.o_gt = c.take((size_t)batch * d * p.nblk * p.tb * p.esz);
  p.o_splitk = c.take(p.split_k > 1 ? (size_t)p.split_k * batch * d * d * 4 : 0);
  p.keep_y = keep_y;
  p.o_yt = c.take(keep_y ? (size_t)batch * d * p.nblk * p.tb * 4 : 0);
  p.total = c.off;
  return p;
}

// The plan kt_workspace_bytes recommends: Y kept when it is small enough and the path has a backward GEMM to save.
static bool keep_y_recommended(int64_t batch, int64_t n, int64_t d, kt_dtype xdt, bool pooled) {
  if (xdt == KT_BF16 && d == 128 && !pooled) return false;  // single-pass kernel
  return batch * round_up(n, 128) * d * 4 <= kKeepYMaxBytes;
}

struct CayleyPlan {
  bool split;  // three-term fp16 products instead of fp32 ones
  size_t o_m, o_b, o_rt, o_zt, o_u0, o_u1, o_delta, o_g2, o_sq, o_scal, total;
  int g2_blocks;  // Cayley Adam: block partials of ||G||^2 per problem
};

// From d = 1024 on the d^3 products run as three-term fp16 ones (22 bits of every value, 3x the flops at 16x the rate of the fp32
// matrix pipe); below, the two launches more and the tripled operands cost more than that gives (steps, us, fp32 / split: d = 640 86 /
// 100, 896 109 / 120).  Steps of 256 tokens, us, d % 256 != 0 fp32 before / this: d = 1152 274 / 159, 2432 885 / 485, 3712 2706 / 1174.
// Errors against 64 bits over d = 1024 .. 2432, (lr / 2) ||A|| = 0.003 .. 0.4, full and rank-two gradients, R Haar and near the identity: new R
// never further off than with fp32 or three-term bf16 products, Cayley Adam's momentum 6.5e-7 .. 1.0e-6 (fp32 8.6e-7 .. 1.25e-6, bf16 5e-6).
// The fp32 form also serves d % 256 != 0 with a workspace that has no room for the split operands.
static bool cayley_use_split(int64_t d) { return d >= 1024; }
// go(tile): 64 x 64 while 128 x 128 ones leave half the CUs without, else the faster of the two large ones (bf16_tile_time).  Same
// steps, us, 64 / 128 / 256: d = 1024 141 / 164 / 319, 1408 239 / 256 / 491, 1664 249 / 239 / 441, 2048 384 / 303 / 510, 2432 584 / 484 / 600, 3072
// 1079 / 888 / 828, 3712 1964 / 1419 / 1178.
template <class Go>
static auto with_f16_tile(int64_t d, int64_t batch, Go go) {
  const int64_t t128 = d / 128 * (d / 128) * batch, t256 = ceil_div(d, 256) * ceil_div(d, 256) * batch, slabs = 3 * d / TH_BIG::BK;
  if (t128 <= kNumCUs / 2) return go(TH_64{});
  return bf16_tile_time(true, t128, slabs, 0, 0.75) < bf16_tile_time(false, t256, slabs, 10, 0) ? go(TH_128{}) : go(TH_BIG{});
}

// The tile of cayley_iterate_kernel: the same, but 128 x 128 instead of more 64 x 64 ones than there are CUs (what an iteration costs there
// beyond a launch of its own grows with the tiles).  us, 24 iterations, all but three inside, 64 / 128: d = 1024 (256 tiles of 64) 869 / 933, 1152
// (324) 1224 / 1062, 1408 (484) 1774 / 1171, 1024, 2 problems (512) 1530 / 1085.  256 instead of 128: 2048 2008 / 3360, 2432 4257 / 4334.
template <class Go>
static auto with_f16_iterate_tile(int64_t d, int64_t batch, Go go) {
  return with_f16_tile(d, batch, [&](auto t) {
    if constexpr (std::is_same_v<decltype(t), TH_64>)
      if (d / 64 * (d / 64) * batch > kNumCUs) return go(TH_128{});
    return go(t);
  });
}

static CayleyPlan plan_cayley(int64_t batch, int64_t d, bool split) {
  CayleyPlan p;
  Carver c;
  p.split = split;
  const size_t mat = (size_t)batch * d * d * 4;
  const size_t smat = (size_t)batch * d * d * 6;  // [d][2d] fp16 (and room that earlier forms needed: sizes stay as they were)
  p.o_m = c.take(mat);  // M = dR R^T; in the fp32 path later reused as the second U buffer
  p.o_b = c.take(p.split ? smat : mat);
  p.o_rt = c.take(mat);
  p.o_zt = c.take(mat);
  p.o_u0 = c.take(p.split ? smat : mat);
  p.o_u1 = p.split ? c.take(smat) : p.o_m;
  p.o_delta = c.take((size_t)batch * kCayleyMaxIters * 4);
  // Cayley Adam scalars: partial sums (fp64) and {r, alpha, ||W||, alpha/(2r)} per problem
  p.g2_blocks = (int)(ceil_div(d * d / 4, 256) < 1024 ? ceil_div(d * d / 4, 256) : 1024);
  p.o_g2 = c.take((size_t)batch * p.g2_blocks * 8);  // (then the control words of the iterations, which are fewer)
  p.o_sq = c.take((size_t)batch * (d / 32) * (d / 32) * 8);
  p.o_scal = c.take((size_t)batch * 4 * 4);
  p.total = c.off;
  return p;
}

// The plan for a workspace of `bytes`.
static CayleyPlan plan_cayley_in(int64_t batch, int64_t d, size_t bytes) {
  const CayleyPlan p = plan_cayley(batch, d, cayley_use_split(d));
  return p.split && d % 256 != 0 && bytes < p.total ? plan_cayley(batch, d, false) : p;
}

struct QuantPlan {
  bool fp32;
  size_t esz;
  int P, PN;
  // Scales computed here AND codes or errors wanted: Y goes through an fp32 staging buffer of at most
  // kQuantStageBytes, `problems` whole problems or `rows` tokens of one problem per launch pair.
  int64_t stage_problems, stage_rows;
  size_t o_rt, o_amax, o_scales, o_errpart, o_y, total;
};

// d = 4096, n = 131072: fake-quant measured alike from 64 MiB to 4 GiB; the quantisation figures, whose row
// kernel is one workgroup per token, lose 7 % at 256 MiB and nothing at 1 GiB
constexpr int64_t kQuantStageBytes = (int64_t)1 << 30;

// How many whole problems, or how many token rows of one problem, an fp32 staging buffer of at most
// kQuantStageBytes takes per launch pair (rotation GEMM + row kernel).
static void stage_slices(int64_t batch, int64_t n, int64_t d, int64_t* problems, int64_t* rows) {
  const int64_t cap = kQuantStageBytes / (4 * d) / 256 * 256;  // >= 16384 token rows at d <= 16384
  *rows = n < cap ? n : cap;
  *problems = n <= cap ? (cap / n < batch ? cap / n : batch) : 1;
}

static QuantPlan plan_quant(int64_t batch, int64_t n, int64_t d, kt_dtype xdt) {
  QuantPlan p;
  p.fp32 = (xdt == KT_F32);
  p.esz = p.fp32 ? 4 : 2;
  if (p.fp32) {
    p.P = (int)ceil_div(d, TF::BM) * TF::WGM;
    p.PN = (int)ceil_div(d, TF::BN) * TF::WGN;
  } else if (d % 256 == 0) {
    p.P = (int)(d / 256) * TB_BIG::WGM;
    p.PN = (int)(d / 256) * TB_BIG::WGN;
  } else {
    p.P = (int)ceil_div(d, TB_M128::BM) * TB_M128::WGM;
    p.PN = (int)ceil_div(d, TB_N128::BN) * TB_N128::WGN;
  }
  Carver c;
  p.o_rt = c.take((size_t)batch * d * d * p.esz);
  p.o_amax = c.take((size_t)batch * p.P * n * 4);
  p.o_scales = c.take((size_t)batch * n * 4);
  p.o_errpart = c.take((size_t)batch * p.P * n * 8);
  stage_slices(batch, n, d, &p.stage_problems, &p.stage_rows);
  p.o_y = c.take((size_t)p.stage_problems * p.stage_rows * d * 4);
  p.total = c.off;
  return p;
}

// ------------------------------------------------------------------ checks --------
static kt_status check_xr(const void* X, int64_t ldx, const void* R, int64_t ldr, int64_t batch,
                          int64_t n, int64_t d, kt_dtype xdt, kt_dtype rdt) {
  if (!X || !R) return fail(KT_ERR_INVALID_ARG, "X and R must not be null");
  if (batch < 1 || n < 1 || d < 1) return fail(KT_ERR_INVALID_ARG, "batch, n, d must be positive");
  if (xdt != KT_F32 && xdt != KT_BF16) return fail(KT_ERR_BAD_DTYPE, "x_dtype must be KT_F32 or KT_BF16");
  if (rdt != KT_F32 && rdt != KT_BF16) return fail(KT_ERR_BAD_DTYPE, "r_dtype must be KT_F32 or KT_BF16");
  if (xdt == KT_F32 && rdt != KT_F32)
    return fail(KT_ERR_BAD_DTYPE, "the fp32 path needs an fp32 R");
  if (d % 128 != 0) return fail(KT_ERR_BAD_SHAPE, "d = %lld is not a multiple of 128", (long long)d);
  // n is bounded so that 255 rows of a token-minor operand stay inside 32-bit byte offsets
  if (d > 16384 || n > (int64_t)1 << 22 || batch > 65535)
    return fail(KT_ERR_BAD_SHAPE, "size out of range (d <= 16384, n <= 2^22, batch <= 65535)");
  const int64_t align = xdt == KT_F32 ? 4 : 8;
  if (ldx < d || ldx % align != 0)
    return fail(KT_ERR_BAD_SHAPE, "ldx = %lld must be >= d and a multiple of %lld", (long long)ldx,
                (long long)align);
  if (ldr < d) return fail(KT_ERR_BAD_SHAPE, "ldr = %lld must be >= d", (long long)ldr);
  // 255 rows of X must stay inside 32-bit byte offsets (tiles are addressed from their first row)
  if (ldx > (int64_t)1 << 22 || ldr > (int64_t)1 << 22)
    return fail(KT_ERR_BAD_SHAPE, "ldx and ldr must not exceed 2^22 elements");
  if ((reinterpret_cast<uintptr_t>(X) & 15) != 0)
    return fail(KT_ERR_BAD_SHAPE, "X must be 16-byte aligned");
  return KT_OK;
}

static kt_status check_ws(void* ws, size_t have, size_t need) {
  if (!ws) return fail(KT_ERR_INVALID_ARG, "workspace must not be null");
  if ((reinterpret_cast<uintptr_t>(ws) & 255) != 0)
    return fail(KT_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
  if (have < need)
    return fail(KT_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", have, need);
  return KT_OK;
}

// R (fp32 or bf16, row-major) -> R^T in the GEMM dtype; `zero_words` words at `zero` are cleared on the way.
template <typename Tout>
static bool prep_rt(const void* R, int64_t ldr, kt_dtype rdt, Tout* RT, int64_t batch, int64_t d,
                    hipStream_t st, unsigned* zero = nullptr, int64_t zero_words = 0) {
  const dim3 grid((unsigned)(d / 64), (unsigned)(d / 64), (unsigned)batch);
  if (rdt == KT_F32)
    hipLaunchKernelGGL((transpose_kernel<float, Tout>), grid, dim3(256), 0, st, static_cast<const float*>(R), ldr, RT, (int)d, zero, (int)zero_words);
  else
    hipLaunchKernelGGL((transpose_kernel<bf16, Tout>), grid, dim3(256), 0, st, static_cast<const bf16*>(R), ldr, RT, (int)d, zero, (int)zero_words);
  return launch_ok();
}

// out = sum of the `splits` partials; with `loss` (batch > 0) also the loss sums.
static bool launch_splitk_reduce(const float* part, int64_t count, int splits, float* out, const LossSum& loss, hipStream_t st) {
  const int64_t wgs = ceil_div(count, 1024) < 2048 ? ceil_div(count, 1024) : 2048;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)(wgs + loss.problems)), dim3(256), 0, st, part, count, splits, out, count, loss);
  return launch_ok();
}
static bool launch_loss_sum(const LossSum& loss, hipStream_t st) {
  hipLaunchKernelGGL(finalize_loss_kernel, dim3((unsigned)loss.problems), dim3(256), 0, st, loss);
  return launch_ok();
}

// ------------------------------------------------------------------ loss + grad ---
struct PooledArgs {  // paper-literal pooled loss (kurtosis over all entries after an RMSNorm)
  float rms_eps;
  float* kappa_out;  // [batch] or null
};

// bf16, d > 128 or pooled.
static kt_status run_loss_grad_bf16(const LossGradPlan& p, const void* X, int64_t ldx, const void* R,
                               int64_t ldr, kt_dtype rdt, int64_t batch, int64_t n, int64_t d,
                               float kappa_target, float* loss, float* row_kurt, float* dR,
                               char* ws, hipStream_t st, const PooledArgs* pooled = nullptr) {
  using T = bf16;
  T* RT = reinterpret_cast<T*>(ws + p.o_rt);
  floatx4* part = reinterpret_cast<floatx4*>(ws + p.o_part);
  floatx4* coef = reinterpret_cast<floatx4*>(ws + p.o_coef);
  double* loss_part = reinterpret_cast<double*>(ws + p.o_losspart);
  T* GT = reinterpret_cast<T*>(ws + p.o_gt);
  float* splitk = reinterpret_cast<float*>(ws + p.o_splitk);
  const T* Xp = static_cast<const T*>(X);

  // a1 - a3 in one launch where a row's statistics are all the gradient needs.  Its words are in the room of the row coefficients,
  // which then stay in the LDS: 8 bytes of loss and a counter per row block and nine counters, 16 bytes per token (packed, they fit in 256 a problem).
  RowSync rs;
  const RowSyncTile rs_tile = dR && !pooled ? loss_row_sync_tile(batch, n, d) : RowSyncTile::none;
  const bool row_sync = rs_tile != RowSyncTile::none;
  if (row_sync) {
    (void)(rs_tile == RowSyncTile::small ? row_sync_shape<TB_128>(batch, n, d, &rs) : row_sync_shape<TB_BIG>(batch, n, d, &rs));
    loss_part = reinterpret_cast<double*>(coef);
    rs.words = reinterpret_cast<unsigned*>(loss_part + rs.rows);
    rs.pitch = (size_t)rs.rows * 8 + (size_t)(kRowSyncWords + rs.rows) * kRowSyncPitch * 4 <= p.o_losspart - p.o_coef ? kRowSyncPitch : 1;
  }
  const LossSum loss_sum = {loss_part, row_sync ? (int)(rs.rows / batch) : p.loss_blocks, (int)n, (int)batch, loss};

  // a0: R -> R^T in the GEMM dtype
  if (!prep_rt<T>(R, ldr, rdt, RT, batch, d, st, row_sync ? rs.words : nullptr, row_sync ? (int64_t)(kRowSyncWords + rs.rows) * rs.pitch : 0))
    return fail(KT_ERR_DEVICE, "prep_rt launch failed");

  // go(tile) with the tile of the forward product (features on m, tokens on n)
  auto with_forward_tile = [&](auto go) -> bool {
    return p.small_fwd ? go(TB_128{}) : go(TB_BIG{});
  };

  if (row_sync) {
    ProfScope prof(0, st);
    auto go = [&](auto tile_tag) -> bool {
      using TL = decltype(tile_tag);
      RowLossGrad<TL> op;
      op.mom.part = part; op.mom.n_tokens = (int)n; op.mom.d = (int)d; op.mom.P = rs.cols;
      op.grad.coef = nullptr; op.grad.GT = GT; op.grad.ldt = p.ldt; op.grad.tb = p.tb; op.grad.batch_stride = d * p.nblk * p.tb;
      op.grad.n_tokens = (int)n; op.grad.d = (int)d;
      op.kappa_target = kappa_target; op.row_kurt = row_kurt; op.loss_part = loss_part; op.tiles_n = (int)(rs.rows / batch);
      return launch_row_sync<TL>(rs, RT, Xp, ldx, n, d, op, st);
    };
    if (!(rs_tile == RowSyncTile::small ? go(TB_128{}) : go(TB_BIG{}))) return fail(KT_ERR_DEVICE, "forward GEMM launch failed");
    if (p.split_k == 1 && !launch_loss_sum(loss_sum, st)) return fail(KT_ERR_DEVICE, "loss sum launch failed");
  } else {
  // a1: forward GEMM with the moment epilogue; with keep_y it also writes Y
  const bool keep = p.keep_y && dR;
  float* YT = reinterpret_cast<float*>(ws + p.o_yt);
  {
    ProfScope prof(0, st);
    const bool ok = with_forward_tile([&](auto tile_tag) -> bool {
      using TL = decltype(tile_tag);
      EpiMoments<TL> e;
      e.part = part; e.n_tokens = (int)n; e.d = (int)d; e.P = p.P;
      if (!keep) return launch_gemm<TL>(RT, d, d * d, (int)d, Xp, ldx, n * ldx, (int)n, d, 0, (int)batch, e, st);
      EpiMomentsKeep<TL> ek;
      ek.mom = e; ek.YT = YT; ek.ldt = p.ldt; ek.tb = p.tb; ek.batch_stride = d * p.nblk * p.tb;
      return launch_gemm<TL>(RT, d, d * d, (int)d, Xp, ldx, n * ldx, (int)n, d, 0, (int)batch, ek, st);
    });
    if (!ok) return fail(KT_ERR_DEVICE, "forward GEMM launch failed");
  }
  if (pooled) {
    // a2, pooled form: pooled sums -> global statistics and loss -> per-token coefficients
    double* gstat = reinterpret_cast<double*>(ws + p.o_gstat);
    hipLaunchKernelGGL(pooled_stage1_kernel, dim3(p.loss_blocks, (unsigned)batch), dim3(256), 0, st, part, p.P,
                       (int)n, (int)d, pooled->rms_eps, loss_part);
    hipLaunchKernelGGL(pooled_stage2_kernel, dim3((unsigned)batch), dim3(256), 0, st, loss_part, p.loss_blocks,
                       (int)n, (int)d, kappa_target, gstat, loss, pooled->kappa_out);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "pooled statistics launch failed");
    if (!dR) return KT_OK;
    hipLaunchKernelGGL(pooled_stage3_kernel, dim3(p.loss_blocks, (unsigned)batch), dim3(256), 0, st, part, p.P,
                       (int)n, (int)d, pooled->rms_eps, gstat, coef);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "pooled coefficient launch failed");
  } else {
  // a2: per-token finalisation and loss
  hipLaunchKernelGGL(finalize_rows_kernel, dim3(p.loss_blocks, (unsigned)batch), dim3(256), 0, st, part,
                     p.P, (int)n, (int)d, kappa_target, coef, row_kurt, loss_part);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "finalize_rows launch failed");
  if ((!dR || p.split_k == 1) && !launch_loss_sum(loss_sum, st)) return fail(KT_ERR_DEVICE, "loss sum launch failed");
  if (!dR) return KT_OK;
  }

  // a3: dL/dY token-minor, from the kept Y entry by entry or from a recomputed Y in the GEMM epilogue
  if (keep) {
    ProfScope prof(1, st);
    constexpr int kFeats = 8;
    dim3 grid((unsigned)ceil_div(p.ldt, 256), (unsigned)ceil_div(d, 4 * kFeats), (unsigned)batch);
    hipLaunchKernelGGL((grad_from_y_kernel<T, kFeats>), grid, dim3(256), 0, st, YT, coef, GT, p.ldt, p.tb,
                       d * p.nblk * p.tb, (int)n, (int)d);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "gradient kernel launch failed");
  } else {
    ProfScope prof(1, st);
    const bool ok = with_forward_tile([&](auto tile_tag) -> bool {
      using TL = decltype(tile_tag);
      EpiGrad<TL> e;
      e.coef = coef; e.GT = GT; e.ldt = p.ldt; e.tb = p.tb; e.batch_stride = d * p.nblk * p.tb;
      e.n_tokens = (int)n; e.d = (int)d;
      return launch_gemm<TL>(RT, d, d * d, (int)d, Xp, ldx, n * ldx, (int)n, d, 0, (int)batch, e, st);
    });
    if (!ok)
      return fail(KT_ERR_DEVICE, "backward recompute GEMM launch failed");
  }
  }
  // a4: dR = X^T G, split over tokens
  {
    ProfScope prof(2, st);
    auto go = [&](auto tile_tag) -> bool {
      using TL = decltype(tile_tag);
      EpiStore<TL> e;
      e.C = p.split_k > 1 ? splitk : dR;
      e.batch_stride = d * d; e.split_stride = p.split_k > 1 ? batch * d * d : 0;
      e.ldc = d; e.M = (int)d; e.N = (int)d;
      return launch_gemm<TL, EpiStore<TL>, true>(Xp, ldx, n * ldx, (int)d, GT, p.tb, d * p.nblk * p.tb, (int)d, p.ldt,
                                                 p.slabs_per_split, (int)batch, e, st, p.tb, d * p.tb, (int)n);
    };
    if (!(p.small_dr ? go(TB_128{}) : go(TB_BIG{}))) return fail(KT_ERR_DEVICE, "gradient GEMM launch failed");
    if (p.split_k > 1 && !launch_splitk_reduce(splitk, batch * d * d, p.split_k, dR, pooled ? LossSum{} : loss_sum, st))
      return fail(KT_ERR_DEVICE, "split-K reduce launch failed");
  }
  return KT_OK;
}

// d = 128, bf16: one pass over X (kt_fused_d128.h), then fixed-order reductions.
static kt_status run_loss_grad_fused(const LossGradPlan& p, const void* X, int64_t ldx, const void* R,
                                     int64_t ldr, kt_dtype rdt, int64_t batch, int64_t n, int64_t d,
                                     float kappa_target, float* loss, float* row_kurt, float* dR,
                                     char* ws, hipStream_t st) {
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(fused_d128_kernel), kF128LdsBytes))
    return fail(KT_ERR_DEVICE, "the fused d=128 kernel needs %d bytes of LDS per workgroup", kF128LdsBytes);
  double* loss_part = reinterpret_cast<double*>(ws + p.o_losspart);
  float* dR_part = p.fused_wgs > 1 ? reinterpret_cast<float*>(ws + p.o_splitk) : dR;
  {
    ProfScope prof(0, st);
    hipLaunchKernelGGL(fused_d128_kernel, dim3(p.fused_wgs, (unsigned)batch), dim3(512), kF128LdsBytes, st,
                       static_cast<const bf16*>(X), ldx, n * ldx, R, ldr, rdt == KT_BF16 ? 1 : 0, (int)n, kappa_target, row_kurt,
                       loss_part, dR_part, dR ? 1 : 0);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "fused kernel launch failed");
  }
  const LossSum loss_sum = {loss_part, p.fused_wgs, (int)n, (int)batch, loss};
  if (dR && p.fused_wgs > 1) {
    if (!launch_splitk_reduce(dR_part, batch * d * d, p.fused_wgs, dR, loss_sum, st)) return fail(KT_ERR_DEVICE, "partial dR reduce launch failed");
  } else if (!launch_loss_sum(loss_sum, st)) {
    return fail(KT_ERR_DEVICE, "loss sum launch failed");
  }
  return KT_OK;
}

// ------------------------------------------------------------------ rotated rows ----
// A few tokens (kt_skinny.h): Y = X R straight from R, partial sums of the row ranges in `scratch` (rt_bytes, the room
// of the transposed copy of R that this path does not make).  R as the caller laid it out, so 16-byte reads of it
// have to be possible.
static bool skinny_ok(kt_dtype xdt, const void* R, int64_t ldr, kt_dtype rdt, int64_t n) {
  return xdt == KT_BF16 && n <= kSkinnyMaxTokens && (reinterpret_cast<uintptr_t>(R) & 15) == 0 && ldr % (rdt == KT_F32 ? 4 : 8) == 0;
}

template <typename TR>
static bool launch_skinny(const bf16* X, int64_t ldx, const TR* R, int64_t ldr, int64_t batch, int64_t n, int64_t d,
                          char* scratch, size_t rt_bytes, float* Y, hipStream_t st, const float** parts = nullptr, int* splits = nullptr) {
  // about two workgroups per CU; every row range at least 256 rows (one round of the four waves); partials must fit
  int64_t s = ceil_div(2 * kNumCUs, (d / 64) * batch);
  const int64_t fit = (int64_t)(rt_bytes / ((size_t)batch * n * d * 4));
  if (s > fit) s = fit;
  if (s < 1) s = 1;
  const int64_t k_per_wg = round_up(ceil_div(d, s), 256);
  s = ceil_div(d, k_per_wg);
  float* part = s > 1 ? reinterpret_cast<float*>(scratch) : Y;
  const int64_t count = batch * n * d;
  auto go = [&](auto tb_c) {
    hipLaunchKernelGGL((skinny_rotate_kernel<TR, decltype(tb_c)::value>), dim3((unsigned)(d / 64), (unsigned)s, (unsigned)batch),
                       dim3(256), 0, st, X, ldx, n * ldx, R, ldr, (int)n, (int)d, (int)k_per_wg, part, count);
  };
  if (n <= 16) go(std::integral_constant<int, 1>{});
  else if (n <= 32) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 4>{});
  if (!launch_ok()) return false;
  if (parts) {  // the caller adds them
    *parts = part;
    *splits = (int)s;
    return true;
  }
  return s == 1 || launch_splitk_reduce(part, count, (int)s, Y, LossSum{}, st);
}

// Y [problems][rows][d] = X R (token-major, tokens on the rows of the GEMM; R as in launch_features_gemm) with the tile that fills the chip: the large one
// (TL) unless it leaves CUs without a tile, then 128 x 128 (bf16) or 64 x 64 (fp32).  Fake-quant calls, us, large / small
// tile: bf16 d = 4096, n = 128: 97 / 58, 1024: 105 / 64, 2048 (128 large tiles): 109 / 91, 2560: 112 / 116; d = 2048,
// n = 4096 (128): 67 / 53, 6144: 72 / 73; fp32 d = 1024, n = 256: 75 / 30, 4096 (256 large tiles): 84 / 80; d = 2048,
// n = 2048 (256): 154 / 142.
// The 256 x 128 tile of d % 256 != 0 wins in one round over the CUs or two nearly full ones, two 128 x 128 on a CU in any
// other number: 144 tiles 35.5 / 37.1, 240: 50.7 / 53.1, 288: 68.6 / 59.0, 320: 50.7 / 43.9, 384: 50.6 / 46.0,
// 432: 72.3 / 73.6, 480: 88.2 / 91.0, 576: 92.2 / 88.1, 1152: 176 / 164.
// Half the CUs or fewer with a 128 x 128 tile: 64 x 64 ones.  us, 128 / 64: d = 256, n = 200 18.8 / 15.4; 1024, 1000 20.4 / 17.7; 1024, 2000
// (128 tiles) 24.2 / 23.6; 2048, 200 31.4 / 28.0; 4096, 65 54.3 / 50.2; 4096, 400 (128) 57.6 / 55.1; 4096, 600 (160) 60.0 / 62.7; 2048, 1400
// (176) 34.2 / 35.9.
template <typename T, class TL>
static bool launch_rows_gemm(const T* X, int64_t ldx, int64_t x_batch_stride, const T* R, int64_t ldr, bool in_place, int64_t problems,
                             int64_t rows, int64_t d, float* Y, int64_t y_batch_stride, hipStream_t st) {
  auto go = [&](auto tile_tag) -> bool {
    using G = decltype(tile_tag);
    EpiStore<G> e;
    e.C = Y; e.ldc = d; e.batch_stride = y_batch_stride; e.split_stride = 0; e.M = (int)rows; e.N = (int)d;
    if constexpr (sizeof(T) == 4) {
      if (in_place)
        return launch_gemm<G, EpiStore<G>, false, true>(X, ldx, x_batch_stride, (int)rows, R, ldr, d * ldr, (int)d, d, 0, (int)problems, e, st);
    }
    return launch_gemm<G>(X, ldx, x_batch_stride, (int)rows, R, d, d * d, (int)d, d, 0, (int)problems, e, st);
  };
  if constexpr (sizeof(T) == 4) {
    return with_f32_tile(rows, d, problems, go);
  } else {
    if (ceil_div(rows, 128) * (d / 128) * problems <= kNumCUs / 2) return go(TB_64{});
    const int64_t tiles = ceil_div(rows, TL::BM) * ceil_div(d, TL::BN) * problems;
    bool small;
    if (TL::BN == 128) small = tiles <= kNumCUs / 2 || (tiles > kNumCUs && (tiles > 2 * kNumCUs || 6 * tiles < 5 * 2 * kNumCUs));
    else small = tiles <= kNumCUs / 2;
    return small ? go(TB_128{}) : go(TL{});
  }
}

// fp32, no gradient: whether Y stays in registers (128 x 128 tiles, features on the rows of the GEMM, row moments in its epilogue, as with
// bf16) instead of being written as rows and read again, 8 bytes a value that short rows do not hide.  Loss, us, rows / this (tiles of 128):
//   d = 128: 8192 tokens (64) 16.5 / 18.4, 12000 (94) 20.1 / 18.4, 20000 (157) 25.9 / 18.4, 131072 135 / 46, 64 problems of 4096 253 / 83,
//            300 of 512 (1200) 111 / 100, of 128 (300, one a problem: the grid rounds up to eight) 61 / 99
//   d = 256: 4096 (64) 18.5 / 26.2, 8192 (128) 27.6 / 26.8, 12000 (188) 34 / 27, 17000 (266) 45 / 41, 34000 (532) 72 / 59
//   d = 384: 8192 (192) 37.5 / 35.1, 12000 (282) 50 / 57, 17000 (399) 65 / 58;  512: 9000 (284) 57 / 73, 13000 (408) 75 / 73, 17000 (532) 94 / 105
//   d = 768, 9000 (426) 100 / 104;  1024, 6000 (376) 110 / 135, 16384 (1024) 269 / 259
static bool f32_moments(int64_t batch, int64_t n, int64_t d) {
  const int64_t own = ceil_div(n, TF::BN) * (d / TF::BM), tiles = own * batch;
  if (own < 4) return false;
  if (d <= 256) return tiles >= kNumCUs / 2;
  return d <= 512 ? 4 * tiles >= 3 * round_up(tiles, kNumCUs) : with_f32_tile(n, d, batch, [](auto t) { return std::is_same_v<decltype(t), TF>; });
}
static kt_status run_loss_f32(const LossGradPlan& p, const float* X, int64_t ldx, const float* R, int64_t ldr, bool in_place, int64_t batch,
                              int64_t n, int64_t d, float kappa_target, float* loss, float* row_kurt, char* ws, hipStream_t st,
                              const PooledArgs* pooled) {
  // (the room of Y is 4 d bytes a token: 0.25 d of partials, 16 of coefficients, 32 bytes of sums per 256)
  const int P = (int)(d / TF::BM) * TF::WGM, blocks = (int)ceil_div(n, 256);
  floatx4* part = reinterpret_cast<floatx4*>(ws + p.o_gt);
  floatx4* coef = part + batch * P * n;
  double* sums = reinterpret_cast<double*>(coef + batch * n);
  {
    ProfScope prof(0, st);
    EpiMoments<TF> e;
    e.part = part; e.n_tokens = (int)n; e.d = (int)d; e.P = P;
    if (!launch_features_gemm<TF>(R, ldr, in_place, X, ldx, batch, n, d, e, st)) return fail(KT_ERR_DEVICE, "forward GEMM launch failed");
  }
  if (pooled) {
    hipLaunchKernelGGL(pooled_stage1_kernel, dim3(blocks, (unsigned)batch), dim3(256), 0, st, part, P, (int)n, (int)d, pooled->rms_eps, sums);
    hipLaunchKernelGGL(pooled_stage2_kernel, dim3((unsigned)batch), dim3(256), 0, st, sums, blocks, (int)n, (int)d, kappa_target,
                       reinterpret_cast<double*>(ws + p.o_gstat), loss, pooled->kappa_out);
    return launch_ok() ? KT_OK : fail(KT_ERR_DEVICE, "pooled statistics launch failed");
  }
  hipLaunchKernelGGL(finalize_rows_kernel, dim3(blocks, (unsigned)batch), dim3(256), 0, st, part, P, (int)n, (int)d, kappa_target, coef,
                     row_kurt, sums);
  if (!launch_ok() || !launch_loss_sum(LossSum{sums, blocks, (int)n, (int)batch, loss}, st)) return fail(KT_ERR_DEVICE, "row statistics launch failed");
  return KT_OK;
}

// fp32: token-major throughout (kt_rows.h).  Y = X R in the workspace, dL/dY over it, dR = X^T (dL/dY) with K as the row index
// of both operands.
static kt_status run_loss_grad_f32(const LossGradPlan& p, const float* X, int64_t ldx, const float* R, int64_t ldr, int64_t batch,
                                   int64_t n, int64_t d, float kappa_target, float* loss, float* row_kurt, float* dR, char* ws,
                                   hipStream_t st, const PooledArgs* pooled = nullptr) {
  float* RT = reinterpret_cast<float*>(ws + p.o_rt);
  float* Y = reinterpret_cast<float*>(ws + p.o_gt);
  floatx4* part = pooled ? reinterpret_cast<floatx4*>(ws + p.o_part) : nullptr;
  double* sums = reinterpret_cast<double*>(ws + p.o_losspart);
  double* gstat = reinterpret_cast<double*>(ws + p.o_gstat);
  float* splitk = reinterpret_cast<float*>(ws + p.o_splitk);
  const bool in_place = f32_in_place(R, ldr);
  if (!in_place && !prep_rt<float>(R, ldr, KT_F32, RT, batch, d, st)) return fail(KT_ERR_DEVICE, "prep_rt launch failed");
  if (!dR && f32_moments(batch, n, d))
    return run_loss_f32(p, X, ldx, in_place ? R : RT, ldr, in_place, batch, n, d, kappa_target, loss, row_kurt, ws, st, pooled);
  {
    ProfScope prof(0, st);
    if (!launch_rows_gemm<float, TF>(X, ldx, n * ldx, in_place ? R : RT, ldr, in_place, batch, n, d, Y, p.ldt * d, st))
      return fail(KT_ERR_DEVICE, "forward GEMM launch failed");
  }
  const int wgs = p.loss_blocks;
  {
    ProfScope prof(1, st);
    auto rows_kernel = d == 128 ? loss_rows_kernel<1, 32> : d <= 1024 ? loss_rows_kernel<4, 64> : d <= 4096 ? loss_rows_kernel<16, 64>
                       : d <= 8192 ? loss_rows_kernel<32, 64> : loss_rows_kernel<0, 64>;
    hipLaunchKernelGGL(rows_kernel, dim3(wgs, (unsigned)batch), dim3(256), 0, st, Y, (int)p.ldt, (int)n, (int)d, kappa_target, row_kurt,
                       sums, dR ? 1 : 0, pooled ? pooled->rms_eps : 0.f, part);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "row statistics launch failed");
    if (pooled) {
      hipLaunchKernelGGL(pooled_stage2_kernel, dim3((unsigned)batch), dim3(256), 0, st, sums, wgs, (int)n, (int)d, kappa_target, gstat,
                         loss, pooled->kappa_out);
      if (dR) {
        auto grad_kernel = d == 128 ? pooled_grad_rows_kernel<32> : pooled_grad_rows_kernel<64>;
        hipLaunchKernelGGL(grad_kernel, dim3((unsigned)ceil_div(n, d == 128 ? 8 : 4), (unsigned)batch), dim3(256), 0, st, Y, (int)p.ldt, (int)n,
                           (int)d, pooled->rms_eps, part, gstat);
      }
      if (!launch_ok()) return fail(KT_ERR_DEVICE, "pooled statistics launch failed");
    }
  }
  const LossSum loss_sum = pooled ? LossSum{} : LossSum{sums, wgs, (int)n, (int)batch, loss};
  if (!dR || p.split_k == 1) {
    if (!pooled && !launch_loss_sum(loss_sum, st)) return fail(KT_ERR_DEVICE, "loss sum launch failed");
    if (!dR) return KT_OK;
  }
  ProfScope prof(2, st);
  auto go = [&](auto tile_tag) -> bool {
    using TL = decltype(tile_tag);
    EpiStore<TL> e;
    e.C = p.split_k > 1 ? splitk : dR;
    e.batch_stride = d * d; e.split_stride = p.split_k > 1 ? batch * d * d : 0;
    e.ldc = d; e.M = (int)d; e.N = (int)d;
    return launch_gemm<TL, EpiStore<TL>, true, true>(X, ldx, n * ldx, (int)d, Y, d, p.ldt * d, (int)d, p.ldt, p.slabs_per_split, (int)batch, e,
                                                     st, 0, 0, (int)n);
  };
  if (!with_f32_tile(d, d, batch * p.split_k, go)) return fail(KT_ERR_DEVICE, "gradient GEMM launch failed");
  if (p.split_k > 1 && !launch_splitk_reduce(splitk, batch * d * d, p.split_k, dR, loss_sum, st))
    return fail(KT_ERR_DEVICE, "split-K reduce launch failed");
  return KT_OK;
}

// ------------------------------------------------------------------ fake-quant ----
// Workgroups per problem for quant_d128_kernel.  A workgroup stages all of R before its first tile (the figures are with the copy of R^T that a launch of
// its own wrote, about 5 us more each).
//  - While one workgroup per CU holds them: one 16-token tile per wave.  us, one tile / two per wave: 1 problem of 4096 tokens
//    12.1 / 12.9, of 16384 12.1 / 13.2; two workgroups on a CU with one tile each: 32768 tokens 15.7 against 13.5.
//  - Beyond: two tiles or more per wave, and as many workgroups as finish first when they start in rounds of 512 (two per
//    CU, what the registers let it hold), a round taking its longest wave's tiles and R^T, about four more.  512 / batch
//    rounded up would leave a second round nearly empty: 100 x 16384 tokens 223 us, here 156; 200 x 16384 415 and 300; 40 x
//    65536 343 and 238.
static int64_t quant_d128_wgs(int64_t batch, int64_t n) {
  const int64_t tiles = ceil_div(n, 16);
  if (ceil_div(tiles, 4) * batch <= kNumCUs) return ceil_div(tiles, 4);
  int64_t best = 1, least = -1;
  for (int64_t k = 1; k <= ceil_div(tiles, 8) && k <= 4 * ceil_div(2 * kNumCUs, batch); ++k) {
    const int64_t cost = ceil_div(k * batch, 2 * kNumCUs) * (ceil_div(tiles, 4 * k) + 4);
    if (least < 0 || cost < least) { best = k; least = cost; }
  }
  return best;
}

// Codes straight from the accumulators, the row's maximum taken between the tiles (kt_rowsync.h): no staged Y.
// KT_ERR_NOT_SUPPORTED: not a size for it.
static kt_status run_quant_row_sync(const QuantPlan& p, const bf16* X, int64_t ldx, const void* R, int64_t ldr, kt_dtype rdt, int64_t batch,
                                    int64_t n, int64_t d, float clip, float* scales_out, int8_t* codes, float* err, char* ws, hipStream_t st) {
  auto go = [&](auto tile_tag) -> kt_status {
    using TL = decltype(tile_tag);
    RowSync rs;
    if (!row_sync_shape<TL>(batch, n, d, &rs)) return KT_ERR_NOT_SUPPORTED;
    const int64_t tiles = (int64_t)rs.rows * rs.cols, P = rs.cols * TL::WGM;
    const int64_t counters = kRowSyncWords + 2 * (int64_t)rs.rows;
    Carver c;  // in the room of the staged rows
    const size_t o_words = c.take((size_t)counters * kRowSyncPitch * 4), o_links = c.take((size_t)tiles * 4);
    const size_t o_amax = c.take((size_t)batch * P * n * 4), o_err = c.take(err ? (size_t)batch * P * n * 8 : 0);
    if (p.o_y + c.off > p.total) return KT_ERR_NOT_SUPPORTED;
    char* room = ws + p.o_y;
    rs.words = reinterpret_cast<unsigned*>(room + o_words);
    rs.pitch = kRowSyncPitch;
    bf16* RT = reinterpret_cast<bf16*>(ws + p.o_rt);
    if (!prep_rt<bf16>(R, ldr, rdt, RT, batch, d, st, rs.words, counters * rs.pitch))
      return fail(KT_ERR_DEVICE, "prep_rt launch failed");
    RowQuant<TL> op;
    op.amax.part = reinterpret_cast<float*>(room + o_amax);
    op.amax.n_tokens = (int)n; op.amax.d = (int)d; op.amax.P = (int)P;
    op.quant.scales = nullptr; op.quant.codes = codes; op.quant.err_part = err ? reinterpret_cast<float2*>(room + o_err) : nullptr;
    op.quant.n_tokens = (int)n; op.quant.d = (int)d; op.quant.P = (int)P;
    op.clip = clip; op.scales_out = scales_out; op.err = reinterpret_cast<float2*>(err);
    op.links = reinterpret_cast<int*>(room + o_links);
    op.added = rs.words + (kRowSyncWords + (int64_t)rs.rows) * rs.pitch;
    op.pitch = rs.pitch;
    op.cols = rs.cols;
    return launch_row_sync<TL>(rs, RT, X, ldx, n, d, op, st) ? KT_OK : fail(KT_ERR_DEVICE, "rotation GEMM launch failed");
  };
  const RowSyncTile tile = quant_row_sync_tile(batch, n, d);
  return tile == RowSyncTile::large ? go(TB_BIG{}) : tile == RowSyncTile::small ? go(TB_128{}) : KT_ERR_NOT_SUPPORTED;
}

template <typename T, class TFWD, class TQ>
static kt_status run_quant(const QuantPlan& p, const void* X, int64_t ldx, const void* R, int64_t ldr,
                           kt_dtype rdt, int64_t batch, int64_t n, int64_t d, float clip,
                           const float* scales_in, float* scales_out, int8_t* codes, float* err,
                           char* ws, hipStream_t st) {
  T* RT = reinterpret_cast<T*>(ws + p.o_rt);
  float* amax = reinterpret_cast<float*>(ws + p.o_amax);
  float* scales_ws = reinterpret_cast<float*>(ws + p.o_scales);
  float2* errpart = reinterpret_cast<float2*>(ws + p.o_errpart);
  const T* Xp = static_cast<const T*>(X);
  const bool staged = !scales_in && (codes || err);
  const bool skinny = staged && p.stage_problems == batch && skinny_ok(sizeof(T) == 2 ? KT_BF16 : KT_F32, R, ldr, rdt, n);
  const bool in_place = sizeof(T) == 4 && f32_in_place(R, ldr);
  if constexpr (sizeof(T) == 2) {
    if (staged && !skinny) {
      const kt_status s = run_quant_row_sync(p, Xp, ldx, R, ldr, rdt, batch, n, d, clip, scales_out, codes, err, ws, st);
      if (s != KT_ERR_NOT_SUPPORTED) return s;
    }
  }
  if (!skinny && !in_place && !prep_rt<T>(R, ldr, rdt, RT, batch, d, st)) return fail(KT_ERR_DEVICE, "prep_rt launch failed");
  const T* Rg = in_place ? static_cast<const T*>(R) : RT;
  const int64_t r_stride = in_place ? d * ldr : d * d;
  const float* scales = scales_in;
  if (staged) {
    // One GEMM instead of two: Y = X R is staged in fp32 (token-major: tokens on the rows of the GEMM), a
    // row kernel takes the maximum and quantises.  4 n d bytes written and read against 2 n d^2 flop saved.
    float* Ybuf = reinterpret_cast<float*>(ws + p.o_y);
    for (int64_t b0 = 0; b0 < batch; b0 += p.stage_problems) {
      const int64_t nb = batch - b0 < p.stage_problems ? batch - b0 : p.stage_problems;
      for (int64_t t0 = 0; t0 < n; t0 += p.stage_rows) {
        const int64_t nt = n - t0 < p.stage_rows ? n - t0 : p.stage_rows;
        bool ok;
        const float* parts = Ybuf;
        int splits = 1;
        if (skinny) {
          const bf16* Xb = reinterpret_cast<const bf16*>(Xp);
          ok = rdt == KT_F32 ? launch_skinny(Xb, ldx, static_cast<const float*>(R), ldr, batch, n, d, ws + p.o_rt, p.o_amax - p.o_rt, Ybuf, st, &parts, &splits)
                             : launch_skinny(Xb, ldx, static_cast<const bf16*>(R), ldr, batch, n, d, ws + p.o_rt, p.o_amax - p.o_rt, Ybuf, st, &parts, &splits);
        } else {
          ok = launch_rows_gemm<T, TQ>(Xp + (b0 * n + t0) * ldx, ldx, n * ldx, Rg + b0 * r_stride, ldr, in_place, nb, nt, d, Ybuf, nt * d, st);
        }
        if (!ok) return fail(KT_ERR_DEVICE, "rotation GEMM launch failed");
        const int64_t rows = nb * nt, row0 = b0 * n + t0;
        float* so = scales_out ? scales_out + row0 : nullptr;
        int8_t* co = codes ? codes + row0 * d : nullptr;
        float2* eo = err ? reinterpret_cast<float2*>(err) + row0 : nullptr;
        const dim3 grid((unsigned)ceil_div(rows, 4));
        if (skinny) {
          auto kern = d <= 4096 ? quant_partials_kernel<1> : d <= 8192 ? quant_partials_kernel<2> : quant_partials_kernel<4>;
          const int64_t threads = round_up(d / 4, 64) < 1024 ? round_up(d / 4, 64) : 1024;
          hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3((unsigned)threads), 0, st, parts, batch * n * d, splits, (int)d, clip, so, co, eo);
        } else if (d <= 1024)
          hipLaunchKernelGGL((quant_rows_kernel<4, true>), grid, dim3(256), 0, st, Ybuf, rows, (int)d, clip, so, co, eo);
        else if (d <= 4096)
          hipLaunchKernelGGL((quant_rows_kernel<16, true>), grid, dim3(256), 0, st, Ybuf, rows, (int)d, clip, so, co, eo);
        else if (d <= 8192)
          hipLaunchKernelGGL((quant_rows_kernel<32, true>), grid, dim3(256), 0, st, Ybuf, rows, (int)d, clip, so, co, eo);
        else
          hipLaunchKernelGGL((quant_rows_kernel<1, false>), grid, dim3(256), 0, st, Ybuf, rows, (int)d, clip, so, co, eo);
        if (!launch_ok()) return fail(KT_ERR_DEVICE, "row quantiser launch failed");
      }
    }
    return KT_OK;
  }
  if (!scales_in) {
    EpiAmax<TFWD> e;
    e.part = amax; e.n_tokens = (int)n; e.d = (int)d; e.P = p.P;
    if (!launch_features_gemm<TFWD>(Rg, ldr, in_place, Xp, ldx, batch, n, d, e, st))
      return fail(KT_ERR_DEVICE, "amax GEMM launch failed");
    hipLaunchKernelGGL(quant_scale_kernel, dim3((unsigned)ceil_div(n, 256), (unsigned)batch), dim3(256),
                       0, st, amax, p.P, n, clip, scales_ws, scales_out);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "scale kernel launch failed");
    scales = scales_ws;
  } else if (scales_out) {
    if (hipMemcpyAsync(scales_out, scales_in, (size_t)batch * n * 4, hipMemcpyDeviceToDevice, st) != hipSuccess)
      return fail(KT_ERR_DEVICE, "scale copy failed");
  }
  if (!codes && !err) return KT_OK;
  {
    EpiQuant<TFWD> e;
    e.scales = scales; e.codes = codes; e.err_part = err ? errpart : nullptr;
    e.n_tokens = (int)n; e.d = (int)d; e.P = p.P;
    if (!launch_features_gemm<TFWD>(Rg, ldr, in_place, Xp, ldx, batch, n, d, e, st))
      return fail(KT_ERR_DEVICE, "quantise GEMM launch failed");
  }
  if (err) {
    hipLaunchKernelGGL(quant_err_kernel, dim3((unsigned)ceil_div(n, 256), (unsigned)batch), dim3(256), 0,
                       st, errpart, p.P, n, reinterpret_cast<float2*>(err));
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "error reduce launch failed");
  }
  return KT_OK;
}

}  // namespace kt

using namespace kt;

// =================================================================== C ABI =========
// d = 128: one workgroup per problem does the whole step (kt_cayley_d128.h).
template <bool ADAM>
static kt_status launch_cayley_d128(float* R, const float* G, void* R_lowp, int64_t batch, float half_coef,
                                    float* ortho_err, int32_t* info, const C128Adam& ad, hipStream_t st) {
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(cayley_d128_kernel<ADAM>), kC128LdsBytes))
    return fail(KT_ERR_DEVICE, "the d=128 Cayley kernel needs %d bytes of LDS per workgroup", kC128LdsBytes);
  hipLaunchKernelGGL(cayley_d128_kernel<ADAM>, dim3((unsigned)batch), dim3(256), kC128LdsBytes, st, R, G,
                     static_cast<__bf16*>(R_lowp), half_coef, ortho_err, info, kCayleyMaxIters, kCayleyTol, ad);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley d=128 launch failed");
  return KT_OK;
}

// Optional Cayley Adam part of a retraction: moments already updated, r in scal[4b].
struct AdamArgs {
  float* M;            // [batch][d][d] momentum: in = beta1 M + (1-beta1) G, out = r W R
  float lr, q, eps;
  float* scal;         // [batch][4] device scalars {r, alpha, ||W||, alpha/(2r)}
  double* sq_part;     // [batch][(d/32)^2] tile partials of ||S||^2
  float* scalars_out;  // [batch][3] {r, alpha, ||W||} for the caller, or null
  AdamScalars first;   // fp16 operands: taken with them (split3_kernel), and their maxima are there (adam_moment_kernel)
};

// Shared by the two optimisers.  P = G R^T, S = half_coef (P - P^T), then the Cayley transform
// Z = (I + c S)^-1 (I - c S) R by the fixed point in transposed space (c = 1, or alpha/(2r) from
// device memory for Adam), R <- Z.  For Adam, between set-up and iteration: step scalars, and
// M <- S R (the momentum moved into the tangent space at R).
static kt_status cayley_run(const CayleyPlan& p, char* ws, float* R, const float* G, void* R_lowp, int64_t batch,
                            int64_t d, float half_coef, const AdamArgs* adam, float* ortho_err, int32_t* info,
                            hipStream_t st) {
  float* Mm = reinterpret_cast<float*>(ws + p.o_m);
  float* Bm = reinterpret_cast<float*>(ws + p.o_b);
  float* Rt = reinterpret_cast<float*>(ws + p.o_rt);
  float* Zt = reinterpret_cast<float*>(ws + p.o_zt);
  float* U[2] = {reinterpret_cast<float*>(ws + p.o_u0), reinterpret_cast<float*>(ws + p.o_u1)};
  unsigned* delta = reinterpret_cast<unsigned*>(ws + p.o_delta);
  const int D = (int)d;
  const int64_t dd = d * d;
  const bool small = small_f32_tiles(d, batch);
  // The control words of the iterations lie where Cayley Adam had its block sums of ||G||^2, cleared by the set-up kernel; a
  // tile grid too large for that room takes that of the sums of ||S||^2, behind the kernel that reads them.
  const int64_t control_words = p.split ? with_f16_iterate_tile(d, batch, [&](auto t) { return cayley_control_words<decltype(t)>(d); })
                                        : (small ? cayley_control_words<TF_64>(d) : cayley_control_words<TF>(d));
  const int64_t room = (int64_t)p.g2_blocks * 8 - (p.split ? (int64_t)sizeof(SplitScales) : 0);
  const bool late_control = control_words * 4 > room;
  SplitScales* scales = reinterpret_cast<SplitScales*>(ws + p.o_g2 + batch * room);
  unsigned* control = reinterpret_cast<unsigned*>(ws + (late_control ? p.o_sq : p.o_g2));
  const int ncontrol = late_control ? 0 : (int)control_words;
  // (fp16: the changes of a second iteration that counts as the last, EpiCayleyIter)
  const float second_tol = 5e-4f / sqrtf((float)d);
  // B and U: rows of ld values
  auto iterations = [&](auto first_tag, auto tile_tag, auto* U0, auto* U1, const auto* B, int64_t K, int64_t ld) -> bool {
    auto epilogue = [&](auto tag, auto phase_c) {
      using TL = decltype(tag);
      EpiCayleyIter<TL, decltype(phase_c)::value> e;
      e.Rt = Rt; e.Zt = Zt; e.Unew = nullptr; e.Usplit = nullptr; e.delta = delta;
      e.d = D; e.it = 0; e.max_iters = kCayleyMaxIters; e.tol = kCayleyTol; e.second_tol = second_tol;
      e.bscale = adam ? adam->scal : nullptr;
      e.scales = scales;
      return e;
    };
    using TL = decltype(tile_tag);
    using First = decltype(first_tag);
    constexpr auto later = std::integral_constant<int, 2>{};
    const int own = cayley_own_launches(ceil_div(d, TL::BM) * ceil_div(d, TL::BN), batch, TL::BM, p.split);
    int it = 0;
    if constexpr (sizeof(*B) == 2) {
      auto e0 = epilogue(first_tag, std::integral_constant<int, 0>{});
      e0.Usplit = U1;
      if (!launch_gemm_few<First>(U0, ld, d * ld, D, B, ld, d * ld, D, K, 0, (int)batch, e0, st, d)) return false;
      auto e1 = epilogue(first_tag, std::integral_constant<int, 1>{});
      e1.it = 1;
      if (!launch_gemm_few<First>(U1, d, dd, D, B, ld, d * ld, D, d, 0, (int)batch, e1, st, d)) return false;
      hipLaunchKernelGGL(cayley_u_kernel, dim3(D / 32, D / 32, (unsigned)batch), dim3(256), 0, st, R, Zt, D, Rt, U0, scales, delta,
                         kCayleyMaxIters, kCayleyTol, second_tol);
      it = 2;
    }
    for (; it < own; ++it) {
      auto e = epilogue(first_tag, later);
      auto *from = it & 1 ? U1 : U0, *to = it & 1 ? U0 : U1;
      e.it = it;
      if constexpr (sizeof(*B) == 2) e.Usplit = to;
      else e.Unew = to;
      if constexpr (sizeof(*B) == 2) {
        if (!launch_gemm_few<First>(from, ld, d * ld, D, B, ld, d * ld, D, K, 0, (int)batch, e, st, d)) return false;
      } else if (!launch_gemm<First>(from, ld, d * ld, D, B, ld, d * ld, D, K, 0, (int)batch, e, st, d)) return false;
    }
    if (own == kCayleyMaxIters) return true;
    if (late_control) hipLaunchKernelGGL(fill_u32_kernel, dim3(64), dim3(256), 0, st, control, batch * control_words, 0u);
    return launch_cayley_iterations<TL>(U0, U1, B, K, d, ld, batch, epilogue(tile_tag, later), control, own, st);
  };

  if (p.split) {
    // three-term path: operands live as [d][2d] fp16, rows of [head | tail]
    _Float16* Bs = reinterpret_cast<_Float16*>(ws + p.o_b);
    _Float16* Us[2] = {reinterpret_cast<_Float16*>(ws + p.o_u0), reinterpret_cast<_Float16*>(ws + p.o_u1)};
    const int64_t sd = 2 * d * d;
    const unsigned sb = (unsigned)(ceil_div(dd, 1024) < 2048 ? ceil_div(dd, 1024) : 2048);
    // M = dR R^T with dR in Us[0] and R in Us[1]; the partial maxima in the room of M
    unsigned* maxima = reinterpret_cast<unsigned*>(Mm);
    if (!adam) hipLaunchKernelGGL(split_max_kernel, dim3(256, 2, (unsigned)batch), dim3(256), 0, st, G, R, dd, maxima);
    hipLaunchKernelGGL(split3_kernel, dim3(sb, adam ? 3 : 2, (unsigned)batch), dim3(256), 0, st, G, R, D, maxima, Us[0], Us[1], scales,
                       adam ? adam->first : AdamScalars{});
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "split launch failed");
    auto product = [&](const _Float16* A3, const _Float16* B3, const int* exp_a, const int* exp_b, float* C, unsigned* max_word, int shift) -> bool {
      return with_f16_tile(d, batch, [&](auto tile_tag) -> bool {
        using TL = decltype(tile_tag);
        EpiStoreScaled<TL> e;
        e.C = C; e.exp_a = exp_a; e.exp_b = exp_b; e.max_word = max_word; e.d = D; e.shift = shift;
        return launch_gemm_few<TL>(A3, 2 * d, sd, D, B3, 2 * d, sd, D, 3 * d, 0, (int)batch, e, st, d);
      });
    };
    if (!product(Us[0], Us[1], &scales->g, &scales->r, Mm, &scales->max_m, 0)) return fail(KT_ERR_DEVICE, "dR R^T GEMM launch failed");
    hipLaunchKernelGGL(cayley_setup_kernel, dim3(D / 32, D / 32, (unsigned)batch), dim3(256), 0, st, Mm, R,
                       D, half_coef, (float*)nullptr, Rt, Zt, (float*)nullptr, Bs, Us[0], scales, adam ? adam->sq_part : nullptr, delta,
                       kCayleyMaxIters, control, ncontrol);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley set-up launch failed");
    if (adam) {
      hipLaunchKernelGGL(adam_scalars2_kernel, dim3((unsigned)batch), dim3(256), 0, st, adam->sq_part,
                         (int)((d / 32) * (d / 32)), adam->lr, adam->q, adam->eps, adam->scal, adam->scalars_out);
      if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley Adam scalar launch failed");
      // M <- S R = (1/2) S (2 Rt)^T: S sits in Bs, 2 Rt in Us[0]
      if (!product(Bs, Us[0], &scales->b, &scales->u, adam->M, nullptr, -1)) return fail(KT_ERR_DEVICE, "momentum projection GEMM launch failed");
    }
    const bool launched = with_f16_tile(d, batch, [&](auto first) {
      return with_f16_iterate_tile(d, batch, [&](auto t) { return iterations(first, t, Us[0], Us[1], Bs, 3 * d, 2 * d); });
    });
    if (!launched) return fail(KT_ERR_DEVICE, "Cayley iteration launch failed");
  } else {
  auto product = [&](const float* A, const float* B, float* C) -> bool {  // C = A B^T
    auto go = [&](auto tile_tag) -> bool {
      using TL = decltype(tile_tag);
      EpiStore<TL> e;
      e.C = C; e.ldc = d; e.batch_stride = dd; e.split_stride = 0; e.M = D; e.N = D;
      return launch_gemm<TL>(A, d, dd, D, B, d, dd, D, d, 0, (int)batch, e, st);
    };
    return with_f32_tile(d, d, batch, go);
  };
  if (!product(G, R, Mm)) return fail(KT_ERR_DEVICE, "dR R^T GEMM launch failed");
  hipLaunchKernelGGL(cayley_setup_kernel, dim3(D / 32, D / 32, (unsigned)batch), dim3(256), 0, st, Mm, R,
                     D, half_coef, Bm, Rt, Zt, U[0], (_Float16*)nullptr, (_Float16*)nullptr, (SplitScales*)nullptr, adam ? adam->sq_part : nullptr,
                     delta, kCayleyMaxIters, control, ncontrol);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley set-up launch failed");
  if (adam) {
    hipLaunchKernelGGL(adam_scalars2_kernel, dim3((unsigned)batch), dim3(256), 0, st, adam->sq_part,
                 (int)((d / 32) * (d / 32)), adam->lr, adam->q, adam->eps, adam->scal, adam->scalars_out);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley Adam scalar launch failed");
    // M <- S R = S (Rt)^T
    if (!product(Bm, Rt, adam->M)) return fail(KT_ERR_DEVICE, "momentum projection GEMM launch failed");
  }
  const bool launched = with_f32_tile(d, d, batch, [&](auto first) {
    return small ? iterations(first, TF_64{}, U[0], U[1], Bm, d, d) : iterations(first, TF{}, U[0], U[1], Bm, d, d);
  });
  if (!launched) return fail(KT_ERR_DEVICE, "Cayley iteration launch failed");
  }
  hipLaunchKernelGGL(p.split ? cayley_finish_kernel<true> : cayley_finish_kernel<false>, dim3(D / 32, D / 32, (unsigned)batch), dim3(256), 0, st, Zt, D,
                     R, static_cast<__bf16*>(R_lowp), delta, kCayleyMaxIters, kCayleyTol, second_tol, ortho_err ? 1 : 0, info);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley wrap-up launch failed");
  if (ortho_err) {
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<unsigned*>(ortho_err),
                       batch, 0u);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "fill launch failed");
    auto off_diagonal = [&](auto tile_tag) -> bool {  // Zt Zt^T = R^T R
      using TL = decltype(tile_tag);
      EpiOrtho<TL> e;
      e.err = reinterpret_cast<unsigned*>(ortho_err); e.d = D;
      return launch_gemm<TL>(Zt, d, dd, D, Zt, d, dd, D, d, 0, (int)batch, e, st);
    };
    if (!with_f32_tile(d, d, batch, off_diagonal))
      return fail(KT_ERR_DEVICE, "orthogonality GEMM launch failed");
    hipLaunchKernelGGL(ortho_diag_kernel, dim3(D, (unsigned)batch), dim3(256), 0, st, Zt, D,
                       reinterpret_cast<unsigned*>(ortho_err));
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "orthogonality diagonal launch failed");
  }
  return KT_OK;
}


// ------------------------------------------------------------- Hadamard rows ----
template <typename T, int LOG2D>
static kt_status launch_hadamard(const void* X, int64_t ldx, void* Y, int64_t ldy, const int8_t* signs, int64_t n,
                                 float scale, int sign_rows, hipStream_t st) {
  constexpr size_t lds = 4 * (size_t)kHadRegion * 4;
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(hadamard_rows_kernel<T, LOG2D>), lds))
    return fail(KT_ERR_DEVICE, "the Hadamard kernel needs %d bytes of LDS per workgroup", (int)lds);
  const int64_t rows = kHadChunk >> LOG2D, chunks = ceil_div(n, rows);
  const int64_t wgs = ceil_div(chunks, 4) < 2 * kNumCUs ? ceil_div(chunks, 4) : 2 * kNumCUs;
  hipLaunchKernelGGL((hadamard_rows_kernel<T, LOG2D>), dim3((unsigned)wgs), dim3(256), lds, st,
                     static_cast<const T*>(X), ldx, static_cast<T*>(Y), ldy, signs, n, scale, sign_rows);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Hadamard launch failed");
  return KT_OK;
}

template <typename T>
static kt_status dispatch_hadamard(int log2d, const void* X, int64_t ldx, void* Y, int64_t ldy,
                                   const int8_t* signs, int64_t n, float scale, int sign_rows, hipStream_t st) {
  switch (log2d) {
    case 7: return launch_hadamard<T, 7>(X, ldx, Y, ldy, signs, n, scale, sign_rows, st);
    case 8: return launch_hadamard<T, 8>(X, ldx, Y, ldy, signs, n, scale, sign_rows, st);
    case 9: return launch_hadamard<T, 9>(X, ldx, Y, ldy, signs, n, scale, sign_rows, st);
    case 10: return launch_hadamard<T, 10>(X, ldx, Y, ldy, signs, n, scale, sign_rows, st);
    case 11: return launch_hadamard<T, 11>(X, ldx, Y, ldy, signs, n, scale, sign_rows, st);
    default: return launch_hadamard<T, 12>(X, ldx, Y, ldy, signs, n, scale, sign_rows, st);
  }
}

static bool is_prime(int64_t q) {
  if (q < 2) return false;
  for (int64_t t = 2; t * t <= q; ++t)
    if (q % t == 0) return false;
  return true;
}

// How a row length splits into H_d = H_m (x) S_p2 (stated in kt.h).  kind 0: H_m Sylvester,
// 1: Paley's first construction, 2: Paley's second.  False when there is no such split.
static bool hadamard_split(int64_t d, int* m, int* p2, int* kind) {
  int64_t r = d;
  int t = 0;
  while (r > 1 && (r & 1) == 0) { r >>= 1; ++t; }
  if (r == 1) {
    int64_t mm = 1;
    if (t > 12) mm = (int64_t(1) << (t - 12)) < 4 ? 4 : (int64_t(1) << (t - 12));
    *m = (int)mm; *p2 = (int)(d / mm); *kind = 0;
    return true;
  }
  for (int j = 2; j <= t; ++j) {
    const int64_t mm = r << j;
    if (mm > 256) break;
    const int k = is_prime(mm - 1) ? 1 : (is_prime(mm / 2 - 1) && (mm / 2 - 1) % 4 == 1) ? 2 : 0;
    if (k) { *m = (int)mm; *p2 = (int)(d / mm); *kind = k; return true; }
  }
  return false;
}

// One pass over bf16 rows (hadamard_onepass_kernel) for H_m (x) S_p2 with m > 1 where a row fits the LDS of a workgroup.
// Returns false when the sizes do not fit its layout.  One exception: 32768 = S_8 (x) S_4096 on few rows, where the set-up
// of eight waves costs more than the second kernel (16 rows: 13.6 us in one pass, 12.4 in two; 64: 14.3 and 13.4, 88: 14.5
// and 14.8, 256: 16.7 and 26.6; from 64 rows on the result is rounded once only).
static bool hadamard_onepass_plan(int64_t n, int64_t d, int m, int p2, int kind, int* log2j, int* logp) {
  if (d > 32768 || (kind == 0 && d > 16384 && n < 64)) return false;
  const int limit = d > 16384 ? 256 : 128;  // 32 outputs per wave, 8 or 4 waves
  int j = 0;
  while ((m << (j + 1)) <= limit && (p2 >> (j + 1)) >= 64) ++j;
  int lp = 0;
  while ((1 << lp) < (p2 >> j)) ++lp;
  *log2j = j; *logp = lp;
  return lp == 7 || (lp == 6 && d <= 16384);
}

template <int LOGP, int WAVES>
static kt_status launch_hadamard_onepass(const bf16* X, int64_t ldx, bf16* Y, int64_t ldy, const int8_t* signs, int64_t n,
                                         int64_t d, const HadamardFactor& f, hipStream_t st) {
  const int M = f.m << f.log2j;
  const size_t lds = (size_t)((M + 15) / 16 * 16) * (2 << LOGP);
  if (!ensure_dynamic_lds(reinterpret_cast<const void*>(hadamard_onepass_kernel<LOGP, WAVES>), lds))
    return fail(KT_ERR_DEVICE, "the Hadamard kernel needs %zu bytes of LDS per workgroup", lds);
  const int64_t wgs = (WAVES == 4 ? 2 : 1) * kNumCUs;  // what the registers let a CU hold
  hipLaunchKernelGGL((hadamard_onepass_kernel<LOGP, WAVES>), dim3((unsigned)(n < wgs ? n : wgs)), dim3(64 * WAVES), lds, st, X, ldx, Y, ldy,
                     signs, n, 65536.0f / sqrtf((float)d), f);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Hadamard launch failed");
  return KT_OK;
}

static HadamardFactor hadamard_factor(int m, int kind, int log2j) {
  HadamardFactor f;
  f.m = m; f.kind = kind; f.log2j = log2j;
  f.h = kind == 2 ? m / 2 : m;
  f.q = f.h - 1;
  f.squares[0] = f.squares[1] = 0;
  if (kind != 0)
    for (int t = 1; t < f.q; ++t) f.squares[t * t % f.q >> 6] |= 1ull << (t * t % f.q & 63);
  return f;
}
static kt_status run_hadamard_onepass(const bf16* X, int64_t ldx, bf16* Y, int64_t ldy, const int8_t* signs, int64_t n,
                                      int64_t d, int m, int kind, int log2j, int logp, hipStream_t st) {
  const HadamardFactor f = hadamard_factor(m, kind, log2j);
  if (d > 16384) return launch_hadamard_onepass<7, 8>(X, ldx, Y, ldy, signs, n, d, f, st);
  return logp == 6 ? launch_hadamard_onepass<6, 4>(X, ldx, Y, ldy, signs, n, d, f, st)
                   : launch_hadamard_onepass<7, 4>(X, ldx, Y, ldy, signs, n, d, f, st);
}

// fp32 rows with m > 1 in one pass (hadamard_f32_onepass_kernel): LDS for a row and H_m, 0 where two kernels are faster or they do not fit a
// workgroup.  us, two kernels / one pass: m = 4, 8: d = 8192, 1 row 14.1 / 12.3, 300 19.6 / 11.7, 8000 228 / 195; 16384, 8000 440 / 358; 32768, 16 14.3 /
// 15.7, 100 21.4 / 16.9, 8000 873 / 730.  m = 108 (13824): 1 51.6 / 51.0, 1000 226 / 177, 8000 1543 / 1376.  m = 12, 20: 5120, 16 15.9 / 11.5, 1000
// 34.3 / 21.7, 8000 153 / 154; 6144, 8000 149 / 161.  m = 28: 14336, 16 17.4 / 19.1, 100 20.6 / 19.8, 1000 55.4 / 49.1, 8000 391 / 385; 28672, 16 17.8 /
// 22.1, 8000 775 / 874.
static size_t hadamard_f32_lds(int64_t n, int64_t d, int m, int kind) {
  const size_t bytes = ((size_t)ceil_div(d, kHadChunk) * kHadRegion + (size_t)m * m) * 4;
  if (d > 8 * kHadChunk || bytes > 160 * 1024) return 0;
  bool faster;
  if (kind == 0) faster = d <= 4 * kHadChunk || n >= 64;
  else if (m >= 64) faster = true;
  else faster = n <= 4 * kNumCUs && (d <= 2 * kHadChunk || (d <= 4 * kHadChunk && n >= 64));
  return faster ? bytes : 0;
}
static kt_status launch_hadamard_f32_onepass(const float* X, int64_t ldx, float* Y, int64_t ldy, const int8_t* signs, int64_t n, int64_t d,
                                             int m, int p2, int kind, size_t lds, hipStream_t st) {
  const HadamardFactor f = hadamard_factor(m, kind, 0);
  int log2p = 0;
  while ((1 << log2p) < p2) ++log2p;
  auto go = [&](auto kernel, int waves) -> kt_status {
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds))
      return fail(KT_ERR_DEVICE, "the Hadamard kernel needs %zu bytes of LDS per workgroup", lds);
    const int64_t wgs = (int64_t)kNumCUs * (160 * 1024 / lds < 2 ? 1 : 2);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n < wgs ? n : wgs)), dim3(64 * waves), lds, st, X, ldx, Y, ldy, signs, n, (int)d, p2, log2p,
                       1.0f / sqrtf((float)d), f);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "Hadamard launch failed");
    return KT_OK;
  };
  return d <= 4 * kHadChunk ? go(&hadamard_f32_onepass_kernel<4>, 4) : go(&hadamard_f32_onepass_kernel<8>, 8);
}

template <typename T>
static kt_status run_hadamard(const void* X, int64_t ldx, void* Y, int64_t ldy, const int8_t* signs, int64_t n,
                              int64_t d, int m, int p2, int kind, hipStream_t st) {
  int log2p = 0;
  while ((1 << log2p) < p2) ++log2p;
  int log2j = 0, logp = 0;
  if (sizeof(T) == 2 && m > 1 && hadamard_onepass_plan(n, d, m, p2, kind, &log2j, &logp))
    return run_hadamard_onepass(static_cast<const bf16*>(X), ldx, static_cast<bf16*>(Y), ldy, signs, n, d, m, kind, log2j, logp, st);
  if constexpr (sizeof(T) == 4) {
    const size_t lds = m > 1 ? hadamard_f32_lds(n, d, m, kind) : 0;
    if (lds && (!signs || (reinterpret_cast<uintptr_t>(signs) & 3) == 0))
      return launch_hadamard_f32_onepass(static_cast<const float*>(X), ldx, static_cast<float*>(Y), ldy, signs, n, d, m, p2, kind, lds, st);
  }
  const float scale = 1.0f / sqrtf((float)d);
  // the Sylvester factor on the m segments of every row (p2 consecutive elements at a * p2), X -> Y:
  // contiguous rows are one matrix of n * m short rows; otherwise one launch per segment
  if (ldx == d && ldy == d && n * m < ((int64_t)1 << 31)) {
    kt_status s = dispatch_hadamard<T>(log2p, X, p2, Y, p2, signs, n * m, scale, m, st);
    if (s != KT_OK) return s;
  } else {
    for (int a = 0; a < m; ++a) {
      kt_status s = dispatch_hadamard<T>(log2p, static_cast<const T*>(X) + (int64_t)a * p2, ldx,
                                         static_cast<T*>(Y) + (int64_t)a * p2, ldy,
                                         signs ? signs + (int64_t)a * p2 : nullptr, n, scale, 1, st);
      if (s != KT_OK) return s;
    }
  }
  if (m == 1) return KT_OK;
  // the order-m factor across the segments, in place on Y
  const int64_t tiles = n * (p2 / 128);
  const int64_t wgs = tiles < 8 * kNumCUs ? tiles : 8 * kNumCUs;
  if (sizeof(T) == 2 && m >= kHadMfmaFrom) {  // bf16: exact on the matrix cores
    const int MB = (m + 31) / 32, KS = (m + 15) / 16;
    int lognb = 0;  // blocks of 32 columns per wave: as many as keep m * NBW <= 128, fit the segment and 64 KiB of LDS
    while ((2 << lognb) * m <= 128 && (256 << lognb) <= p2 && 2 * 16 * KS * (512 << lognb) <= 65536) ++lognb;
    const size_t lds = (size_t)32 * MB * 32 * KS + (size_t)16 * KS * (256 << lognb) + (size_t)32 * MB * ((256 << lognb) + 16);
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(hadamard_cross_mfma_kernel), lds))
      return fail(KT_ERR_DEVICE, "the Hadamard factor kernel needs %zu bytes of LDS per workgroup", lds);
    const int64_t tiles_m = n * (p2 / (128 << lognb));
    const int64_t wgs_m = tiles_m < 8 * kNumCUs ? tiles_m : 8 * kNumCUs;
    hipLaunchKernelGGL(hadamard_cross_mfma_kernel, dim3((unsigned)wgs_m), dim3(256), lds, st,
                       reinterpret_cast<__bf16*>(Y), ldy, n, m, p2, kind, lognb);
  } else {
    int cgroups = m >= 12 ? 1 : (m == 8 ? 2 : 4);  // as in the kernel
    while (cgroups > 1 && p2 / 128 < cgroups) cgroups /= 2;
    const size_t lds = ((size_t)m * m + 128 * (size_t)cgroups * m) * 4 + (size_t)m;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(hadamard_cross_kernel<T>), lds))
      return fail(KT_ERR_DEVICE, "the Hadamard factor kernel needs %zu bytes of LDS per workgroup", lds);
    hipLaunchKernelGGL((hadamard_cross_kernel<T>), dim3((unsigned)wgs), dim3(256), lds, st, static_cast<T*>(Y), ldy,
                       n, m, p2, kind);
  }
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Hadamard factor launch failed");
  return KT_OK;
}

extern "C" {

int32_t kt_version(void) { return 100; }

#ifndef KT_BUILD_ID
#define KT_BUILD_ID "unknown"
#endif
const char* kt_build_id(void) { return KT_BUILD_ID; }

const char* kt_last_error(void) { return g_err; }

size_t kt_workspace_bytes(kt_op op, int64_t batch, int64_t n, int64_t d, kt_dtype x_dtype) {
  if (batch < 1 || d < 1 || d % 128 != 0) return 0;
  if (x_dtype != KT_F32 && x_dtype != KT_BF16) return 0;
  switch (op) {
    case KT_OP_LOSS_GRAD:
      if (n < 1) return 0;
      return plan_loss_grad(batch, n, d, x_dtype, false, keep_y_recommended(batch, n, d, x_dtype, false)).total;
    case KT_OP_LOSS_GRAD_RECOMPUTE:
      if (n < 1) return 0;
      return plan_loss_grad(batch, n, d, x_dtype).total;
    case KT_OP_POOLED_LOSS_GRAD:
      if (n < 1) return 0;
      return plan_loss_grad(batch, n, d, x_dtype, true, keep_y_recommended(batch, n, d, x_dtype, true)).total;
    case KT_OP_POOLED_LOSS_GRAD_RECOMPUTE:
      if (n < 1) return 0;
      return plan_loss_grad(batch, n, d, x_dtype, true).total;
    case KT_OP_QUANT_METRICS:
      if (n < 1) return 0;
      {  // R^T and, when the caller does not ask for Y, an fp32 staging slice of it
        int64_t sp, sr;
        stage_slices(batch, n, d, &sp, &sr);
        return round_up(batch * d * d * (x_dtype == KT_F32 ? 4 : 2), 256) + (size_t)sp * sr * d * 4;
      }
    case KT_OP_FUSE_ROTATION:  // n = the other dimension k of the weight
      if (n < 1) return 0;
      return round_up(d * d * 4, 256) + (size_t)n * d * 4;
    case KT_OP_SENSITIVITY:
      return (size_t)kSensBlocks * kSensSteps * 8 + 1024;
    case KT_OP_CAYLEY:
      return plan_cayley(batch, d, cayley_use_split(d)).total;
    case KT_OP_FAKEQUANT:
      if (n < 1) return 0;
      return plan_quant(batch, n, d, x_dtype).total;
    default:
      return 0;
  }
}

kt_status kt_kurtosis_loss_grad(const void* X, int64_t ldx, const void* R, int64_t ldr,
                                int64_t batch, int64_t n, int64_t d, kt_dtype x_dtype,
                                kt_dtype r_dtype, float kappa_target, float* loss, float* row_kurt,
                                float* dR, void* workspace, size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  kt_status s = check_xr(X, ldx, R, ldr, batch, n, d, x_dtype, r_dtype);
  if (s != KT_OK) return s;
  if (!loss) return fail(KT_ERR_INVALID_ARG, "loss must not be null");
  if (!(kappa_target >= 0.f)) return fail(KT_ERR_INVALID_ARG, "kappa_target must be >= 0");
  LossGradPlan p = plan_loss_grad(batch, n, d, x_dtype);
  if (p.fused && workspace_bytes < p.total) {
    // A smaller workspace still serves while the loss partials of one workgroup per problem fit: as many workgroups as there is room for
    // (8 bytes of loss and, from two on, a d x d partial each; the loss partials end at a multiple of 256 bytes).
    const int64_t room = (int64_t)(workspace_bytes / ((size_t)batch * (8 + d * d * 4)));
    const int64_t k = room < 1 ? 1 : room < p.fused_wgs ? room : p.fused_wgs - 1;
    if (k < p.fused_wgs) p = plan_loss_grad(batch, n, d, x_dtype, false, false, k);
    if (k > 1 && workspace_bytes < p.total) p = plan_loss_grad(batch, n, d, x_dtype, false, false, k - 1);
  }
  s = check_ws(workspace, workspace_bytes, p.total);
  if (s != KT_OK) return s;
  if (!p.fused && dR) {  // room for Y: keep it instead of recomputing it (same result)
    const LossGradPlan pk = plan_loss_grad(batch, n, d, x_dtype, false, true);
    if (workspace_bytes >= pk.total) p = pk;
  }
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (p.fused)
    return run_loss_grad_fused(p, X, ldx, R, ldr, r_dtype, batch, n, d, kappa_target, loss, row_kurt, dR,
                               ws, st);
  return p.fp32 ? run_loss_grad_f32(p, static_cast<const float*>(X), ldx, static_cast<const float*>(R), ldr, batch, n, d, kappa_target, loss, row_kurt, dR, ws, st)
                : run_loss_grad_bf16(p, X, ldx, R, ldr, r_dtype, batch, n, d, kappa_target, loss, row_kurt, dR, ws, st);
}

kt_status kt_pooled_kurtosis_loss_grad(const void* X, int64_t ldx, const void* R, int64_t ldr,
                                       int64_t batch, int64_t n, int64_t d, kt_dtype x_dtype,
                                       kt_dtype r_dtype, float kappa_target, float rms_eps, float* loss,
                                       float* kappa, float* dR, void* workspace, size_t workspace_bytes,
                                       void* stream) {
  g_err[0] = 0;
  kt_status s = check_xr(X, ldx, R, ldr, batch, n, d, x_dtype, r_dtype);
  if (s != KT_OK) return s;
  if (!loss) return fail(KT_ERR_INVALID_ARG, "loss must not be null");
  if (!(kappa_target >= 0.f)) return fail(KT_ERR_INVALID_ARG, "kappa_target must be >= 0");
  if (!(rms_eps >= 0.f)) return fail(KT_ERR_INVALID_ARG, "rms_eps must be >= 0");
  LossGradPlan p = plan_loss_grad(batch, n, d, x_dtype, true);
  s = check_ws(workspace, workspace_bytes, p.total);
  if (s != KT_OK) return s;
  if (dR) {
    const LossGradPlan pk = plan_loss_grad(batch, n, d, x_dtype, true, true);
    if (workspace_bytes >= pk.total) p = pk;
  }
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  PooledArgs pa;
  pa.rms_eps = rms_eps; pa.kappa_out = kappa;
  return p.fp32 ? run_loss_grad_f32(p, static_cast<const float*>(X), ldx, static_cast<const float*>(R), ldr, batch, n, d, kappa_target, loss, nullptr, dR, ws, st, &pa)
                : run_loss_grad_bf16(p, X, ldx, R, ldr, r_dtype, batch, n, d, kappa_target, loss, nullptr, dR, ws, st, &pa);
}

kt_status kt_cayley_step(float* R, const float* dR, void* R_lowp, int64_t batch, int64_t d, float lr,
                         float* ortho_err, int32_t* info, void* workspace, size_t workspace_bytes,
                         void* stream) {
  g_err[0] = 0;
  if (!R || !dR) return fail(KT_ERR_INVALID_ARG, "R and dR must not be null");
  if ((reinterpret_cast<uintptr_t>(R) | reinterpret_cast<uintptr_t>(dR)) & 15)
    return fail(KT_ERR_BAD_SHAPE, "R and dR must be 16-byte aligned");
  if (batch < 1 || d < 1) return fail(KT_ERR_INVALID_ARG, "batch and d must be positive");
  if (d % 128 != 0) return fail(KT_ERR_BAD_SHAPE, "d = %lld is not a multiple of 128", (long long)d);
  if (d > 16384 || batch > 65535) return fail(KT_ERR_BAD_SHAPE, "size out of range (d <= 16384, batch <= 65535)");
  if (!(lr == lr) || lr - lr != 0.f) return fail(KT_ERR_INVALID_ARG, "lr must be finite");
  const CayleyPlan p = plan_cayley_in(batch, d, workspace_bytes);
  kt_status s = check_ws(workspace, workspace_bytes, p.total);
  if (s != KT_OK) return s;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  ProfScope prof(4, st);
  if (d == 128)  // whole retraction of a problem inside one workgroup (kt_cayley_d128.h)
    return launch_cayley_d128<false>(R, dR, R_lowp, batch, 0.5f * lr, ortho_err, info, C128Adam{}, st);
  return cayley_run(p, ws, R, dR, R_lowp, batch, d, 0.5f * lr, nullptr, ortho_err, info, st);
}

kt_status kt_cayley_step_static(float* R, const float* dR, void* R_lowp, int64_t batch, int64_t d, float lr,
                                float* ortho_err, int32_t* info, void* stream) {
  g_err[0] = 0;
  if (!R || !dR) return fail(KT_ERR_INVALID_ARG, "R and dR must not be null");
  if (batch < 1 || d < 1) return fail(KT_ERR_INVALID_ARG, "batch and d must be positive");
  if (d % 128 != 0) return fail(KT_ERR_BAD_SHAPE, "d = %lld is not a multiple of 128", (long long)d);
  if (d > 16384 || batch > 65535) return fail(KT_ERR_BAD_SHAPE, "size out of range (d <= 16384, batch <= 65535)");
  if (!(lr == lr) || lr - lr != 0.f) return fail(KT_ERR_INVALID_ARG, "lr must be finite");
  const size_t need = plan_cayley_in(batch, d, kStaticScratchBytes).total;
  if (need > kStaticScratchBytes)
    return fail(KT_ERR_NOT_SUPPORTED,
                "batch = %lld, d = %lld needs %zu bytes of scratch; the library's static scratch holds %zu "
                "(use kt_cayley_step with a workspace)", (long long)batch, (long long)d, need, kStaticScratchBytes);
  void* ws = static_scratch_of_current_device();
  if (!ws) return KT_ERR_DEVICE;
  // same checks, plan and launches as the workspace form; the kernels ahead of the iterations clear their counters,
  // so whatever the previous call left in the array does not matter
  return kt_cayley_step(R, dR, R_lowp, batch, d, lr, ortho_err, info, ws, kStaticScratchBytes, stream);
}

kt_status kt_cayley_adam_step(float* R, const float* dR, float* M, float* v, int64_t step, void* R_lowp,
                              int64_t batch, int64_t d, float lr, float beta1, float beta2, float eps, float q,
                              float* ortho_err, int32_t* info, float* scalars, void* workspace,
                              size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  if (!R || !dR || !M || !v) return fail(KT_ERR_INVALID_ARG, "R, dR, M and v must not be null");
  if ((reinterpret_cast<uintptr_t>(R) | reinterpret_cast<uintptr_t>(dR) | reinterpret_cast<uintptr_t>(M)) & 15)
    return fail(KT_ERR_BAD_SHAPE, "R, dR and M must be 16-byte aligned");
  if (batch < 1 || d < 1) return fail(KT_ERR_INVALID_ARG, "batch and d must be positive");
  if (d % 128 != 0) return fail(KT_ERR_BAD_SHAPE, "d = %lld is not a multiple of 128", (long long)d);
  if (d > 16384 || batch > 65535) return fail(KT_ERR_BAD_SHAPE, "size out of range (d <= 16384, batch <= 65535)");
  if (step < 1) return fail(KT_ERR_INVALID_ARG, "step counts from 1");
  if (!(lr == lr) || lr - lr != 0.f) return fail(KT_ERR_INVALID_ARG, "lr must be finite");
  if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f))
    return fail(KT_ERR_INVALID_ARG, "beta1 and beta2 must lie in [0, 1)");
  if (!(eps >= 0.f) || !(q > 0.f)) return fail(KT_ERR_INVALID_ARG, "eps must be >= 0 and q > 0");
  const CayleyPlan p = plan_cayley_in(batch, d, workspace_bytes);
  kt_status s = check_ws(workspace, workspace_bytes, p.total);
  if (s != KT_OK) return s;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  ProfScope prof(4, st);
  const double c1 = 1.0 - pow((double)beta1, (double)step), c2 = 1.0 - pow((double)beta2, (double)step);
  if (d == 128) {
    C128Adam ad;
    ad.M = M; ad.v = v; ad.scalars_out = scalars; ad.lr = lr; ad.beta1 = beta1; ad.beta2 = beta2;
    ad.eps = eps; ad.q = q; ad.c1 = c1; ad.c2 = c2;
    return launch_cayley_d128<true>(R, dR, R_lowp, batch, 0.5f, ortho_err, info, ad, st);
  }
  AdamArgs a;
  a.M = M; a.lr = lr; a.q = q; a.eps = eps; a.scalars_out = scalars;
  a.scal = reinterpret_cast<float*>(ws + p.o_scal);
  a.sq_part = reinterpret_cast<double*>(ws + p.o_sq);
  double* g2_part = reinterpret_cast<double*>(ws + p.o_g2);
  // (with 256 partial sums a problem the SplitScales at the end of their room are clear of them: split3_kernel reads the ones and writes the others)
  const int blocks = p.split ? 256 : p.g2_blocks;
  a.first = AdamScalars{g2_part, blocks, v, beta2, c1, c2, eps, a.scal};
  if (p.split) {
    hipLaunchKernelGGL(adam_moment_kernel<true>, dim3((unsigned)blocks, (unsigned)batch), dim3(256), 0, st, M, dR, d * d, beta1, g2_part, R,
                       reinterpret_cast<unsigned*>(ws + p.o_m));
  } else {
    hipLaunchKernelGGL(adam_moment_kernel<false>, dim3((unsigned)blocks, (unsigned)batch), dim3(256), 0, st, M, dR, d * d, beta1, g2_part,
                       (const float*)nullptr, (unsigned*)nullptr);
    hipLaunchKernelGGL(adam_scalars1_kernel, dim3((unsigned)batch), dim3(256), 0, st, a.first);
  }
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "Cayley Adam moment launch failed");
  // P = M1 R^T, S = (P - P^T)/2 (= r W for orthogonal R), then the transform with c = alpha/(2r)
  return cayley_run(p, ws, R, M, R_lowp, batch, d, 0.5f, &a, ortho_err, info, st);
}

kt_status kt_rotate_fakequant_int4(const void* X, int64_t ldx, const void* R, int64_t ldr,
                                   int64_t batch, int64_t n, int64_t d, kt_dtype x_dtype,
                                   kt_dtype r_dtype, float clip_ratio, const float* scales_in,
                                   float* scales_out, int8_t* codes, float* err, void* workspace,
                                   size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  kt_status s = check_xr(X, ldx, R, ldr, batch, n, d, x_dtype, r_dtype);
  if (s != KT_OK) return s;
  if (!(clip_ratio > 0.f && clip_ratio <= 1.f))
    return fail(KT_ERR_INVALID_ARG, "clip_ratio must be in (0, 1]");
  if (!scales_out && !codes && !err) return fail(KT_ERR_INVALID_ARG, "no output requested");
  if (reinterpret_cast<uintptr_t>(codes) & 15) return fail(KT_ERR_BAD_SHAPE, "codes must be 16-byte aligned");
  const QuantPlan p = plan_quant(batch, n, d, x_dtype);
  s = check_ws(workspace, workspace_bytes, p.total);
  if (s != KT_OK) return s;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  ProfScope prof(5, st);
  if (!p.fp32 && d == 128) {  // one pass over X (kt_fused_d128.h)
    hipLaunchKernelGGL(quant_d128_kernel, dim3((unsigned)quant_d128_wgs(batch, n), (unsigned)batch), dim3(256), 0, st,
                       static_cast<const bf16*>(X), ldx, n * ldx, R, ldr, r_dtype == KT_BF16 ? 1 : 0, (int)n, clip_ratio, scales_in, scales_out, codes,
                       reinterpret_cast<float2*>(err));
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "d=128 fake-quant launch failed");
    return KT_OK;
  }
  if (p.fp32)
    return run_quant<float, TF, TF>(p, X, ldx, R, ldr, r_dtype, batch, n, d, clip_ratio, scales_in,
                                    scales_out, codes, err, ws, st);
  if (d % 256 == 0)
    return run_quant<bf16, TB_BIG, TB_BIG>(p, X, ldx, R, ldr, r_dtype, batch, n, d, clip_ratio, scales_in,
                                           scales_out, codes, err, ws, st);
  return run_quant<bf16, TB_M128, TB_N128>(p, X, ldx, R, ldr, r_dtype, batch, n, d, clip_ratio, scales_in,
                                           scales_out, codes, err, ws, st);
}

kt_status kt_rotate_quant_metrics(const void* X, int64_t ldx, const void* R, int64_t ldr, int64_t batch,
                                  int64_t n, int64_t d, kt_dtype x_dtype, kt_dtype r_dtype, float quantile,
                                  float* Y, float* amax, float* threshold, float* err_sym, float* err_asym,
                                  int64_t* success, void* workspace, size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  kt_status s = check_xr(X, ldx, R, ldr, batch, n, d, x_dtype, r_dtype);
  if (s != KT_OK) return s;
  if (!(quantile > 0.f && quantile <= 1.f)) return fail(KT_ERR_INVALID_ARG, "quantile must be in (0, 1]");
  if (d > 8192) return fail(KT_ERR_NOT_SUPPORTED, "quantisation metrics keep a token row in registers: d <= 8192");
  const bool fp32 = x_dtype == KT_F32;
  const size_t rt_bytes = (size_t)round_up(batch * d * d * (fp32 ? 4 : 2), 256);
  // With Y wanted the whole rotation is one launch pair into the caller's buffer; without it Y passes through
  // a bounded staging slice, some problems or some token rows of one problem at a time.
  int64_t sp = batch, sr = n;
  if (!Y) stage_slices(batch, n, d, &sp, &sr);
  const size_t need = rt_bytes + (Y ? 0 : (size_t)sp * sr * d * 4);
  s = check_ws(workspace, workspace_bytes, need);
  if (s != KT_OK) return s;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* Yb = Y ? Y : reinterpret_cast<float*>(ws + rt_bytes);
  ProfScope prof(5, st);
  // Y = X R, token-major (tokens on the rows of the GEMM): Y never feeds another GEMM here, the
  // row kernel wants whole token rows
  auto rotate = [&](auto t_tag, auto tile_tag) -> kt_status {
    using T = decltype(t_tag);
    using TL = decltype(tile_tag);
    T* RT = reinterpret_cast<T*>(ws);
    const T* Xp = static_cast<const T*>(X);
    const bool skinny = sp == batch && skinny_ok(x_dtype, R, ldr, r_dtype, n);
    const bool in_place = sizeof(T) == 4 && f32_in_place(R, ldr) && !(Y && overlap(Y, batch * n * d * 4, R, ((batch * d - 1) * ldr + d) * 4));
    if (!skinny && !in_place && !prep_rt<T>(R, ldr, r_dtype, RT, batch, d, st)) return fail(KT_ERR_DEVICE, "prep_rt launch failed");
    const T* Rg = in_place ? static_cast<const T*>(R) : RT;
    if (success) {
      hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<unsigned*>(success),
                         2 * batch, 0u);
    }
    for (int64_t b0 = 0; b0 < batch; b0 += sp) {
      const int64_t nb = batch - b0 < sp ? batch - b0 : sp;
      for (int64_t t0 = 0; t0 < n; t0 += sr) {
        const int64_t nt = n - t0 < sr ? n - t0 : sr, row0 = b0 * n + t0;
        bool ok;
        if (skinny) {
          const bf16* Xb = static_cast<const bf16*>(X);
          ok = r_dtype == KT_F32 ? launch_skinny(Xb, ldx, static_cast<const float*>(R), ldr, batch, n, d, ws, rt_bytes, Yb, st)
                                 : launch_skinny(Xb, ldx, static_cast<const bf16*>(R), ldr, batch, n, d, ws, rt_bytes, Yb, st);
        } else {
          ok = launch_rows_gemm<T, TL>(Xp + row0 * ldx, ldx, n * ldx, Rg + b0 * (in_place ? d * ldr : d * d), ldr, in_place, nb, nt, d, Yb, nt * d, st);
        }
        if (!ok) return fail(KT_ERR_DEVICE, "rotation GEMM launch failed");
        // the row in 4 / 8 / 16 / 32 float4 registers per lane; rows that fill them exactly skip every bounds test
        auto rows_kernel = d == 1024   ? quant_metrics_row_kernel<T, 4, true>
                           : d < 1024  ? quant_metrics_row_kernel<T, 4, false>
                           : d == 2048 ? quant_metrics_row_kernel<T, 8, true>
                           : d < 2048  ? quant_metrics_row_kernel<T, 8, false>
                           : d == 4096 ? quant_metrics_row_kernel<T, 16, true>
                           : d < 4096  ? quant_metrics_row_kernel<T, 16, false>
                           : d == 8192 ? quant_metrics_row_kernel<T, 32, true>
                                       : quant_metrics_row_kernel<T, 32, false>;
        // us, 32768 rows, 8 / 16 workgroups a CU: d = 256 71 / 81, 1024 136 / 140, 2048 347 / 342, 4096 987 / 970
        const int64_t most = ceil_div((d <= 1024 ? 8 : 16) * kNumCUs, nb), row_wgs = ceil_div(nt, 4) < most ? ceil_div(nt, 4) : most;
        hipLaunchKernelGGL(rows_kernel, dim3((unsigned)row_wgs, (unsigned)nb), dim3(256), 0, st, Yb,
                           Xp + row0 * ldx, ldx, n * ldx, (int)nt, (int)d, (double)quantile,
                           amax ? amax + 2 * row0 : nullptr, threshold ? threshold + row0 : nullptr,
                           err_sym ? err_sym + 2 * row0 : nullptr, err_asym ? err_asym + 2 * row0 : nullptr,
                           success ? reinterpret_cast<unsigned long long*>(success) + b0 : nullptr);
        if (!launch_ok()) return fail(KT_ERR_DEVICE, "metrics kernel launch failed");
      }
    }
    return KT_OK;
  };
  if (fp32) return rotate(float{}, TF{});
  if (d % 256 == 0) return rotate(bf16{}, TB_BIG{});
  return rotate(bf16{}, TB_N128{});
}

kt_status kt_hadamard_rows(const void* X, int64_t ldx, void* Y, int64_t ldy, const int8_t* signs, int64_t n,
                           int64_t d, kt_dtype dtype, void* stream) {
  g_err[0] = 0;
  if (!X || !Y) return fail(KT_ERR_INVALID_ARG, "X and Y must not be null");
  if (n < 1) return fail(KT_ERR_INVALID_ARG, "n must be positive");
  if (dtype != KT_F32 && dtype != KT_BF16) return fail(KT_ERR_BAD_DTYPE, "dtype must be KT_F32 or KT_BF16");
  int m = 0, p2 = 0, kind = 0;
  if (d < 128 || d > 524288 || !hadamard_split(d, &m, &p2, &kind) || p2 < 128 || p2 > 4096 || m > 128)
    return fail(KT_ERR_BAD_SHAPE,
                "d = %lld: the Hadamard transform here needs d = m 2^k with 128 <= 2^k <= 4096 and m = 1, a power "
                "of two or a Paley order (q + 1 or 2 (q + 1), q prime) up to 128",
                (long long)d);
  const int64_t vec = dtype == KT_F32 ? 4 : 8;
  if (ldx < d || ldy < d || ldx % vec != 0 || ldy % vec != 0)
    return fail(KT_ERR_BAD_SHAPE, "ldx / ldy must be >= d and keep rows 16-byte aligned");
  if ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y)) & 15)
    return fail(KT_ERR_BAD_SHAPE, "X and Y must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  ProfScope prof(5, st);
  if (dtype == KT_F32) return run_hadamard<float>(X, ldx, Y, ldy, signs, n, d, m, p2, kind, st);
  return run_hadamard<bf16>(X, ldx, Y, ldy, signs, n, d, m, p2, kind, st);
}

kt_status kt_fuse_rotation(const float* W, int64_t ldw, const float* R, int64_t ldr, float* Wout, int64_t ldo,
                           int64_t k, int64_t d, int32_t side, void* workspace, size_t workspace_bytes,
                           void* stream) {
  g_err[0] = 0;
  if (!W || !R || !Wout) return fail(KT_ERR_INVALID_ARG, "W, R and Wout must not be null");
  if (k < 1 || d < 1) return fail(KT_ERR_INVALID_ARG, "k and d must be positive");
  if (side != 0 && side != 1) return fail(KT_ERR_INVALID_ARG, "side must be 0 (W R) or 1 (R^T W)");
  if (d % 128 != 0 || d > 16384) return fail(KT_ERR_BAD_SHAPE, "d = %lld is not a multiple of 128 (<= 16384)", (long long)d);
  if (k > (int64_t(1) << 22)) return fail(KT_ERR_BAD_SHAPE, "k out of range");
  const int64_t wcols = side == 0 ? d : k;
  if (ldw < wcols || ldo < wcols || ldr < d || ldw % 4 != 0 || ldo % 4 != 0 || ldr % 4 != 0)
    return fail(KT_ERR_BAD_SHAPE, "leading dimensions must cover the rows and keep them 16-byte aligned");
  if (side == 1 && k % 4 != 0) return fail(KT_ERR_BAD_SHAPE, "k must be a multiple of 4 for side 1");
  const size_t rt_bytes = (size_t)round_up(d * d * 4, 256);
  kt_status s = check_ws(workspace, workspace_bytes, rt_bytes + (side == 1 ? (size_t)k * d * 4 : 0));
  if (s != KT_OK) return s;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  // C [M][N] = A B^T, contraction over d; 64 x 64 tiles while 128 x 128 ones would leave CUs idle.  R and (side 1) W are read as
  // they lie where their rows are 16-byte aligned and the result does not go over them, transposed into the workspace first where not.
  ProfScope prof(5, st);
  const size_t out_bytes = ((side == 0 ? k : d) - 1) * ldo * 4 + wcols * 4;
  const bool r_here = f32_in_place(R, ldr) && !overlap(Wout, out_bytes, R, ((d - 1) * ldr + d) * 4);
  const bool w_here = f32_in_place(W, ldw) && !overlap(Wout, out_bytes, W, ((d - 1) * ldw + wcols) * 4);
  float* RT = reinterpret_cast<float*>(ws);
  if (!r_here && !prep_rt<float>(R, ldr, KT_F32, RT, 1, d, st)) return fail(KT_ERR_DEVICE, "prep_rt launch failed");
  auto product = [&](auto atn_c, auto btn_c, const float* A, int64_t lda, int64_t M, const float* B, int64_t ldb, int64_t N) -> bool {
    auto go = [&](auto tile_tag) -> bool {
      using TL = decltype(tile_tag);
      EpiStore<TL> e;
      e.C = Wout; e.ldc = ldo; e.batch_stride = 0; e.split_stride = 0; e.M = (int)M; e.N = (int)N;
      return launch_gemm<TL, EpiStore<TL>, decltype(atn_c)::value, decltype(btn_c)::value>(A, lda, 0, (int)M, B, ldb, 0, (int)N, d, 0, 1, e, st,
                                                                                          0, 0, (int)d);
    };
    return with_f32_tile(M, N, 1, go);
  };
  const std::true_type yes;
  const std::false_type no;
  if (side == 0) {  // Wout [k][d] = W R
    if (!(r_here ? product(no, yes, W, ldw, k, R, ldr, d) : product(no, no, W, ldw, k, RT, d, d)))
      return fail(KT_ERR_DEVICE, "fusion GEMM launch failed");
  } else {          // Wout [d][k] = R^T W
    float* Wt = reinterpret_cast<float*>(ws + rt_bytes);
    if (!w_here) {
      hipLaunchKernelGGL(transpose_f32_kernel, dim3((unsigned)ceil_div(k, 32), (unsigned)ceil_div(d, 32)), dim3(256),
                         0, st, W, ldw, Wt, d, (int)d, (int)k);
      if (!launch_ok()) return fail(KT_ERR_DEVICE, "weight transpose launch failed");
    }
    if (!(r_here && w_here ? product(yes, yes, R, ldr, d, W, ldw, k)
          : r_here         ? product(yes, no, R, ldr, d, Wt, d, k)
          : w_here         ? product(no, yes, RT, d, d, W, ldw, k)
                           : product(no, no, RT, d, d, Wt, d, k)))
      return fail(KT_ERR_DEVICE, "fusion GEMM launch failed");
  }
  return KT_OK;
}

kt_status kt_quant_sensitivity(const float* Y, int64_t count, int32_t bits, const float* alphas, int32_t n_alpha,
                               float* out, float* gamma, void* workspace, size_t workspace_bytes, void* stream) {
  g_err[0] = 0;
  if (!Y || !out) return fail(KT_ERR_INVALID_ARG, "Y and out must not be null");
  if (count < 1) return fail(KT_ERR_INVALID_ARG, "count must be positive");
  if (bits < 2 || bits > 8) return fail(KT_ERR_INVALID_ARG, "bits must be in [2, 8]");
  if (n_alpha < 0 || n_alpha > kSensSteps - 1) return fail(KT_ERR_INVALID_ARG, "at most 31 step fractions");
  if (n_alpha > 0 && (!alphas || !gamma)) return fail(KT_ERR_INVALID_ARG, "alphas and gamma must not be null");
  const size_t need = (size_t)kSensBlocks * kSensSteps * 8 + 1024;
  kt_status s = check_ws(workspace, workspace_bytes, need);
  if (s != KT_OK) return s;
  char* ws = static_cast<char*>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  double* part = reinterpret_cast<double*>(ws);
  double* dst = reinterpret_cast<double*>(ws + (size_t)kSensBlocks * kSensSteps * 8);
  float* stt = reinterpret_cast<float*>(ws + (size_t)kSensBlocks * kSensSteps * 8 + 64);
  const float L = (float)((1 << (bits - 1)) - 1);
  const int nblocks = (int)(ceil_div(count, 256) < kSensBlocks ? ceil_div(count, 256) : kSensBlocks);
  ProfScope prof(5, st);
  hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<unsigned*>(stt), 64, 0u);
  hipLaunchKernelGGL(sens_amax_kernel, dim3(nblocks), dim3(256), 0, st, Y, count,
                     reinterpret_cast<unsigned*>(stt + 35));
  hipLaunchKernelGGL(sens_select_kernel, dim3(1), dim3(256), 0, st, part, nblocks, 0, count, -1, L, stt, dst, alphas,
                     (int)n_alpha, out, gamma);
  if (!launch_ok()) return fail(KT_ERR_DEVICE, "sensitivity set-up launch failed");
  for (int round = 0; round < 4; ++round) {
    const int ns = round < 3 ? kSensSteps : 1 + n_alpha;
    hipLaunchKernelGGL(sens_sweep_kernel, dim3(nblocks, (unsigned)ceil_div(ns, kSensPerBlock)), dim3(256), 0, st, Y, count, stt,
                       ns, L, part);
    hipLaunchKernelGGL(sens_select_kernel, dim3(1), dim3(256), 0, st, part, nblocks, ns, count, round, L, stt, dst,
                       alphas, (int)n_alpha, out, gamma);
    if (!launch_ok()) return fail(KT_ERR_DEVICE, "sensitivity sweep launch failed");
  }
  return KT_OK;
}

#ifdef KT_PHASE_STAMPS
// Developer build only: arm the phase stamps (the next kStampSlots GEMM launches record into slots 0, 1, ...) and
// read them back (synchronises the device).
void kt_debug_stamps_arm(void) { g_stamp_next = 0; }
int kt_debug_stamps_read(void* host_dst, size_t bytes) {
  g_stamp_next = -1;
  if (hipDeviceSynchronize() != hipSuccess) return -1;
  const size_t all = sizeof(unsigned long long) * kStampSlots * kStampWgs * kStampWords;
  return hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(g_phase_stamps), bytes < all ? bytes : all) == hipSuccess ? 0 : -1;
}
#endif

kt_status kt_profile_reset(void) {
  g_prof_used.store(0);
  return KT_OK;
}

kt_status kt_profile_enable(int32_t max_records) {
  g_err[0] = 0;
  if (max_records < 0) return fail(KT_ERR_INVALID_ARG, "max_records must be >= 0");
  for (int i = 0; i < g_prof_cap; ++i) {
    (void)hipEventDestroy(g_prof[i].start);
    (void)hipEventDestroy(g_prof[i].stop);
  }
  delete[] g_prof;
  g_prof = nullptr;
  g_prof_cap = 0;
  g_prof_used.store(0);
  if (max_records == 0) return KT_OK;
  g_prof = new (std::nothrow) ProfRecord[max_records];  // no exception may cross the C boundary
  if (!g_prof) return fail(KT_ERR_INVALID_ARG, "cannot hold %d profile records", (int)max_records);
  for (int i = 0; i < max_records; ++i) {
    if (hipEventCreate(&g_prof[i].start) != hipSuccess || hipEventCreate(&g_prof[i].stop) != hipSuccess)
      return fail(KT_ERR_DEVICE, "hipEventCreate failed");
    g_prof_cap = i + 1;
  }
  return KT_OK;
}

kt_status kt_profile_read(int32_t kernel_id, double* total_ms, int32_t* launches) {
  g_err[0] = 0;
  if (!total_ms || !launches) return fail(KT_ERR_INVALID_ARG, "outputs must not be null");
  double tot = 0.0;
  int cnt = 0;
  const int used = g_prof_used.load() < g_prof_cap ? g_prof_used.load() : g_prof_cap;
  for (int i = 0; i < used; ++i) {
    if (g_prof[i].id != kernel_id) continue;
    if (hipEventSynchronize(g_prof[i].stop) != hipSuccess) return fail(KT_ERR_DEVICE, "event sync failed");
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, g_prof[i].start, g_prof[i].stop) != hipSuccess)
      return fail(KT_ERR_DEVICE, "event elapsed failed");
    tot += ms;
    ++cnt;
  }
  *total_ms = tot;
  *launches = cnt;
  return KT_OK;
}

}  // extern "C"
