// kt_gemm.h -- MFMA GEMM core for gfx950 shared by every contraction on the path.
//
// One device-side main loop computes a BM x BN tile of  C = A * B^T  where both
// operands are stored with the contraction index contiguous ("NT" form):
//   A [M][lda], B [N][ldb], C[m][n] = sum_k A[m][k] * B[n][k].
// An operand may also come with K as its row index (ATN, BTN of gemm_mainloop): activations
// X [token][feature] in X^T G, fp32 R, W and dL/dY as they lie in memory.  The bf16 path keeps
// R^T (rows are output features) and dL/dY token-minor, which are NT operands.
//
// Tiling: 64-wide wavefronts, each wave owns WTM x WTN of the tile as a grid of
// 16x16 MFMA blocks (v_mfma_f32_16x16x32_bf16, or 4 x v_mfma_f32_16x16x4_f32 per
// 16-byte fragment on the fp32 path).  In the accumulator layout of these
// instructions a lane owns ONE column n (= lane & 15) and 4 consecutive rows
// m = 4*(lane>>4) + r, r = 0..3.  Callers put the index they reduce over (the hidden
// dimension of a token row) on m, so row statistics accumulate in registers with no
// cross-lane traffic until one final exchange between the four lane quarters; callers
// that store C row-major take the operands in swapped order (SWAP) and own four
// consecutive columns of one row instead.
//
// Why 16x16x32 and not 32x32x16: both issue at the same 1024 flop per cycle and SIMD, but
// the large products here run at the board's power limit, and per flop the 16x16 form reads
// and writes half as many accumulator words.  Matrix instructions alone, random bf16
// operands, 256 accumulator registers per lane, whole chip: 2075 TFLOP/s against 1800 (all-zero
// operands: 2475 for both, the 2.4 GHz clock).
//
// LDS: stages of 128 bytes of K (a slab) per row, two of the A operand's rows and three of the B
// operand's, filled straight from global memory (buffer_load ... lds); 16-byte chunks are
// XOR-swizzled with the row pair so that the MFMA fragment reads are bank-conflict free.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace kt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int kRowBytes = 128;  // bytes of K per LDS tile row: a slab, the unit in which K is counted and blocked
constexpr int kStagesA = 2, kStagesB = 3;

template <typename T>
struct Mma;

// One 16x16 block, one 16-byte fragment of each operand per lane: lane l holds row l & 15 and the
// 16 bytes of K at chunk l >> 4 (bf16: K = 32 in one instruction; fp32: K = 16 in four, each taking
// one of the four values; which value of K is multiplied in which instruction does not matter as
// long as both operands agree).
//
// The bf16 instruction is inline assembly so that its accumulators stay in accumulation registers: the 64
// blocks of a 128 x 128 wave tile are all 256 of them, and left to the register allocator (builtin) the
// loop body moved ~950 accumulators between the two files and spilled 130-185 registers.  The compiler
// does not know it is a matrix instruction: accumulators are read by anything else only behind
// settle(), and the fragments are only ever written by LDS reads.
template <>
struct Mma<__bf16> {
  static __device__ __forceinline__ void run(const intx4& a, const intx4& b, floatx4& c) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  }
};

template <>
struct Mma<_Float16> {
  static __device__ __forceinline__ void run(const intx4& a, const intx4& b, floatx4& c) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  }
};

template <>
struct Mma<float> {
  static __device__ __forceinline__ void run(const intx4& a, const intx4& b, floatx4& c) {
    const floatx4 fa = __builtin_bit_cast(floatx4, a);
    const floatx4 fb = __builtin_bit_cast(floatx4, b);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0], fb[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[1], fb[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[2], fb[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[3], fb[3], c, 0, 0, 0);
  }
};


// Tile shape: BM x BN per workgroup, WGM x WGN waves.
template <typename T_, int BM_, int BN_, int WGM_, int WGN_>
struct Tile {
  using T = T_;
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_;
  static constexpr int NT = WGM * WGN * 64;
  static constexpr int WTM = BM / WGM, WTN = BN / WGN;
  static constexpr int MB = WTM / 16, NB = WTN / 16;
  static constexpr int BK = kRowBytes / (int)sizeof(T);  // elements of K per slab
  static constexpr int A_BYTES = BM * kRowBytes, B_BYTES = BN * kRowBytes;
  static constexpr int LDS_BYTES = kStagesA * A_BYTES + kStagesB * B_BYTES;
  static constexpr int A_LD = A_BYTES / (16 * NT);  // 16-byte loads per thread per stage
  static constexpr int B_LD = B_BYTES / (16 * NT);
  static_assert(BM % (16 * WGM) == 0 && BN % (16 * WGN) == 0, "wave tile must be 16-blocked");
  static_assert(A_BYTES % (16 * NT) == 0 && B_BYTES % (16 * NT) == 0, "loads must divide evenly");
};

// Holds every use of the accumulators behind this point (after the matrix instructions: 16 wait states, more than
// the 8-pass forms need before another instruction type reads their result).  One wait for all of them: one for every pair
// of blocks, twice a tile, was 2 us of a call with few slabs of K (fake-quant with given scales, d = 256, 2048 tokens: 24.2 -> 22.6 us).
template <class TL>
__device__ __forceinline__ void settle_all(floatx4 (&acc)[TL::MB][TL::NB]) {
  if constexpr (sizeof(typename TL::T) == 2) {
    asm volatile("s_nop 15" ::: "memory");
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) asm volatile("" : "+a"(acc[mb][nb]));  // (volatile statements stay in order)
  }
}

// LDS has 64 banks of 4 bytes: two 128-byte tile rows share one bank window, and a
// 16-byte access is served 16 lanes at a time.  XOR-ing the chunk index with (row >> 1)
// makes 16 consecutive rows at the same logical chunk hit 16 distinct 16-byte slots of
// the 256-byte window (measured: 194 B/clk/CU, against 122 with a plain row & 7 key).
__device__ __forceinline__ int swizzle_key(int row) { return (row >> 1) & 7; }

// Two transposing 8-byte LDS reads (ds_read_b64_tr_b16) -> one MFMA operand: 8 values along K for
// this lane's row, taken from a tile that is stored with K as the ROW index.  In a group of 16
// lanes, lane r supplies the address of 4 consecutive columns of tile row k0 + r/4 starting at
// column c0 + 4*(r%4); lane L of the group receives column c0 + L of rows k0..k0+3.
// `addr_lo` / `addr_hi` are this lane's addresses for rows +0..3 / +4..7.
typedef short shortx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ intx4 read_tr_operand(const char* lds, int addr_lo, int addr_hi) {
  typedef __attribute__((address_space(3))) shortx4* lds_ptr;
  const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lds + addr_lo));
  const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lds + addr_hi));
  typedef short shortx8 __attribute__((ext_vector_type(8)));
  const shortx8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(intx4, v);
}

// threadIdx.x, AGAIN: not known to be the same on every call.  In a kernel that walks tiles, what follows from it (lane constants of the
// main loop and of the epilogue) is then made anew for each tile instead of being kept, or spilled, across the other's registers.
template <bool AGAIN>
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  if constexpr (AGAIN) asm volatile("" : "+v"(t));
  return t;
}

// Geometry of one accumulator element, shared by every epilogue.
template <class TL>
struct Frag {
  int lane, l16, q, wm, wn;
  __device__ __forceinline__ explicit Frag(int t = threadIdx.x) {
    const int wave = t >> 6;
    lane = t & 63;
    l16 = lane & 15;
    q = lane >> 4;
    wm = wave / TL::WGN;
    wn = wave % TL::WGN;
  }
  // offsets inside the workgroup tile of accumulator register r of block (mb, nb): row m_of, column n_of ...
  __device__ __forceinline__ int m_of(int mb, int r) const { return m_block(mb) + 4 * q + r; }
  __device__ __forceinline__ int m_block(int mb) const { return wm * TL::WTM + mb * 16; }
  __device__ __forceinline__ int n_of(int nb) const { return wn * TL::WTN + nb * 16 + l16; }
  // ... and with the operands swapped (SWAP): row m_row, columns n_quad .. n_quad + 3 in r = 0..3
  __device__ __forceinline__ int m_row(int mb) const { return m_block(mb) + l16; }
  __device__ __forceinline__ int n_quad(int nb) const { return wn * TL::WTN + nb * 16 + 4 * q; }
};

template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
// Calls f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), fully unrolled.
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Wait for this wave's outstanding LDS operations only (vmcnt and expcnt left at their
// maxima), then meet the other waves.  A full __syncthreads() would also drain the
// global loads that are deliberately kept in flight across the barrier.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Launch description of one batched NT GEMM.
struct GemmShape {
  const void* A;
  const void* B;
  int64_t lda, ldb;
  int64_t batch_stride_a, batch_stride_b;  // elements
  int M, N;
  int tiles_m, tiles_n;
  int split_k;       // number of K splits (>= 1)
  int slabs_total;   // K / BK
  int slabs_per_split;
  int tiles_total;   // tiles_m * tiles_n * split_k
  int grid_padded;   // tiles_total rounded up to a multiple of 8
  int slabs_per_block;             // K blocking of the rows of B, the slabs of a term with fp16 (see gemm_mainloop)
  int64_t block_bytes_b;
  int k_valid;                     // ATN: rows of A that exist (K may be padded beyond them)
#ifdef KT_PHASE_STAMPS
  int stamp_slot;                  // developer build only: which launch record the stamps go to
#endif
};

#ifdef KT_PHASE_STAMPS
// Developer build (-DKT_PHASE_STAMPS, never the shipped library): wave 0 of every workgroup records the
// shader-clock counter at kernel entry, after the prologue, after the main loop and after the epilogue,
// plus the constant-rate (100 MHz) counter at entry and exit and the hardware id of its CU, so that a
// launch can be broken down into phases and the clock the chip actually held can be read off.
constexpr int kStampSlots = 8, kStampWgs = 16384, kStampWords = 8;
__device__ unsigned long long g_phase_stamps[kStampSlots * kStampWgs * kStampWords];
__device__ __forceinline__ void phase_stamp(const GemmShape& g, int word, bool wall = false) {
  if (threadIdx.x != 0 || g.stamp_slot < 0) return;
  const size_t wg = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (wg >= (size_t)kStampWgs) return;
  unsigned long long* rec = g_phase_stamps + ((size_t)g.stamp_slot * kStampWgs + wg) * kStampWords;
  rec[word] = wall ? __builtin_amdgcn_s_memrealtime() : __builtin_readcyclecounter();
}
#define KT_STAMP(g, word) phase_stamp(g, word)
#define KT_STAMP_WALL(g, word) phase_stamp(g, word, true)
#define KT_STAMP_PARAM , const GemmShape* stamp_g = nullptr
#define KT_STAMP_ARG , &g
#define KT_STAMP_LOOP_START() do { if (stamp_g) phase_stamp(*stamp_g, 1); } while (0)
#else
#define KT_STAMP(g, word)
#define KT_STAMP_WALL(g, word)
#define KT_STAMP_PARAM
#define KT_STAMP_ARG
#define KT_STAMP_LOOP_START()
#endif

// 16 bytes per lane from global memory straight into LDS: lane l lands at LDS byte lds_base + OFF + 16 l (lds_base
// wave-uniform).  Assembly, so that the compiler does not tie the LDS reads to these loads with a full
// wait: the waits are placed by hand (vmcnt, in issue order).
typedef int sgprx4 __attribute__((ext_vector_type(4)));
template <int OFF>
__device__ __forceinline__ void buffer_to_lds_16(uint32_t voffset, const sgprx4& rsrc, unsigned lds_base) {
  asm volatile("s_add_u32 m0, %1, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds"
               :: "v"(voffset), "s"(lds_base), "s"(rsrc), "n"(OFF)
               : "memory", "scc", "m0");
}
// Raw buffer over everything from `base` on (offsets are unsigned 32-bit, checked by the host).  The loads are hidden from the
// compiler, and a vector instruction that writes a scalar register (v_readfirstlane) has to be five issue slots old before
// a buffer instruction reads it: the descriptor is in scalar registers from here on, and the caller sees to the slots.
__device__ __forceinline__ sgprx4 raw_buffer(const char* base) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  sgprx4 r = {(int)(uint32_t)p, (int)(uint32_t)((p >> 32) & 0xffff), -1, 0x00027000};
  asm volatile("" : "+s"(r));
  return r;
}
__device__ __forceinline__ void raw_buffer_wait() { asm volatile("s_nop 4" ::: "memory"); }

// Waits until at most N vector-memory operations of this wave are in flight (LDS operations: none), then
// meets the other waves.
template <int N>
__device__ __forceinline__ void stage_barrier() {
  static_assert(N < 64, "the counter has six bits");
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x70);  // vmcnt(N) expcnt(7) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Slot of one step (0 .. MB NB - 1) behind which LDS read r of the next step's fragments is issued: the B fragments
// first (r < NB), then A fragment i = r - NB, which must wait for the last MFMA that uses the old one.
template <int MB, int NB>
constexpr int fragment_read_slot(int r, int base, int spacing) {
  if (r < NB) return base + r * spacing;
  const int i = r - NB;
  int slot = base + NB * spacing;
  for (int k = 0; k <= i; ++k) {
    const int free_at = NB * (k + 1) - 1;
    if (slot < free_at) slot = free_at;
    if (k < i) slot += spacing;
  }
  return slot < MB * NB ? slot : MB * NB - 1;
}

// Main loop.  Rows of A beyond M (and of B beyond N) are read from the last valid
// row, so every load stays inside the operand; the epilogue masks them out.
// K is addressed in slabs: slab g of a row of B starts at byte
//   (g / slabs_per_block) * block_bytes + (g % slabs_per_block) * 128
// of the row (of A: at g * 128), which is the plain g * 128 for an ordinary row-major operand
// (slabs_per_block = number of slabs in a row) and lets the token-minor dL/dY of
// dR = X^T G be stored in blocks of a few thousand tokens, so that the 256 rows a tile
// reads at any one time lie within a couple of MiB instead of 256 separate pages.
// fp16 (heads and tails, split3_kernel): a row is [head | tail], slabs_per_block slabs each, and K walks head head + head tail + tail head:
// A head, head, tail, B head, tail, head (and stops after the first of them where there are no more slabs).
// The slab range [slab0, slab0 + k_slabs) must lie inside both operands' rows, and
// (BM-1)*lda*sizeof(T) + 128 (same for B) must fit 32 bits (the host checks this).
//
// Schedule.  A slab is two steps of MB*NB MFMA "slots", each on one set of fragments (64 bytes of K)
// that was read from LDS during the step before.  Everything that is not an MFMA is dealt out
// over the slots, one instruction behind an MFMA, and pinned there with sched_barrier, so the
// matrix pipe never waits for a block of memory instructions to issue.  Slab s:
//   first step:  read the fragments of the second step
//   second step, slot BAR (half of it): wait for this wave's loads of slab s + 1, barrier.  Behind it
//     slab s + 1 is complete, and the stages of slab s are free: every wave has its fragments.  Read the
//     fragments of the next step; load A of slab s + 2 into the stage A of slab s had, then B of slab
//     s + 3 into the stage of B's; the loads are spread over the slots up to the next BAR
// A step walks the blocks row by row (snake: neighbouring MFMAs share an operand).  The B
// fragments are double-buffered; A fragment i is used by one row of blocks only, so the next
// step's is read into the same registers once that row is done.  With the large tile an A load has
// 1600 cycles or more until the barrier that waits for it, a B load 2000 to 3400; three stages of
// both operands would not fit the LDS.
//
// What bounds it: the board's power limit for the large tile (the clock falls as the matrix pipe
// fills).  Cycles of the main loop of a 256 x 256 x 4096 tile (131 072 is the matrix pipe back to back):
//   173 000  loads through registers: an LDS store and the load behind it hold the only wave of a SIMD up by
//            ~20 cycles each; fragment reads and barriers cost next to nothing
//   163 000 - 170 000  straight into LDS in stages of 64 bytes of K: every 128-byte line is fetched twice
//   151 000  this form (and the scalar address arithmetic of the next slab ahead of its barrier; behind it: 153 600)
//
// ATN (bf16): operand A is given with K as its ROW index instead, A[k][lda] with the tile's
// rows m as consecutive columns (the activations X [token][feature] for dR = X^T G: no
// token-minor copy of X is needed).  K is walked in the order the other operand stores it
// (EpiGrad's: position 4a + b of a 64-token group is token a + 16 b), one
// group per slab.  A stage is then 64 tile rows of BM values, columns beyond M read from the last valid ones.  Fragments come from read_tr_operand,
// two lane quarters at a time reading 32 bytes of rows k .. k+3 and of rows k+8 .. k+11: the 32-byte
// pieces of a row are XOR-swizzled with 2 (row % 4) + (row / 8) % 2, which puts those eight into
// different banks.  Rows k >= k_valid are not read (the last valid row is read instead; the other
// operand is zero there).
//
// ATN / BTN in fp32: A (B) is given with K as its row index, in the order of the rows: R, W and X are read as they lie in
// memory and no launch writes a transposed copy of them first.  A stage is 32 tile rows of BM (BN) values; a fragment is four
// 4-byte LDS reads at rows 4 q .. 4 q + 3 (the fp32 matrix instruction is slow enough to hide them), the 64-byte pieces of a
// row XOR-swizzled with (row / 4) % 4, which puts the four lane quarters into different banks.  Columns beyond M (N) are read
// from the last four valid ones, so M (N) is a multiple of 4; rows of A beyond k_valid as above, B has all of its rows.
// With copies / in place, us: kt_fuse_rotation, side 1, d = 256, k = 4000: 19.4 / 11.5, d = 1024, k = 1000: 40.5 / 25.7,
// d = 3072, k = 9000: 1312 / 1240; fp32 fake-quant, d = 1024, 16 tokens: 30.2 / 25.6.
template <class TL, bool ATN, bool BTN, bool SWAP, bool AGAIN = false>
__device__ __forceinline__ void gemm_mainloop(const typename TL::T* __restrict__ A, int64_t lda,
                                              int M, int m0,
                                              const typename TL::T* __restrict__ B, int64_t ldb,
                                              int N, int n0, int slab0, int k_slabs,
                                              int slabs_per_block,
                                              int64_t block_bytes_b,
                                              floatx4 (&acc)[TL::MB][TL::NB], char* lds, int k_valid,
                                              int first_thread
                                              KT_STAMP_PARAM) {
  using T = typename TL::T;
  constexpr bool F32 = sizeof(T) == 4, F16 = std::is_same_v<T, _Float16>;
  static_assert(!BTN || F32, "BTN: fp32");
  constexpr int EPC = 16 / (int)sizeof(T);  // elements per 16-byte chunk
  constexpr int MB = TL::MB, NB = TL::NB, SLOTS = MB * NB, NFRAG = MB + NB;
  constexpr int A_LD = TL::A_LD, B_LD = TL::B_LD, NLD = A_LD + B_LD;
  constexpr int WAVE_LD = TL::NT * 16;  // bytes of a stage one load of every thread fills
  constexpr int A_PITCH = TL::BM * (int)sizeof(T);  // ATN: bytes of a stage row
  static_assert(!ATN || (A_PITCH >= 256 && WAVE_LD % A_PITCH == 0), "ATN: whole bank windows a row, whole rows a load");
  constexpr int BAR = SLOTS / 2, SPACE0 = SLOTS >= 4 * NFRAG ? 3 : 1, SPACE1 = SLOTS >= 4 * NFRAG ? 2 : 1;
  // load i is issued LOAD_AT(i) slots behind the barrier: the A loads in the first quarter of the interval
  // (a 256 x 256 x 4096 tile takes 163 000 cycles with 1/8, 157 000 with 3/16 or 3/8, 153 600 with this)
  constexpr int A_GAP = 2 * SLOTS / 4 / A_LD, B_GAP = (2 * SLOTS - 4 - A_LD * A_GAP) / B_LD;
  constexpr auto load_slot = [](int i) constexpr {
    return SLOTS + BAR + 1 + (i < A_LD ? i * A_GAP : A_LD * A_GAP + (i - A_LD) * B_GAP);
  };
  static_assert(A_GAP >= 1 && B_GAP >= 1 && load_slot(NLD - 1) - 2 * SLOTS < SLOTS + BAR - 3 && BAR + NB * SPACE1 <= SLOTS && BAR >= 2,
                "not enough MFMA slots to hide the memory instructions");

  const int tid = thread_id<AGAIN>() - first_thread;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // global addressing: uniform 64-bit base + 32-bit byte offsets.  Load i of a thread fills 16 bytes at
  // WAVE_LD i + 16 tid of a stage: row (NT / 8) i + tid / 8, chunk position tid % 8
  const char* Ab = reinterpret_cast<const char*>(ATN ? A + m0 : A + (int64_t)m0 * lda);
  const char* Bb = reinterpret_cast<const char*>(BTN ? B + n0 : B + (int64_t)n0 * ldb);
  uint32_t og[NLD];
  static_assert(TL::NT / 8 % 16 == 0, "swizzle key must not change between the loads of a thread");
  const int chunk = (tid & 7) ^ swizzle_key(tid >> 3);
  // ATN: stage row and 16-byte position of load i; tile row pr of a slab holds position pr of its 64-token group, i.e. token
  // pr / 4 + 16 (pr % 4) of the group (fp32: token pr of 32).  Columns as swizzled, at most the last ones of the operand.
  auto atn_row = [&](int i) __attribute__((always_inline)) { return (WAVE_LD * i + 16 * tid) / A_PITCH; };
  auto atn_token = [&](int i) __attribute__((always_inline)) { return F32 ? atn_row(i) : (atn_row(i) >> 2) + 16 * (atn_row(i) & 3); };
  auto f32_column = [&](int row, int pos, int left) __attribute__((always_inline)) {
    const int c = 4 * (pos ^ (((row >> 2) & 3) << 2));
    return c < left ? c : left - 4;
  };
  auto atn_offset = [&](int i, int token) __attribute__((always_inline)) {
    const int r = atn_row(i);
    if constexpr (F32) return (uint32_t)(((int64_t)token * lda + f32_column(r, tid % (TL::BM / 4), M - m0)) * 4);
    const int c = (tid % (A_PITCH / 16) ^ (2 * (2 * (r & 3) + ((r >> 3) & 1)))) * EPC, left = M - m0;
    return (uint32_t)(((int64_t)token * lda + (c < left ? c : left - EPC)) * (int64_t)sizeof(T));
  };
#pragma unroll
  for (int i = 0; i < A_LD; ++i) {
    if constexpr (ATN) {
      og[i] = atn_offset(i, atn_token(i));
    } else {
      int row = i * (TL::NT / 8) + (tid >> 3);
      row = (m0 + row < M) ? row : (M - 1 - m0);
      og[i] = (uint32_t)(((int64_t)row * lda + chunk * EPC) * (int64_t)sizeof(T));
    }
  }
#pragma unroll
  for (int i = 0; i < B_LD; ++i) {
    if constexpr (BTN) {
      const int row = (WAVE_LD * i + 16 * tid) / (TL::BN * 4);
      og[A_LD + i] = (uint32_t)(((int64_t)row * ldb + f32_column(row, tid % (TL::BN / 4), N - n0)) * 4);
    } else {
      int row = i * (TL::NT / 8) + (tid >> 3);
      row = (n0 + row < N) ? row : (N - 1 - n0);
      og[A_LD + i] = (uint32_t)(((int64_t)row * ldb + chunk * EPC) * (int64_t)sizeof(T));
    }
  }

  // The slabs to request next (A, B) and where they start inside a row: uniform values, advanced slab by slab; past
  // the last one: the last one again.
  int req_a = slab0, req_b = slab0, in_block_b = slab0 % slabs_per_block;
  const int last_slab = slab0 + k_slabs - 1;
  const int from_a = F16 && slab0 >= slabs_per_block ? slab0 - slabs_per_block : slab0, from_b = F16 && slab0 >= 2 * slabs_per_block ? slab0 - 2 * slabs_per_block : slab0;
  const char* an = Ab + (ATN ? (int64_t)slab0 * TL::BK * lda * (int64_t)sizeof(T)
                             : (int64_t)from_a * kRowBytes);
  const char* bn = Bb + (BTN ? (int64_t)slab0 * TL::BK * ldb * (int64_t)sizeof(T) : F16 ? (int64_t)from_b * kRowBytes
                             : (slab0 / slabs_per_block) * block_bytes_b + (int64_t)in_block_b * kRowBytes);
  const int64_t b_wrap = block_bytes_b - (int64_t)(slabs_per_block - 1) * kRowBytes;
  sgprx4 rsrc_a, rsrc_b;
  // take the next slab as the one gload() loads
  auto locate_a = [&]() __attribute__((always_inline)) {
    const char* a0 = an;
    if constexpr (ATN) {
      const int grp0 = req_a * TL::BK;
      if (grp0 + TL::BK > k_valid) {  // the last, partial group (and groups of padding behind it): re-read the last valid token
        const int base = grp0 < k_valid ? grp0 : (k_valid - 1) & ~(TL::BK - 1);
        a0 = Ab + (int64_t)base * lda * (int64_t)sizeof(T);
        const int last = k_valid - 1 - base;  // >= 0: the group starts inside the operand
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
          const int t = atn_token(i);
          og[i] = atn_offset(i, grp0 < k_valid && t < last ? t : last);
        }
      }
    }
    rsrc_a = raw_buffer(a0);
    if (req_a < last_slab) {
      ++req_a;
      an += ATN ? (int64_t)TL::BK * lda * (int64_t)sizeof(T) : (int64_t)kRowBytes;
      if constexpr (F16)
        if (req_a == slabs_per_block) an -= (int64_t)slabs_per_block * kRowBytes;
    }
  };
  auto locate_b = [&]() __attribute__((always_inline)) {
    rsrc_b = raw_buffer(bn);
    if (req_b < last_slab) {
      ++req_b;
      if constexpr (BTN) {
        bn += (int64_t)TL::BK * ldb * (int64_t)sizeof(T);
      } else if constexpr (F16) {
        bn += kRowBytes;
        if (req_b == 2 * slabs_per_block) bn -= 2 * (int64_t)slabs_per_block * kRowBytes;
      } else {
        const bool wrap = ++in_block_b == slabs_per_block;
        if (wrap) in_block_b = 0;
        bn += wrap ? b_wrap : (int64_t)kRowBytes;
      }
    }
  };

  // LDS layout: [A stage 0, 1][B stage 0, 1, 2]
  constexpr int B_BASE = kStagesA * TL::A_BYTES;
  const unsigned lds_wave = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds + wave * 1024u;
  unsigned b_write = 0;  // byte offset of the B stage to fill next
  int b_read = 0;        // ... of the B stage whose fragments are read
  const Frag<TL> f(tid);
  // fragment addresses, one per step of a slab: blocks and the A stage are instruction immediates
  const int key = swizzle_key(f.l16);
  int fa_s[2], fb_s[2], fb_now[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int coff = ((4 * h + f.q) ^ key) << 4;
    fa_s[h] = (f.wm * TL::WTM + f.l16) * kRowBytes + coff;
    fb_now[h] = fb_s[h] = B_BASE + (f.wn * TL::WTN + f.l16) * kRowBytes + coff;
  }
  // ATN: rows 8 q + l16 / 4 (+4), 32-byte piece wm WTM / 16 + block, column 4 (l16 % 4) of it; fp32: rows 4 q .. + 3 (and 16 h),
  // 64-byte piece wm WTM / 16 + block, column l16 of it
  int ft[ATN ? MB : 1], fbt[BTN ? NB : 1];
  if constexpr (ATN) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
      ft[i] = F32 ? 4 * f.q * (TL::BM * 4) + (((f.wm * TL::WTM / 16 + i) ^ f.q) << 6) + 4 * f.l16
                  : (8 * f.q + (f.l16 >> 2)) * A_PITCH + (((f.wm * TL::WTM / 16 + i) ^ (2 * (f.l16 >> 2) + (f.q & 1))) << 5) + 8 * (f.l16 & 3);
  }
  if constexpr (BTN) {
#pragma unroll
    for (int i = 0; i < NB; ++i) fbt[i] = B_BASE + 4 * f.q * (TL::BN * 4) + (((f.wn * TL::WTN / 16 + i) ^ f.q) << 6) + 4 * f.l16;
  }
  auto read_rows = [&](int addr, auto pitch_c) __attribute__((always_inline)) {
    constexpr int pitch = decltype(pitch_c)::value;
    const floatx4 v = {*reinterpret_cast<const float*>(lds + addr), *reinterpret_cast<const float*>(lds + addr + pitch),
                       *reinterpret_cast<const float*>(lds + addr + 2 * pitch), *reinterpret_cast<const float*>(lds + addr + 3 * pitch)};
    return __builtin_bit_cast(intx4, v);
  };

  intx4 fra[MB], frb[2][NB];  // MFMA fragments

  // load i of the slabs the locates took: A into A stage `stage`, B into the stage at b_write
  auto gload = [&](auto i_c, auto stage_c) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value, stage = decltype(stage_c)::value;
    if constexpr (i < A_LD)
      buffer_to_lds_16<stage * TL::A_BYTES + i * WAVE_LD>(og[i], rsrc_a, lds_wave);
    else
      buffer_to_lds_16<B_BASE + (i - A_LD) * WAVE_LD>(og[i], rsrc_b, lds_wave + b_write);
  };
  // LDS read r of the fragments of step h of the slab in A stage `stage` (r < NB: B fragment r, else A fragment r - NB)
  auto fread = [&](auto r_c, auto stage_c, auto h_c) __attribute__((always_inline)) {
    constexpr int r = decltype(r_c)::value, stage = decltype(stage_c)::value, h = decltype(h_c)::value;
    if constexpr (r < NB) {
      if constexpr (BTN) frb[h][r] = read_rows(fbt[r] + b_read + h * 16 * TL::BN * 4, std::integral_constant<int, TL::BN * 4>{});
      else frb[h][r] = *reinterpret_cast<const intx4*>(lds + fb_now[h] + r * 16 * kRowBytes);
    } else {
      constexpr int i = r - NB, off = stage * TL::A_BYTES;
      if constexpr (ATN && F32)
        fra[i] = read_rows(ft[i] + off + h * 16 * TL::BM * 4, std::integral_constant<int, TL::BM * 4>{});
      else if constexpr (ATN)
        fra[i] = read_tr_operand(lds, ft[i] + off + h * 32 * A_PITCH, ft[i] + off + h * 32 * A_PITCH + 4 * A_PITCH);
      else
        fra[i] = *reinterpret_cast<const intx4*>(lds + fa_s[h] + off + i * 16 * kRowBytes);
    }
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;

  // Slab s with s % 2 = STAGE.  The body is the same for every slab, so that the compiler sees one loop and no
  // accumulator-carrying branches: near the end of K the requests are clamped to the last slab (redundant,
  // in-bounds loads into stages nobody reads) and the last slab reads fragments nobody uses.
  auto one_slab = [&](auto stage_c) __attribute__((always_inline)) {
    constexpr int STAGE = decltype(stage_c)::value;
    using Cur = std::integral_constant<int, STAGE>;
    using Nxt = std::integral_constant<int, STAGE ^ 1>;
    static_for<2 * SLOTS>([&](auto g_c) __attribute__((always_inline)) {
      constexpr int g = decltype(g_c)::value, h = g / SLOTS, j = g % SLOTS;
      if constexpr (g == SLOTS + BAR) {
        stage_barrier<B_LD>();  // in flight at most: B of slab s + 2
      }
      // every load of the former requests has been issued; the next one comes after four MFMAs and a barrier (raw_buffer)
      if constexpr (g == SLOTS + BAR - 3) locate_a();
      if constexpr (g == SLOTS + BAR - 2) locate_b();
      if constexpr (g == SLOTS + BAR - 1) {
        b_write = b_write == 2 * TL::B_BYTES ? 0 : b_write + TL::B_BYTES;
        b_read = b_read == 2 * TL::B_BYTES ? 0 : b_read + TL::B_BYTES;
        fb_now[0] = fb_s[0] + b_read;
        fb_now[1] = fb_s[1] + b_read;
      }
      constexpr int mb = j / NB, nb = (mb & 1) ? NB - 1 - j % NB : j % NB;
      if constexpr (SWAP) Mma<T>::run(frb[h][nb], fra[mb], acc[mb][nb]);
      else Mma<T>::run(fra[mb], frb[h][nb], acc[mb][nb]);
      static_for<NFRAG>([&](auto r_c) __attribute__((always_inline)) {
        constexpr int r = decltype(r_c)::value;
        if constexpr (h == 0) {
          if constexpr (fragment_read_slot<MB, NB>(r, 0, SPACE0) == j) fread(r_c, Cur{}, S1{});
        } else {
          if constexpr (fragment_read_slot<MB, NB>(r, BAR, SPACE1) == j) fread(r_c, Nxt{}, S0{});
        }
      });
      static_for<NLD>([&](auto i_c) __attribute__((always_inline)) {
        constexpr int at = load_slot(decltype(i_c)::value);
        if constexpr (at == g) gload(i_c, Cur{});
        else if constexpr (at - 2 * SLOTS == g) gload(i_c, Nxt{});  // the stage of the slab before this one
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Prologue, as if slabs -2 and -1 had run: A and B of slab 0, B of slab 1, and of A(1), B(2) the loads that slab -1
  // issues behind its barrier; slab 0 issues the others.  Then the fragments of its first step.
  constexpr auto early_loads = [load_slot](int n) constexpr {
    int c = 0;
    for (int i = 0; i < n; ++i) c += load_slot(i) < 2 * SLOTS;
    return c;
  };
  locate_a();
  locate_b();
  raw_buffer_wait();
  static_for<NLD>([&](auto i_c) __attribute__((always_inline)) { gload(i_c, S0{}); });
  locate_b();
  raw_buffer_wait();
  b_write = TL::B_BYTES;
  static_for<B_LD>([&](auto i_c) __attribute__((always_inline)) { gload(std::integral_constant<int, A_LD + decltype(i_c)::value>{}, S0{}); });
  locate_a();
  locate_b();
  raw_buffer_wait();
  b_write = 2 * TL::B_BYTES;
  static_for<NLD>([&](auto i_c) __attribute__((always_inline)) {
    if constexpr (load_slot(decltype(i_c)::value) < 2 * SLOTS) gload(i_c, S1{});
  });
  stage_barrier<B_LD + early_loads(NLD)>();
  static_for<NFRAG>([&](auto r_c) __attribute__((always_inline)) { fread(r_c, S0{}, S0{}); });
  __builtin_amdgcn_sched_barrier(0);
  KT_STAMP_LOOP_START();

  int slab = 0;
  for (; slab + 1 < k_slabs; slab += 2) {
    one_slab(S0{});
    one_slab(S1{});
  }
  if (slab < k_slabs) one_slab(S0{});
  // no load into LDS outlives the loop
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  asm volatile("" ::: "memory");
}

// Tile L of the walk in bands of 4 tile-rows.
__device__ __forceinline__ void tile_in_bands(const GemmShape& g, int L, int& tm, int& tn) {
  constexpr int BAND = 4;
  const int band_tiles = BAND * g.tiles_n;
  const int band = L / band_tiles;
  const int first_m = band * BAND;
  const int rows = (g.tiles_m - first_m) < BAND ? (g.tiles_m - first_m) : BAND;
  const int in_band = L - band * band_tiles;
  tm = first_m + in_band % rows;
  tn = in_band / rows;
}

// Workgroup -> tile.  Consecutive workgroup ids land on different XCDs (8 of them,
// each with its own L2), so ids are first regrouped so that each XCD walks a
// contiguous range of tiles, then the range is walked in bands of 4 tile-rows so
// that the ~32 tiles an XCD holds at once share few A and B slabs.
__device__ __forceinline__ bool tile_of_block(const GemmShape& g, int& tm, int& tn, int& ks) {
  const int id = blockIdx.x;
  const int per_xcd = g.grid_padded >> 3;
  int L = (id & 7) * per_xcd + (id >> 3);
  if (L >= g.tiles_total) return false;
  const int per_split = g.tiles_m * g.tiles_n;
  ks = L / per_split;
  L -= ks * per_split;
  tile_in_bands(g, L, tm, tn);
  return true;
}

template <class TL, class Epi, bool ATN = false, bool BTN = false>
__global__ __launch_bounds__(TL::NT) void gemm_nt_kernel(GemmShape g, Epi epi) {
  extern __shared__ __align__(16) char lds[];
  using T = typename TL::T;
  const int batch = blockIdx.y;
  int tm, tn, ks;
  if (!tile_of_block(g, tm, tn, ks)) return;
  if (epi.skip(batch)) return;
  KT_STAMP_WALL(g, 4);
  KT_STAMP(g, 0);
  const int m0 = tm * TL::BM, n0 = tn * TL::BN;
  const int slab0 = ks * g.slabs_per_split;
  int slabs = g.slabs_total - slab0;
  slabs = slabs < g.slabs_per_split ? slabs : g.slabs_per_split;

  floatx4 acc[TL::MB][TL::NB];
#pragma unroll
  for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < TL::NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
  settle_all<TL>(acc);

  const T* A = static_cast<const T*>(g.A) + (int64_t)batch * g.batch_stride_a;
  const T* B = static_cast<const T*>(g.B) + (int64_t)batch * g.batch_stride_b;
  gemm_mainloop<TL, ATN, BTN, Epi::kSwap>(A, g.lda, g.M, m0, B, g.ldb, g.N, n0, slab0, slabs, g.slabs_per_block,
                         g.block_bytes_b, acc, lds, g.k_valid, 0 KT_STAMP_ARG);
  settle_all<TL>(acc);
  KT_STAMP(g, 2);
  epi(acc, batch, tm, tn, ks, m0, n0);
  KT_STAMP(g, 3);
  KT_STAMP_WALL(g, 5);
#ifdef KT_PHASE_STAMPS
  if (threadIdx.x == 0 && g.stamp_slot >= 0) {
    const size_t wg = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (wg < (size_t)kStampWgs)
      g_phase_stamps[((size_t)g.stamp_slot * kStampWgs + wg) * kStampWords + 6] = __builtin_amdgcn_s_getreg((4 << 0) | (0 << 6) | (31 << 11));
  }
#endif
}

// The same with K halved between two groups of four waves, each with LDS stages of its own, whose sums meet in the LDS; the first group has the epilogue.
// For tiles that leave a CU to one or two workgroups: the chain of a slab (barrier, fragments, matrix instructions) is longer than what it
// keeps busy, and two of them side by side fill it.  An even number of slabs, so that both groups meet at the same barriers.
template <class TL, class Epi>
__global__ __launch_bounds__(2 * TL::NT) void gemm_two_kernel(GemmShape g, Epi epi) {
  extern __shared__ __align__(16) char lds[];
  using T = typename TL::T;
  const int batch = blockIdx.y, group = __builtin_amdgcn_readfirstlane(threadIdx.x / TL::NT);
  int tm, tn, ks;
  if (!tile_of_block(g, tm, tn, ks)) return;
  if (epi.skip(batch)) return;
  const int m0 = tm * TL::BM, n0 = tn * TL::BN, slabs = g.slabs_total / 2;
  floatx4 acc[TL::MB][TL::NB];
#pragma unroll
  for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < TL::NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
  settle_all<TL>(acc);
  gemm_mainloop<TL, false, false, Epi::kSwap>(static_cast<const T*>(g.A) + (int64_t)batch * g.batch_stride_a, g.lda, g.M, m0,
                                              static_cast<const T*>(g.B) + (int64_t)batch * g.batch_stride_b, g.ldb, g.N, n0, group * slabs, slabs,
                                              g.slabs_per_block, g.block_bytes_b, acc, lds + group * TL::LDS_BYTES, 0, group * TL::NT);
  settle_all<TL>(acc);
  __syncthreads();
  floatx4* other = reinterpret_cast<floatx4*>(lds) + threadIdx.x % TL::NT;
  if (group == 1) {
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) other[(mb * TL::NB + nb) * TL::NT] = acc[mb][nb];
  }
  __syncthreads();
  if (group == 1) return;  // (barriers count the waves that are left)
#pragma unroll
  for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < TL::NB; ++nb) acc[mb][nb] += other[(mb * TL::NB + nb) * TL::NT];
  epi(acc, batch, tm, tn, 0, m0, n0);
}

}  // namespace kt
