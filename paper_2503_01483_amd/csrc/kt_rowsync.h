// kt_rowsync.h -- Y = X R with an epilogue that needs statistics of whole token rows, in one launch.
//
// The kurtosis gradient of a value (Eq. 3 and its chain rule) needs the moments of its token row, and an int4 code the row's largest
// magnitude; no output tile sees a whole row.  Here a tile publishes what it knows of its rows, waits for the other tiles of the same
// rows with its part of Y still in the accumulators, and then writes the result itself: Y does not reach memory.
//
// "Row block": the BN tokens of a column of tiles (features on the rows of the GEMM).  r row blocks x all `cols` tiles of their features
// are in flight at a time (r cols at most what the chip holds), one tile a workgroup.
//
// No workgroup relies on another one being resident.  Tiles are drawn in order (one queue per XCD, so that neighbours share an L2; a
// workgroup whose queue is empty goes to the next one), and the part of a row block that is in a queue is drawn before anything of
// the next row block: with at least that many workgroups to a queue (an eighth of the chip for 4096 features) the
// first row block that is not complete always gets there, whatever else runs on the chip.  With fewer (a stream with a few CUs) the wait
// ends after kRowWaitTicks a slab, the tile is put on the workgroup's own list, nobody waits from then on, and the lists are worked off,
// by a second product, once every tile has been drawn: whatever is waited for then has been published or is being computed.
// (That wait is bounded too: a row that never completes leaves NaN behind.)
//
// Against three launches (Y written in fp32 and read again, 8 bytes a value) with the products at the board's power limit: step of d = 4096, 131072 tokens
// 7910 -> 7390 us, d = 2048, 65536 tokens 1286 -> 1134; fake-quant of d = 4096, 16384 tokens 476 -> 436.  A tile of 4096 features, us: main loop 86
// (1.8 GHz), row moments and their exchange 6.1, wait 2.3, the row's coefficients 3.0, dL/dY 3.9.
//
// What is published goes past the L2 and is read past it: stores of a wave waited for, a barrier, a count per row block raised at
// device scope, and loads at device scope behind the count.  A release and an acquire would write back and drop an L2 that the
// products of the other 31 CUs live on.
#pragma once
#include "kt_aux.h"

namespace kt {

constexpr int kRowWaitTicks = 1200;  // of the 100 MHz counter: 12 us; a slab takes 1.0 to 1.5, and a tile ten slabs' time more
constexpr long long kRowLastWaitTicks = 20ll * 100000000;
// Counters, all zero at the start: of the queues at 0 .. 7, stop at 8, tiles of row block r that are published at 9 + r (and, RowQuant, whose
// error sums are at 9 + rows + r), `pitch` words apart.  A line takes an atomic every 10 ns or so: 512 workgroups that count in two lines
// spend 10 us on it (loss + gradient, d = 1024, 4096 tokens, 128 x 128 tiles, one word / kRowSyncPitch apart: 65 / 48 us).
constexpr int kRowSyncWords = 9, kRowSyncPitch = 32, kRowSyncMost = 512;

struct RowSync {
  unsigned* words;
  int pitch;
  int rows, cols;   // row blocks (of all problems), tiles of one
  int at_once;      // row blocks in flight
  int per_queue;    // tiles of a queue among those
  int items;        // length of a queue
  uint16_t order[kRowSyncMost];  // entry e of queue q among those: order[q per_queue + e], row block << 6 | column, 0xffff: none
  __device__ __forceinline__ unsigned* queue(int q) const { return words + q * pitch; }
  __device__ __forceinline__ unsigned* stop() const { return words + 8 * pitch; }
  __device__ __forceinline__ unsigned* done(int row) const { return words + (int64_t)(kRowSyncWords + row) * pitch; }
  // The row blocks in flight in bands of four, column by column; of that order every queue has a contiguous piece (the 32 tiles
  // an XCD works on share few slabs of either operand), which it walks row block by row block.
  __host__ void arrange() {
    int count[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int row = 0; row < at_once; ++row) {
      const int first = row & ~3, height = at_once - first < 4 ? at_once - first : 4;
      for (int col = 0; col < cols; ++col) {
        const int q = (first * cols + col * height + (row - first)) / per_queue;
        order[q * per_queue + count[q]++] = (uint16_t)(row << 6 | col);
      }
    }
    for (int q = 0; q < 8; ++q)
      while (count[q] < per_queue) order[q * per_queue + count[q]++] = 0xffff;
  }
  // entry i of queue q as row block * cols + column, -1: none
  __device__ __forceinline__ int tile(int q, int i) const {
    const int k = i / per_queue;
    const unsigned e = order[q * per_queue + (i - k * per_queue)];
    const int row = k * at_once + (int)(e >> 6);
    return e != 0xffffu && row < rows ? row * cols + (int)(e & 63u) : -1;
  }
};

template <class Op>
struct RowSyncArgs {
  GemmShape g;
  RowSync rs;
  Op op;
};

__device__ __forceinline__ unsigned past_load(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float past_load(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float2 past_load(const float2* p) {
  return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ floatx4 past_load(const floatx4* p) {
  const float2 a = past_load(reinterpret_cast<const float2*>(p)), b = past_load(reinterpret_cast<const float2*>(p) + 1);
  return floatx4{a.x, a.y, b.x, b.y};
}

// The epilogue: publish(acc, batch, tm, n0) stores the tile's share, finish(acc, complete, ...) has the rows' statistics; link(tile) is a
// word of scratch of that tile.  LDS: the first 16 bytes are the kernel's, `lds + 256` is free in finish().
template <class TL, class Op>
__global__ __launch_bounds__(TL::NT, (160 * 1024 / TL::LDS_BYTES)) void row_sync_kernel(RowSyncArgs<Op>) {
  extern __shared__ __align__(16) char lds[];
  // The arguments are read where they are needed: held across the tiles they are 106 scalar registers and spills of both kinds, and a
  // reload from scratch waits for every store in flight (the epilogue took twice as long).
  auto args = []() __attribute__((always_inline)) -> const RowSyncArgs<Op>& {
    typedef const __attribute__((address_space(4))) char* ConstPtr;
    ConstPtr p = (ConstPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const RowSyncArgs<Op>*)p;
  };
  using T = typename TL::T;
  int* said = reinterpret_cast<int*>(lds);
  // thread 0: the queue it takes from, its latest draw from it, the last tile of its list
  int queue = blockIdx.x & 7, tried = 0, drawn = 0, list = -1;
  auto draw = [&](const RowSync& rs) __attribute__((always_inline)) {
    drawn = (int)__hip_atomic_fetch_add(rs.queue(queue), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // the tile that was drawn, or the next one there is, or -1
  auto next_tile = [&]() __attribute__((always_inline)) {
    const RowSync& rs = args().rs;
    while (tried < 8) {
      if (drawn >= rs.items) {
        queue = (queue + 1) & 7;
        ++tried;
      } else {
        const int t = rs.tile(queue, drawn);
        if (t >= 0) return t;
      }
      if (tried < 8) draw(rs);
    }
    return -1;
  };
  // whether the row block is complete (wave 0)
  auto wait = [&](const RowSync& rs, int row, bool last) __attribute__((always_inline)) {
    unsigned* stop = rs.stop();
    const long long t0 = __builtin_amdgcn_s_memrealtime();
    auto load = [](const unsigned* p) __attribute__((always_inline)) { return (unsigned)__builtin_amdgcn_readfirstlane((int)past_load(p)); };
    for (int polls = 0; load(rs.done(row)) < (unsigned)rs.cols; ++polls) {
      if ((polls & 15) == 15) {
        const bool late = (long long)__builtin_amdgcn_s_memrealtime() - t0 > (last ? kRowLastWaitTicks : (long long)kRowWaitTicks * (args().g.slabs_total + 10));
        if (late || (!last && load(stop) != 0u)) {
          if (threadIdx.x == 0) __hip_atomic_store(stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return false;
        }
      }
      __builtin_amdgcn_s_sleep(1);
    }
    return true;
  };

  if (threadIdx.x == 0) draw(args().rs);
#pragma unroll 1
  for (;;) {
    if (threadIdx.x == 0) {
      const int next = next_tile();
      const bool again = next < 0 && list >= 0;
      said[0] = again ? list : next;
      said[1] = again;
      if (again) list = (int)past_load(reinterpret_cast<const unsigned*>(args().op.link(list, args().rs.cols)));
    }
    __syncthreads();
    const int tile = __builtin_amdgcn_readfirstlane(said[0]);
    const bool again = __builtin_amdgcn_readfirstlane(said[1]) != 0;
    __syncthreads();
    if (tile < 0) return;
    const int cols = args().rs.cols, tiles_n = args().g.tiles_n;
    const int row = tile / cols, tm = tile - row * cols, batch = row / tiles_n, tn = row - batch * tiles_n;
    const int m0 = tm * TL::BM, n0 = tn * TL::BN;
    floatx4 acc[TL::MB][TL::NB];
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
    settle_all<TL>(acc);
    {
      const GemmShape& g = args().g;
      gemm_mainloop<TL, false, false, false, true>(static_cast<const T*>(g.A) + (int64_t)batch * g.batch_stride_a, g.lda, g.M, m0,
                                             static_cast<const T*>(g.B) + (int64_t)batch * g.batch_stride_b, g.ldb, g.N, n0, 0, g.slabs_total,
                                             g.slabs_per_block, 0, acc, lds, 0, 0);
    }
    settle_all<TL>(acc);
    if (!again) {
      args().op.publish(acc, batch, tm, n0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores are where everybody reads them
    }
    __syncthreads();  // (and the main loop's LDS is free)
    if (threadIdx.x < 64) {
      const RowSync& rs = args().rs;
      if (!again && threadIdx.x == 0) __hip_atomic_fetch_add(rs.done(row), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool ok = wait(rs, row, again);
      if (threadIdx.x == 0) {
        said[0] = ok;
        if (!again) draw(rs);  // not before: while it waits, a workgroup holds no tile that others may wait for
      }
    }
    __syncthreads();
    const bool complete = __builtin_amdgcn_readfirstlane(said[0]) != 0;
    if (!complete && !again) {
      if (threadIdx.x == 0) {
        __hip_atomic_store(reinterpret_cast<unsigned*>(args().op.link(tile, cols)), (unsigned)list, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        list = tile;
      }
    } else {
      args().op.finish(acc, complete, lds, batch, row, tm, tn, m0, n0);
    }
    __syncthreads();  // the LDS is free again
  }
}

// row_central_sums of partials of BM features, the last of what is left of d.  CH > 0: P <= CH, all loads in flight at once (past the last
// partial: that one again).
template <int CH, int BM, class Load>
__device__ __forceinline__ void row_sums_of_tiles(Load load, int P, int d, double& mu, double (&M)[3]) {
  const double cnt = (double)BM, rest = (double)(d - (P - 1) * BM);
  double m = 0.0;
  M[0] = M[1] = M[2] = 0.0;
  if constexpr (CH > 0) {
    floatx4 v[CH];
#pragma unroll
    for (int p = 0; p < CH; ++p) v[p] = load(p < P ? p : P - 1);
#pragma unroll
    for (int p = 0; p < CH; ++p)
      if (p < P) m += (p == P - 1 ? rest : cnt) * (double)v[p][0];
    mu = m / (double)d;
#pragma unroll
    for (int p = 0; p < CH; ++p)
      if (p < P) add_partial(v[p], p == P - 1 ? rest : cnt, mu, M);
  } else {
#pragma unroll 8
    for (int p = 0; p < P; ++p) m += (p == P - 1 ? rest : cnt) * (double)load(p)[0];
    mu = m / (double)d;
#pragma unroll 8
    for (int p = 0; p < P; ++p) add_partial(load(p), p == P - 1 ? rest : cnt, mu, M);
  }
}

// ---- kurtosis loss and dL/dY ("Learning the Rotations"; Eq. 3) ------------------------------
// Publishes the moments of EpiMoments; with those of the whole row (merged in fp64, as in finalize_rows_kernel) the accumulators become dL/dY in
// the layout of EpiGrad.  The tile of the first features also takes the loss terms of its tokens: loss_part[row block].
template <class TL>
struct RowLossGrad {
  EpiMoments<TL, true> mom;
  EpiGrad<TL> grad;
  float kappa_target;
  float* row_kurt;  // or null
  double* loss_part;
  int tiles_n;
  __device__ __forceinline__ int* link(int tile, int cols) const {
    const int row = tile / cols, batch = row / tiles_n, n0 = (row - batch * tiles_n) * TL::BN, m0 = (tile - row * cols) * TL::BM;
    const int64_t blk = n0 / grad.tb;
    return reinterpret_cast<int*>(grad.GT + (int64_t)batch * grad.batch_stride + blk * grad.d * grad.tb + (n0 - blk * grad.tb) + (int64_t)m0 * grad.tb);
  }
  __device__ __forceinline__ void publish(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm, int n0) const {
    mom(acc, batch, tm, 0, 0, tm * TL::BM, n0);
  }
  __device__ __forceinline__ void finish(floatx4 (&acc)[TL::MB][TL::NB], bool complete, char* lds, int batch, int row, int tm, int, int m0,
                                         int n0) const {
    floatx4* coef = reinterpret_cast<floatx4*>(lds + 256);
    const int n = mom.n_tokens, token = n0 + (int)threadIdx.x, P = mom.P;
    double term = 0.0;
    if ((int)threadIdx.x < TL::BN) {
      floatx4 c = {0.f, 0.f, 0.f, 0.f};
      if (token < n) {
        const floatx4* part = mom.part + (int64_t)batch * P * n + token;
        auto load = [&](int p) __attribute__((always_inline)) { return past_load(part + (int64_t)p * n); };
        double mu, M[3], kappa;
        if (P <= 8) row_sums_of_tiles<8, TL::BM>(load, P, grad.d, mu, M);
        else if (P <= 16) row_sums_of_tiles<16, TL::BM>(load, P, grad.d, mu, M);
        else row_sums_of_tiles<0, TL::BM>(load, P, grad.d, mu, M);
        c = row_coefficients(mu, M, n, grad.d, kappa_target, kappa, term);
        if (!complete) c = floatx4{0.f, 0.f, 0.f, 0.f} * __builtin_nanf("");
        if (tm == 0 && row_kurt) row_kurt[(int64_t)batch * n + token] = complete ? (float)kappa : __builtin_nanf("");
      }
      coef[threadIdx.x] = c;
    }
    if (tm == 0) {  // uniform
      double* sh = reinterpret_cast<double*>(lds + 256 + TL::BN * 16);
      const double s = block_sum_256(complete ? term : (double)__builtin_nanf(""), sh);
      if (threadIdx.x == 0) loss_part[row] = s;
    }
    __syncthreads();
    grad.template store<true>(acc, batch, m0, n0, [&](int t) __attribute__((always_inline)) { return coef[t]; });
  }
};

// ---- int4 codes of Y = X R (Eq. 1, one scale per token) -------------------------------------
// Publishes the largest magnitudes of EpiAmax; with the row's maximum the accumulators become the codes of EpiQuant.  The error sums are
// published too, and the last tile of a row block adds them.
template <class TL>
struct RowQuant {
  EpiAmax<TL, true> amax;
  EpiQuant<TL, true> quant;
  float clip;
  float* scales_out;  // or null
  float2* err;        // or null
  int* links;         // [rows * cols]
  unsigned* added;    // of row block 0, `pitch` words apart
  int pitch, cols;
  __device__ __forceinline__ int* link(int tile, int) const { return links + tile; }
  __device__ __forceinline__ void publish(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm, int n0) const {
    amax(acc, batch, tm, 0, 0, tm * TL::BM, n0);
  }
  __device__ __forceinline__ void finish(floatx4 (&acc)[TL::MB][TL::NB], bool complete, char* lds, int batch, int row, int tm, int, int m0,
                                         int n0) const {
    float2* scale = reinterpret_cast<float2*>(lds + 256);
    const int n = amax.n_tokens, token = n0 + (int)threadIdx.x, P = amax.P;
    const bool mine = (int)threadIdx.x < TL::BN && token < n;
    if ((int)threadIdx.x < TL::BN) {
      float s = 0.f;
      if (mine) {
        const float* part = amax.part + (int64_t)batch * P * n + token;
        float a = 0.f;
#pragma unroll 8
        for (int p = 0; p < P; ++p) a = fmaxf(a, past_load(part + (int64_t)p * n));
        s = complete ? __fdiv_rn(__fmul_rn(clip, a), 7.0f) : __builtin_nanf("");
        if (tm == 0 && scales_out) scales_out[(int64_t)batch * n + token] = s;
      }
      scale[threadIdx.x] = make_float2(s, s > 0.f ? __fdiv_rn(1.0f, s) : 0.f);
    }
    __syncthreads();
    quant.apply(acc, batch, tm, m0, n0, [&](int t) __attribute__((always_inline)) { return scale[t]; });
    if (!err) return;  // uniform
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* said = reinterpret_cast<int*>(lds);
    if (threadIdx.x == 0) said[0] = (int)__hip_atomic_fetch_add(added + (int64_t)row * pitch, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(said[0]) != cols - 1 || !mine) return;
    const float2* part = quant.err_part + (int64_t)batch * P * n + token;
    float e2 = 0.f, y2 = 0.f;
#pragma unroll 8
    for (int p = 0; p < P; ++p) {
      const float2 v = past_load(part + (int64_t)p * n);
      e2 += v.x;
      y2 += v.y;
    }
    err[(int64_t)batch * n + token] = make_float2(e2, y2);
  }
};

}  // namespace kt
