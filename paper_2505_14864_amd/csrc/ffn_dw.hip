// Weight gradients of the grouped SwiGLU FFN, dW[e] = P_e^T Q_e over the rows of expert e (bf16 in, fp32 accumulate), where the
// sums are too short or the tiles too few for the 256 x 256 tiles of ffn_mfma.hip.  The three gradients are one launch.
//
// One workgroup of four wavefronts (2 x 2) per output tile of 128 x 256 (64 x 128 per wavefront), 128 x 128 (64 x 64) or
// 64 x 64 (32 x 32); two (three, five) of them share a compute unit.  k goes in steps of 32 (one MFMA deep) through a ring of
// three (64 x 64: four) LDS stages, filled by buffer loads with an LDS destination.  Both operands lie [k][row] in memory and
// in LDS and are read with ds_read_b64_tr_b16, free of bank conflicts: the LDS cycles lost to conflicts are the same for a tile of 64
// k steps as for one of 8 (480 and 510 per tile of 128 x 256, 3.6 and 17.5 % of the LDS cycles), so they are the epilogue patch's.
//
// What bounds it: with 64 experts of about 256 rows (2048 x 1024; 12288 tiles of eight k steps) the time is the same without the
// MFMAs, and half without the loads: memory and the start of a tile.  Hence
//   * the results leave through a bf16 patch in the one LDS stage that is free then: the MFMAs have their operands swapped, so
//     that a lane holds four neighbours of a row, one 8-byte LDS store, where accumulators in column order were four
//     4-byte ones in fp32;
//   * 128 x 256 tiles, where there are thousands of short ones (AHEAD): a workgroup walks several of them; the loads run NS - 1 k
//     steps ahead of the arithmetic across the end of a tile, so that the next tile's first steps are on their way while the
//     last ones of this tile are computed and stored;
//   * there, and where tiles are long, a step's fragments are read while the step before is computed.
#include "ffn_gemm.h"
#include "tile_list.h"

namespace dynmo {

constexpr int kDwThreads = 256;

// One weight gradient dW[e] = P_e^T Q_e (M x N per expert)
struct DwSet {
  const bf16_t* P;
  const bf16_t* Q;
  bf16_t* C;
  int M, N;
  int tiles;  // output tiles per expert
};

struct DwParams {
  const int32_t* seg;
  int E;
  DwSet dw[3];  // the products of this launch
  int sets;
  int per_expert;  // tiles of them per expert
  TileList list;
  int walk;        // tiles per workgroup (AHEAD)
};

// WBM x WBN blocks of 16 x 16 per wavefront
template <int WBM, int WBN>
struct DwShape {
  static constexpr int kRows = 32 * WBM, kCols = 32 * WBN;  // of the output tile
  static constexpr int kStages = WBN == 2 ? 4 : 3;
  static constexpr int kBytesA = kRows * kTileK * 2, kBytesB = kCols * kTileK * 2;
  static constexpr int kStage = kBytesA + kBytesB;
  static constexpr int kPiecesA = kBytesA / 4096, kPiecesB = kBytesB / 4096;  // pieces of 1 KB a wavefront loads per stage
  static constexpr int kLoads = kPiecesA + kPiecesB;
  static constexpr int kPatchBytes = 16 * WBN * 32;     // a wavefront's epilogue patch: 16 rows of bf16
  static constexpr int kLds = kStages * kStage;
  static_assert(4 * kPatchBytes <= kStage, "the epilogue patches lie in one stage");
};

// The lane index behind a compiler barrier: what is derived from it is recomputed where it is used, once per tile,
// instead of being computed at kernel entry and kept in scratch memory across the k loop.
__device__ __forceinline__ int lane_now() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

// Byte offsets, from the tile's (row 0, k 0) element, of the 16 bytes this lane moves in each of the
// wavefront's pieces (kOob: nothing).
template <int ROWS>
struct DwPieces {
  static constexpr int N = ROWS * kTileK * 2 / 4096;
  uint32_t off[N];

  __device__ __forceinline__ void init(uint32_t ld_bytes, int rows_left) {
    const int lane = lane_now(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int q = wave * N + j;
      off[j] = krow_piece<ROWS>(q, lane, ld_bytes, rows_left);
    }
  }
};

// Where 16-byte unit `unit` of row `row` of an epilogue patch with ROW_BYTES per row is kept: the accumulators are
// written by sixteen lanes of one column group, each into its own row, and read back along rows.
template <int ROW_BYTES>
__device__ __forceinline__ uint32_t patch_at(int row, int unit) {
  constexpr int kUnits = ROW_BYTES / 16, kShift = kUnits >= 16 ? 0 : kUnits == 8 ? 1 : kUnits == 4 ? 2 : 3;
  return row * ROW_BYTES + ((unit ^ ((row >> kShift) & (kUnits - 1))) << 4);
}

// A fragment in registers, read by two transposing 8-byte reads.  They are assembly with the fragment as an in-out operand, so
// that a new value takes the registers of the old one; the waits for them are written out (wait_lds).
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
constexpr int kReads = 2;
struct DwFrag {
  u32x2_t lo, hi;
  __device__ __forceinline__ DwFrag() { asm volatile("" : "=v"(lo), "=v"(hi)); }  // any value, in registers of its own
  __device__ __forceinline__ bf16x8_t operand() const {
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
  }
  template <int K_STRIDE>
  __device__ __forceinline__ void read(uint32_t addr) {
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "+v"(lo) : "v"(addr) : "memory");
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "+v"(hi) : "v"(addr), "n"(4 * K_STRIDE) : "memory");
  }
};

// The same as ordinary reads, which the compiler waits for
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
template <int K_STRIDE>
__device__ __forceinline__ bf16x8_t read_now(uint32_t addr) {
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(uintptr_t)addr);
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(uintptr_t)(addr + 4 * K_STRIDE));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Waits until at most N LDS reads are outstanding (they complete in order); nothing moves across.
template <int N>
__device__ __forceinline__ void wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N < 15 ? N : 15) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <int WBM, int WBN, bool AHEAD>
__global__ __launch_bounds__(kDwThreads, WBN == 8 ? 2 : WBN == 4 ? 3 : 4) void ffn_dw_kernel(const DwParams p) {
  using S = DwShape<WBM, WBN>;
  __shared__ __attribute__((aligned(1024))) char smem[S::kLds];
  constexpr int TM = S::kRows, TN = S::kCols, NS = S::kStages;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;

  // ---- which tiles.  Workgroup b runs on XCD b % 8; every XCD takes runs of `group` consecutive tiles, which share
  // operand tiles in its L2.  A workgroup takes `walk` tiles, the i-th one from the i-th run.
  struct Job {
    int m0, n0, M, N, k_begin, k_end;
    const bf16_t *P, *Q;
    bf16_t* C;
  };
  auto job_at = [&](int step, Job& j) {
    const int slot = blockIdx.x >> 3, run = run_of(p.list, slot);
    const int pos = ((AHEAD ? run * p.walk + step : run) * 8 + (blockIdx.x & 7)) * p.list.group + slot - run * p.list.group;
    const int e = pos / p.per_expert;
    if (e >= p.E) return false;  // past the last tile
    int r = pos - e * p.per_expert, set = 0;
    while (r >= p.dw[set].tiles) r -= p.dw[set++].tiles;
    const DwSet& w = p.dw[set];
    int mi, ni;
    tile_of(r, (w.M + TM - 1) / TM, (w.N + TN - 1) / TN, &mi, &ni);
    j.m0 = mi * TM;
    j.n0 = ni * TN;
    j.M = w.M;
    j.N = w.N;
    j.k_begin = __builtin_amdgcn_readfirstlane(p.seg[e]);
    j.k_end = __builtin_amdgcn_readfirstlane(p.seg[e + 1]);
    j.P = w.P;
    j.Q = w.Q;
    j.C = w.C + (long)e * w.M * w.N;
    return true;
  };

  // ---- the stream of k steps to load: those of this tile, then those of the next one
  DwPieces<TM> pa;
  DwPieces<TN> pb;
  const bf16_t *na = nullptr, *nb = nullptr;
  uint32_t lda_b = 0, ldb_b = 0;
  int k_left = 0;  // rows left to load
  auto steps_of = [&](const Job& j) { return (j.k_end - j.k_begin + kTileK - 1) / kTileK; };
  auto stream_from = [&](const Job& j) {
    lda_b = (uint32_t)j.M * 2;
    ldb_b = (uint32_t)j.N * 2;
    pa.init(lda_b, j.M - j.m0);
    pb.init(ldb_b, j.N - j.n0);
    na = j.P + (long)j.k_begin * j.M + j.m0;
    nb = j.Q + (long)j.k_begin * j.N + j.n0;
    k_left = j.k_end - j.k_begin;
  };
  struct Descs {
    desc_t a, b;
    uint32_t to_a, to_b;
  };
  // descriptors of the next k step, to go into the stage at byte `stage`.  k-rows are whole records, so the record count is
  // the k mask; past the last step the loads fetch nothing
  auto next_step = [&](uint32_t stage) {
    Descs q;
    const uint32_t k_rows = (uint32_t)max(0, min(k_left, kTileK));
    q.a = make_desc(na, k_rows * lda_b);
    q.b = make_desc(nb, k_rows * ldb_b);
    q.to_a = __builtin_amdgcn_readfirstlane(lds0 + stage + wave * S::kPiecesA * 1024);
    q.to_b = __builtin_amdgcn_readfirstlane(lds0 + stage + wave * S::kPiecesB * 1024);
    na += (long)kTileK * (lda_b / 2);
    nb += (long)kTileK * (ldb_b / 2);
    k_left -= kTileK;
    return q;
  };
  auto load_piece = [&](const Descs& q, auto J) {
    constexpr int j = decltype(J)::value;
    if constexpr (j < S::kPiecesA) load_to_lds<j * 1024>(q.a, q.to_a, pa.off[j]);
    else load_to_lds<S::kBytesA + (j - S::kPiecesA) * 1024>(q.b, q.to_b, pb.off[j - S::kPiecesA]);
  };
  auto issue = [&](uint32_t stage) {
    const Descs q = next_step(stage);
    static_for<S::kLoads>([&](auto J) { load_piece(q, J); });
  };

  Job job;
  if (!job_at(0, job)) return;
  stream_from(job);
  uint32_t stage = 0;  // of the tile's next k step
  auto following = [](uint32_t s) { return s + S::kStage == S::kLds ? 0u : s + S::kStage; };
  auto last_of_ring = [&](uint32_t s) { return s == 0 ? (uint32_t)(S::kLds - S::kStage) : s - S::kStage; };
  static_for<NS - 1>([&](auto J) { issue(decltype(J)::value * S::kStage); });
  if constexpr (AHEAD) {
    wait_stage<(NS - 2) * S::kLoads>();  // the first k step has landed
    __builtin_amdgcn_s_barrier();
  }
  // A whole tile's stores per wavefront, which the first wait of the next tile need not include.
  constexpr int kStores = WBM * (WBN / 2);
  bool stores_out = false;

  for (int step = 0;; ++step) {
    // Every tile is walked in at least NS - 1 steps (zeros past the last one), so that the loads that run ahead of the
    // arithmetic are never more than one tile ahead.
    const bool more_asked = AHEAD && step + 1 < p.walk;
    const int n_kt = max(steps_of(job), more_asked ? NS - 1 : 1);
    Job next;
    const bool more = more_asked && job_at(step + 1, next);
    const int valid16 = min(2 * WBM, (job.M - job.m0 + 15) / 16);
    const bool cols_ok = job.n0 + wn * (TN / 2) < job.N;
    // row blocks with work: blocks wm, wm + 2, .. of the tile (in a ragged tile the valid rows are a prefix, and every
    // wavefront keeps its share)
    const int my_rows = cols_ok && valid16 > wm ? (valid16 - wm + 1) / 2 : 0;
    // before k step kt + NS is issued: past this tile's last step the loads are the next tile's
    auto switch_tiles = [&](int kt) {
      if (kt + NS == n_kt && more) stream_from(next);
    };
    f32x4_t acc[WBM][WBN] = {};

    // ---- k loop.  On entry k step 0 has landed for all wavefronts and steps 1 .. NS - 2 are on their way.  A step's MFMAs go
    // row block by row block.  Behind the first row this wavefront's pieces of the next step have landed and all reads of
    // this step's stage are done; behind the barrier that holds for all: the stage is refilled and the next step's
    // fragments are read between the remaining MFMAs, each into the registers of the old one once that has been used up
    // (A 0 .. LAST - 1 after their rows, B in the last row, A LAST), so that neither latency is waited for.
    auto loop = [&](auto ROWS_C) {
      constexpr int ROWS = decltype(ROWS_C)::value, LAST = ROWS - 1, kSlots = WBN * ROWS, kFrom = WBN;
      const int lane = lane_now();
      uint32_t ra[WBM], rb[WBN];
#pragma unroll
      for (int i = 0; i < WBM; ++i) ra[i] = lds0 + krow_frag<TM>(lane, wm + 2 * i);
#pragma unroll
      for (int j = 0; j < WBN; ++j) rb[j] = lds0 + S::kBytesA + krow_frag<TN>(lane, wn * WBN + j);
      DwFrag fa[ROWS], fb[WBN];
      auto read_a = [&](int i, uint32_t from) { fa[i].template read<TM * 2>(ra[i] + from); };
      auto read_b = [&](int j, uint32_t from) { fb[j].template read<TN * 2>(rb[j] + from); };
#pragma unroll
      for (int i = 0; i < LAST; ++i) read_a(i, stage);
#pragma unroll
      for (int j = 0; j < WBN; ++j) read_b(j, stage);
      read_a(LAST, stage);
      // the epilogue's patches are free: the last one of the first NS k steps goes there
      __builtin_amdgcn_s_barrier();
      switch_tiles(-1);
      issue(last_of_ring(stage));
      auto body = [&](auto REFILL_C, auto FIRST_C) {
        constexpr bool refill = decltype(REFILL_C)::value;
        constexpr int kInFlight = (NS - 2) * S::kLoads + (decltype(FIRST_C)::value ? kStores : 0);
        const uint32_t freed = stage, to_read = following(stage);
        Descs q = {};
        if constexpr (refill) q = next_step(freed);
        static_for<kSlots>([&](auto M) {
          constexpr int m = decltype(M)::value, i = m / WBN, j = m % WBN;
          if constexpr (ROWS == 1 && m == 0) wait_lds<0>();
          if constexpr (ROWS > 1 && i == 0) wait_lds<(WBN - 1 - j) * kReads + kReads>();
          if constexpr (ROWS > 1 && m == kFrom) {
            if constexpr (refill) {
              wait_stage<kInFlight>();
              __builtin_amdgcn_s_barrier();
            } else {
              wait_lds<0>();
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (ROWS > 1 && refill && m >= kFrom) {
            static_for<S::kLoads>([&](auto L) {  // at even distances
              if constexpr (kFrom + decltype(L)::value * (kSlots - kFrom) / S::kLoads == m) load_piece(q, L);
            });
            if constexpr (j == 0) read_a(i - 1, to_read);
          }
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j].operand(), fa[i].operand(), acc[i][j], 0, 0, 0);
          if constexpr (ROWS > 1 && refill && i == LAST) {
            read_b(j, to_read);
            if constexpr (j == WBN - 1) read_a(LAST, to_read);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (ROWS == 1 && refill) {
          wait_stage<kInFlight>();
          __builtin_amdgcn_s_barrier();
#pragma unroll
          for (int j = 0; j < WBN; ++j) read_b(j, to_read);
          read_a(0, to_read);
          static_for<S::kLoads>([&](auto L) { load_piece(q, L); });
          __builtin_amdgcn_sched_barrier(0);
        }
        stage = to_read;
      };
      int kt = 0;
      if (ROWS == WBM && stores_out && n_kt > 1) {
        switch_tiles(0);
        body(std::true_type{}, std::true_type{});
        kt = 1;
      }
      for (; kt + 1 < n_kt; ++kt) {
        switch_tiles(kt);
        body(std::true_type{}, std::false_type{});
      }
      body(std::false_type{}, std::false_type{});
    };
    // Short tiles that are not walked: the other workgroups of the compute unit cover what the loop above reads ahead for, and its code
    // is more than twice as long.
    auto plain_loop = [&](auto ROWS_C) {
      constexpr int ROWS = decltype(ROWS_C)::value;
      const int lane = lane_now();
      uint32_t ra[WBM], rb[WBN];
#pragma unroll
      for (int i = 0; i < WBM; ++i) ra[i] = lds0 + krow_frag<TM>(lane, wm + 2 * i);
#pragma unroll
      for (int j = 0; j < WBN; ++j) rb[j] = lds0 + S::kBytesA + krow_frag<TN>(lane, wn * WBN + j);
      for (int kt = 0; kt < n_kt; ++kt) {
        wait_stage<(NS - 2) * S::kLoads>();
        __builtin_amdgcn_s_barrier();
        issue(last_of_ring(stage));
        if constexpr (ROWS > 0) {
          bf16x8_t a[ROWS], b[WBN];
#pragma unroll
          for (int i = 0; i < ROWS; ++i) a[i] = read_now<TM * 2>(ra[i] + stage);
#pragma unroll
          for (int j = 0; j < WBN; ++j) b[j] = read_now<TN * 2>(rb[j] + stage);
#pragma unroll
          for (int j = 0; j < WBN; ++j)
#pragma unroll
            for (int i = 0; i < ROWS; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
        }
        stage = following(stage);
      }
    };
    if constexpr (!AHEAD) {
      if (my_rows == WBM) plain_loop(std::integral_constant<int, WBM>{});
      else if (WBM > 3 && my_rows == 3) plain_loop(std::integral_constant<int, WBM - 1>{});
      else if (my_rows == 2) plain_loop(std::integral_constant<int, WBM < 2 ? WBM : 2>{});
      else if (my_rows == 1) plain_loop(std::integral_constant<int, 1>{});
      else plain_loop(std::integral_constant<int, 0>{});
    } else if (my_rows == WBM) {
      loop(std::integral_constant<int, WBM>{});
    } else if (my_rows == 0) {  // a wavefront without work only keeps up the loads and the barriers
      __builtin_amdgcn_s_barrier();
      switch_tiles(-1);
      issue(last_of_ring(stage));
      for (int kt = 0; kt + 1 < n_kt; ++kt) {
        wait_stage<(NS - 2) * S::kLoads>();
        __builtin_amdgcn_s_barrier();
        switch_tiles(kt);
        issue(stage);
        stage = following(stage);
      }
      stage = following(stage);
    } else {
      if (my_rows == 1) loop(std::integral_constant<int, 1>{});
      else if (my_rows == 2) loop(std::integral_constant<int, 2>{});
      else loop(std::integral_constant<int, 3>{});
    }
    if (more) wait_stage<(NS - 2) * S::kLoads>();  // the next tile's first k step has landed
    else wait_stage<0>();                          // nothing is on its way to LDS when the workgroup ends
    __builtin_amdgcn_s_barrier();

    // ---- epilogue.  `stage` is the next tile's first k step's; the last one of the ring behind it is free.  Accumulator element r
    // of block (i, j) is column 16 j + 4 (lane / 16) + r of row lane % 16.  A wavefront passes sixteen rows at a time through
    // its own patch, so that global memory sees 16-byte accesses along rows; no barrier, a wavefront's LDS accesses complete in order.
    const int lane = lane_now();
    char* const patch = smem + last_of_ring(stage) + wave * S::kPatchBytes;
    constexpr int kRowBytes = WBN * 32, kLanesPerRow = WBN * 2, kRowsPerPass = 64 / kLanesPerRow;
    const int row_l = lane & 15, quad = lane >> 4;
    const int c0 = lane % kLanesPerRow, col = job.n0 + wn * (TN / 2) + c0 * 8;
#pragma unroll
    for (int i = 0; i < WBM; ++i) {
      if (i >= my_rows) break;
#pragma unroll
      for (int j = 0; j < WBN; ++j) {
        const f32x4_t v = acc[i][j];
        *(u32x2_t*)(patch + patch_at<kRowBytes>(row_l, 2 * j + (quad >> 1)) + (quad & 1) * 8) =
            u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      }
#pragma unroll
      for (int s = 0; s < 16 / kRowsPerPass; ++s) {
        const int rl = s * kRowsPerPass + lane / kLanesPerRow, row = job.m0 + (2 * i + wm) * 16 + rl;
        if (row >= job.M || col >= job.N) continue;
        *(u32x4*)(job.C + (long)row * job.N + col) = *(const u32x4*)(patch + patch_at<kRowBytes>(rl, c0));
      }
    }
    if (!more) return;
    stores_out = my_rows == WBM && job.m0 + TM <= job.M && job.n0 + TN <= job.N;
    job = next;
  }
}

template <int WBM, int WBN>
static int32_t launch_dw(DwParams p, double rows, const ProfRoles& roles, hipStream_t st) {
  const int tiles = p.E * p.per_expert;
  // Several tiles per workgroup where a tile is short and the chip is filled many times, else one; read ahead there and where tiles
  // are long; runs of 32 there if there are many, else of 16.  us, four tiles in runs of 32 / one ahead in runs of 16, of 32 / one in the plain loop (H F, experts;
  // rows per expert):
  //   2048 1024, 32       128: 126 / 135, 133 / 133     512: 238 / 243, 246 / 247     1024: 392 / 389, 389 / 389     1536: 553 / 544, 542 / 554
  //   1024 1024, 64        64: 105 / 111, 113 / 108     512: 259 / 254, 262 / 256     1024: 426 / 401, 419 / 403
  //   2048 4096, 8        200: 142 / 152, 152 / 151     700: 286 / 288, 290 / 289     1024: 377 / 385, 387 / 384     1300: 454 / 459, 464 / 455
  //   4096 688, 16       2048: 538 / 511, 522 / 541, with four slots per token - / 506, 501 / -     (four tiles in runs of 16: 569; up to 5 %
  //                            slower than of 32 everywhere but at 1024 1024)
  //   4096 2048, 8        875: 322 / 330, - / -
  //   2048 1024, 16 (3072 tiles)   300: 92 / 88, 88 / 87     1000: 201 / 191, 196 / 193     3328 1152, 7 (2457)   1941: - / 266, - / 279
  // On 128 x 128 tiles the plain loop is the faster one at all lengths (1152 768, 6 experts, 528 rows: 31.9 / 30.0; 184 9216, 2, 11221: 478 /
  // 478), as on 64 x 64 (128 4736, 1, 2608: 25.4 / 22.7).
  p.walk = WBN == 8 && tiles >= 4096 && rows <= 896.0 * p.E ? 4 : 1;
  const bool ahead = p.walk > 1 || rows > 1400.0 * p.E;
  p.list = tile_list(tiles, WBN == 8 && ahead && tiles >= 4096 ? 32 : 16, p.walk);
  const dim3 grid(p.list.blocks);
  if constexpr (WBN == 8) {
    if (ahead) {
      DYNMO_TIMED_LAUNCH(roles, st, ffn_dw_kernel<WBM, WBN, true><<<grid, dim3(kDwThreads), 0, st>>>(p));
      return DYNMO_OK;
    }
  }
  DYNMO_TIMED_LAUNCH(roles, st, ffn_dw_kernel<WBM, WBN, false><<<grid, dim3(kDwThreads), 0, st>>>(p));
  return DYNMO_OK;
}

int32_t ffn_dw_tiles(TileKind kind, const dynmo_desc* d, const int32_t* seg, const bf16_t* dy_p, const bf16_t* x_p,
                     const bf16_t* A, const bf16_t* dG, const bf16_t* dU, bf16_t* dWg, bf16_t* dWu, bf16_t* dWd, hipStream_t st) {
  if (kind != TILE_128x256 && kind != TILE_128 && kind != TILE_64) return DYNMO_EINVAL;
  const int E = d->E, H = d->H, F = d->F;
  const int r = kind == TILE_64 ? 64 : 128, c = kind == TILE_64 ? 64 : kind == TILE_128 ? 128 : 256;
  const int hf = ((H + r - 1) / r) * ((F + c - 1) / c), fh = ((F + r - 1) / r) * ((H + c - 1) / c);
  const DwSet all[3] = {{dy_p, A, dWd, H, F, hf}, {dG, x_p, dWg, F, H, fh}, {dU, x_p, dWu, F, H, fh}};
  const KernelId ids[3] = {K_FFN_DWD, K_FFN_DWG, K_FFN_DWU};
  DwParams p = {};
  p.seg = seg;
  p.E = E;
  // One launch for the three products; one each if a gradient is to be written over the rows
  const double routed = (double)d->T * d->k;
  const size_t rows = (size_t)d->T * d->k * H * 2, weights = (size_t)E * F * H * 2;
  p.sets = any_overlap({{dWd, weights}, {dWg, weights}, {dWu, weights}}, {{dy_p, rows}, {x_p, rows}}) ? 1 : 3;
  for (int s = 0; s < 3; s += p.sets) {
    p.per_expert = 0;
    ProfRoles roles;  // equal flops
    for (int i = 0; i < p.sets; ++i) {
      p.dw[i] = all[s + i];
      p.per_expert += all[s + i].tiles;
      roles.add(ids[s + i], 1.0);
    }
    const int32_t rc = kind == TILE_128x256 ? launch_dw<4, 8>(p, routed, roles, st)
                       : kind == TILE_128   ? launch_dw<4, 4>(p, routed, roles, st)
                                            : launch_dw<2, 2>(p, routed, roles, st);
    if (rc) return rc;
  }
  return DYNMO_OK;
}

}  // namespace dynmo
