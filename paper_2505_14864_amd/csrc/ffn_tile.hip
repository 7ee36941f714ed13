// Grouped SwiGLU FFN on the gfx950 matrix cores (bf16 in, fp32 accumulate): the kernel for row-segmented
// products that are too small, or cut into too many short pieces, for the 256 x 256 tiles of ffn_mfma.hip.
//
// One workgroup of four wavefronts (2 x 2) per output tile of 128 x 256 (64 x 128 per wavefront), 128 x 128
// (64 x 64) or 64 x 64 (32 x 32), not persistent: the hardware deals the workgroups, and two (three, three) of
// them share a compute unit, so that one's prologue and epilogue run under the other's matrix instructions.
// The 256 x 256 kernel keeps one workgroup per compute unit and cannot overlap them; it needs two thirds of the L2
// traffic per MFMA and wins where a tile's k range is long and the tiles fill the chip.
//
// k goes in steps of 32 (one MFMA deep) through a ring of three LDS stages of one step (64 x 64: two); buffer loads with an
// LDS destination fill a stage two stages before it is read.  Two steps per barrier cost 64 x 64 tiles two of five workgroups per
// compute unit and gain on every product all the same, also where a handful of rows waits for weights out of HBM (one step in
// four stages / two in three, us; rows x H x F, experts): dX 16 x 1024 x 2048, 8 22.8 / 21.2, 64 x 2048 x 2048, 4 29.4 / 26.5, 256 x
// 1024 x 1024, 1 15.0 / 14.2; dA 32 x 4096 x 4096, 1 22.5 / 19.8; gate/up and down 0 to 4 %, none of 44 slower by more than 1 %.  Deeper rings are no faster (64 x 64 tiles, eight stages of one step: 0 to
// 7 % slower), nor are two steps per stage of 128 x 128 (0 to 20 % slower: a workgroup less per compute unit).  Operands that lie [row][k] in memory
// keep that layout in LDS, operands that lie [k][row] are read with ds_read_b64_tr_b16; 16-byte pieces
// are placed so that the lanes that the hardware serves together fall into different banks (placed for the sixteen lanes of a k group
// instead, 22 to 44 % of the LDS cycles were conflicts, and down of 64 experts took 112 us instead of 109).
//   [row][k]: 64 bytes per row; the piece with k = 8 c .. of row r sits at r * 64 + ((c ^ (0, 2, 3, 1)[(r >> 2) & 3]) << 4)
//   [k][row]: 64-byte blocks of 32 rows; block b of k-row k is stored as block b ^ (k & 3) (64 rows:
//             b ^ ((k >> 1) & 1)), its two 32-byte halves swapped when bit 3 of k is set
#include "ffn_gemm.h"
#include "tile_list.h"

namespace dynmo {

constexpr int kTileThreads = 256;

struct TileParams {
  GemmParams g;
  TileList list;
};

// WBM x WBN blocks of 16 x 16 per wavefront
template <int WBM, int WBN>
struct TileShape {
  static constexpr int kRows = 32 * WBM, kCols = 32 * WBN;  // of the output tile
  static constexpr int kSteps = WBN == 2 ? 2 : 1;  // k steps per stage, and per barrier
  static constexpr int kStages = 3;
  static constexpr int kBytesA = kRows * kTileK * 2, kBytesB = kCols * kTileK * 2;
  static constexpr int kStep = kBytesA + kBytesB, kStage = kSteps * kStep;
  static constexpr int kPiecesA = kBytesA / 4096, kPiecesB = kBytesB / 4096;  // pieces of 1 KB a wavefront loads per stage
  static constexpr int kLoads = kPiecesA + kPiecesB;
  static constexpr int kPitch = 16 * WBN + 4;           // floats per row of an epilogue patch
  static constexpr int kPatchBytes = 16 * kPitch * 4;
  static constexpr int kLds = kStages * kStage;
  static_assert(4 * kPatchBytes <= kLds, "the epilogue patches reuse the stages");
};

// [row][k]: what the slot of a 16-byte piece is mixed with, by (row / 4) % 4: 0, 2, 3, 1.  The hardware serves a 16-byte read
// in groups of sixteen lanes, 0..3, 12..15, 20..27 the first: rows 0..3 and 12..15 of one k group, 4..11 of the next.
__device__ __forceinline__ int rowk_swizzle(int quad) { return ((quad << 1) & 2) ^ ((quad >> 1) * 3); }

// Byte offsets, from the tile's (row 0, k 0) element, of the 16 bytes this lane moves in each of the
// wavefront's pieces (kOob: nothing), and their k where that needs a mask.
template <int ROWS, bool KROW>
struct TilePieces {
  static constexpr int N = ROWS * kTileK * 2 / 4096;
  uint32_t off[N];
  int kpos[N];  // [row][k]

  // [row][k]: a piece is 16 rows; WRAP: rows from there on are rows 0.. of a second matrix
  __device__ __forceinline__ void init(uint32_t ld_bytes, int rows_left, int wrap, const int32_t* __restrict__ rowmap, int rowdiv) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int q = wave * N + j;
      if constexpr (!KROW) {
        const int lrow = q * 16 + (lane >> 2), c = (lane & 3) ^ rowk_swizzle(lane >> 4);
        int row = lrow % wrap;
        const bool ok = row < rows_left;
        if (rowmap != nullptr) row = ok ? rowmap[row] / rowdiv : 0;
        off[j] = ok ? (uint32_t)row * ld_bytes + c * 16 : kOob;
        kpos[j] = c * 8;
      } else {
        off[j] = krow_piece<ROWS>(q, lane, ld_bytes, rows_left);
      }
    }
  }
};

// LDS byte offsets (inside an operand's stage) from which this lane reads its fragments: lane l holds, for row
// l % 16 of a 16-row block, the eight k values (l / 16) * 8 .. + 7.
template <int ROWS, bool KROW>
__device__ __forceinline__ uint32_t frag_offset(int block16) {
  const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
  if constexpr (!KROW) {
    return (block16 * 16 + s) * 64 + ((g ^ rowk_swizzle(s >> 2)) << 4);
  } else {
    return krow_frag<ROWS>(lane, block16);
  }
}

typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;

template <int ROWS, bool KROW>
__device__ __forceinline__ bf16x8_t read_tile_frag(uint32_t addr) {
  if constexpr (!KROW) {
    return *(const lds_bf16x8_t*)(uintptr_t)addr;
  } else {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(uintptr_t)addr);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(uintptr_t)(addr + 4 * ROWS * 2));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

template <int MODE, int WBM, int WBN, bool WHOLE_K>
__global__ __launch_bounds__(kTileThreads, WBN == 8 ? 2 : 3) void ffn_tile_kernel(const TileParams tp) {
  using S = TileShape<WBM, WBN>;
  __shared__ __attribute__((aligned(1024))) char smem[S::kLds];
  constexpr bool IS_DX = MODE == MODE_DX || MODE == MODE_DX_FOLD;
  constexpr bool FOLDS = MODE == MODE_DOWN_FOLD || MODE == MODE_DX_FOLD;
  constexpr bool B_KROW = MODE == MODE_DA || IS_DX;
  constexpr int TM = S::kRows, TILE_N = MODE == MODE_GATEUP ? S::kCols / 2 : S::kCols;
  const GemmParams& p = tp.g;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // ---- which tile
  // lane e of every wavefront counts the row tiles of expert e; a prefix sum and a ballot find the owner
  const int nt = (p.N + TILE_N - 1) / TILE_N;
  const int begin = lane < p.E ? p.seg[lane] : 0, end = lane < p.E ? p.seg[lane + 1] : 0;
  const int mt = (end - begin + TM - 1) / TM;
  int upto = mt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(upto, d, 64);
    if (lane >= d) upto += o;
  }
  const int total = __builtin_amdgcn_readlane(upto, 63) * nt;
  const int pos = list_position(tp.list, blockIdx.x, total, TM, S::kCols, p.E, __ballot(mt > 1) == 0);
  const unsigned long long owners = __ballot(upto * nt > pos);
  if (owners == 0) return;  // past the last tile
  const int e = __builtin_ctzll(owners);
  const int mt_e = __builtin_amdgcn_readlane(mt, e);
  int mi, ni;
  tile_of(pos - (__builtin_amdgcn_readlane(upto, e) - mt_e) * nt, mt_e, nt, &mi, &ni);
  const int m0 = __builtin_amdgcn_readlane(begin, e) + mi * TM, m_end = __builtin_amdgcn_readlane(end, e);
  const int n0 = ni * TILE_N, n_end = p.N;
  bf16_t* const C0 = p.C0;
  const long lda = p.lda, ldb = p.ldb, ldc = p.ldc;

  // ---- operands
  const uint32_t lda_b = (uint32_t)lda * 2, ldb_b = (uint32_t)ldb * 2;
  const bool gathered = MODE == MODE_GATEUP && p.gather != nullptr;
  const bool second_b = MODE == MODE_GATEUP && wave >= 2;  // operand B: gate rows, then the matching up rows
  TilePieces<S::kRows, false> pa;
  TilePieces<S::kCols, B_KROW> pb;
  pa.init(lda_b, m_end - m0, S::kRows, gathered ? p.gather + m0 : nullptr, p.gather_div);
  pb.init(ldb_b, n_end - n0, TILE_N, nullptr, 1);
  const long b_off = (long)e * p.b_expert_stride;
  auto a_at = [&](const bf16_t* A, int k) { return A + (gathered ? 0 : (long)m0 * lda) + k; };
  auto b_at = [&](const bf16_t* B, int k) { return B_KROW ? B + b_off + (long)k * ldb + n0 : B + b_off + (long)n0 * ldb + k; };
  const int kt_phase = (p.K + kTileK - 1) / kTileK;
  const int n_kt = kt_phase * (IS_DX ? 2 : 1);
  const bf16_t* na = a_at(p.A1, 0);
  const bf16_t* nb = b_at(second_b ? p.B2 : p.B1, 0);
  int k_left = p.K, issued = 0;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  // the next k step into the stage at byte `stage`; past the last one the loads fetch nothing
  auto issue = [&](uint32_t stage) {
    const int left = issued < n_kt ? k_left : 0;
    const uint32_t k_rows = (uint32_t)max(0, min(left, kTileK));
    const uint32_t any = left > 0 ? 0x7ffffffeu : 0u;
    // a [k][row] operand's k-rows are whole records, so the record count is its k mask
    const desc_t da = make_desc(na, any), db = make_desc(nb, B_KROW ? k_rows * ldb_b : any);
    const uint32_t to_a = __builtin_amdgcn_readfirstlane(lds0 + stage + wave * S::kPiecesA * 1024);
    const uint32_t to_b = __builtin_amdgcn_readfirstlane(lds0 + stage + wave * S::kPiecesB * 1024);
    static_for<S::kPiecesA>([&](auto J) {
      constexpr int j = decltype(J)::value;
      load_to_lds<j * 1024>(da, to_a, WHOLE_K || pa.kpos[j] < left ? pa.off[j] : kOob);
    });
    static_for<S::kPiecesB>([&](auto J) {
      constexpr int j = decltype(J)::value;
      load_to_lds<S::kBytesA + j * 1024>(db, to_b, B_KROW || WHOLE_K || pb.kpos[j] < left ? pb.off[j] : kOob);
    });
    ++issued;
    na += kTileK;
    nb += B_KROW ? (long)kTileK * ldb : kTileK;
    k_left -= kTileK;
    if (IS_DX && issued == kt_phase) {  // the second phase: dU Wu
      na = a_at(p.A2, 0);
      nb = b_at(p.B2, 0);
      k_left = p.K;
    }
  };

  // ---- fragments.  Wavefront (wm, wn): 16-row blocks wm, wm + 2, .. of the tile (in a ragged tile the valid
  // rows are a prefix, and every wavefront keeps its share) and columns 16 WBN wn .. .
  uint32_t fa[WBM], fb[WBN];
#pragma unroll
  for (int i = 0; i < WBM; ++i) fa[i] = lds0 + frag_offset<S::kRows, false>(wm + 2 * i);
#pragma unroll
  for (int j = 0; j < WBN; ++j) {
    const int n16 = MODE != MODE_GATEUP ? wn * WBN + j : j < WBN / 2 ? wn * (WBN / 2) + j : WBN + wn * (WBN / 2) + j - WBN / 2;
    fb[j] = lds0 + S::kBytesA + frag_offset<S::kCols, B_KROW>(n16);
  }
  const int valid16 = min(2 * WBM, (m_end - m0 + 15) / 16);
  const bool cols_ok = n0 + wn * (TILE_N / 2) < n_end;
  const int my_rows = cols_ok && valid16 > wm ? (valid16 - wm + 1) / 2 : 0;  // row blocks with work

  f32x4_t acc[WBM][WBN] = {};
  for (int s = 0; s < (S::kStages - 1) * S::kSteps; ++s) issue(s * S::kStep);
  auto loop = [&](auto ROWS_C) {
    constexpr int ROWS = decltype(ROWS_C)::value;
    uint32_t stage = 0, freed = (S::kStages - 1) * S::kStage;  // the stage read, the stage filled
    for (int kt = 0; kt < n_kt; kt += S::kSteps) {
      // this wavefront's share of the stage has landed and its reads of the previous stage are done; behind
      // the barrier that holds for all
      wait_stage<(S::kStages - 2) * S::kSteps * S::kLoads>();
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int h = 0; h < S::kSteps; ++h) issue(freed + h * S::kStep);
      if constexpr (ROWS > 0) {
        bf16x8_t a[S::kSteps][WBM], b[S::kSteps][WBN];
#pragma unroll
        for (int h = 0; h < S::kSteps; ++h) {
#pragma unroll
          for (int i = 0; i < ROWS; ++i) a[h][i] = read_tile_frag<S::kRows, false>(fa[i] + stage + h * S::kStep);
#pragma unroll
          for (int j = 0; j < WBN; ++j) b[h][j] = read_tile_frag<S::kCols, B_KROW>(fb[j] + stage + h * S::kStep);
        }
#pragma unroll
        for (int h = 0; h < S::kSteps; ++h)
#pragma unroll
          for (int j = 0; j < WBN; ++j)
#pragma unroll
            for (int i = 0; i < ROWS; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[h][i], b[h][j], acc[i][j], 0, 0, 0);
      }
      freed = stage;
      stage = stage + S::kStage == S::kLds ? 0 : stage + S::kStage;
    }
  };
  if (my_rows == WBM) loop(std::integral_constant<int, WBM>{});
  else if (my_rows == 0) loop(std::integral_constant<int, 0>{});
  else if (WBM == 2 || my_rows == 1) loop(std::integral_constant<int, 1>{});
  else if constexpr (WBM == 4) {
    if (my_rows == 2) loop(std::integral_constant<int, 2>{});
    else loop(std::integral_constant<int, 3>{});
  }
  wait_stage<0>();  // every load (masked ones included) has landed
  __builtin_amdgcn_s_barrier();

  // ---- epilogue.  A wavefront passes sixteen rows at a time through its own LDS patch (fp32), so that global
  // memory sees 16-byte accesses along rows; no barrier, a wavefront's LDS accesses complete in order.
  float* ep = (float*)(smem + wave * S::kPatchBytes);
  constexpr int kLanesPerRow = 16 * WBN / 8 / (MODE == MODE_GATEUP ? 2 : 1);
  constexpr int kRowsPerPass = 64 / kLanesPerRow < 16 ? 64 / kLanesPerRow : 16;
  constexpr int kPasses = 16 / kRowsPerPass;
  const int c0 = lane % kLanesPerRow * 8;
  const int col = n0 + wn * (TILE_N / 2) + c0;
#pragma unroll
  for (int i = 0; i < WBM; ++i) {
    if (i >= my_rows) break;
    const int band = m0 + (2 * i + wm) * 16;
    bool ok[kPasses];
    long at[kPasses];
#pragma unroll
    for (int s = 0; s < kPasses; ++s) {
      const int rl = s * kRowsPerPass + lane / kLanesPerRow;
      ok[s] = rl < 16 && band + rl < m_end && col < n_end;
      at[s] = (long)(band + rl) * ldc + col;
    }
    // what the stores need from global memory is asked for before the LDS pass
    u32x4 g_[kPasses], u_[kPasses];
    if constexpr (MODE == MODE_DA) {
#pragma unroll
      for (int s = 0; s < kPasses; ++s) {
        g_[s] = u_[s] = u32x4{0u, 0u, 0u, 0u};
        if (ok[s]) {
          g_[s] = *(const u32x4*)(p.G + at[s]);
          u_[s] = *(const u32x4*)(p.U + at[s]);
        }
      }
    }
    int token[kPasses];
    if constexpr (FOLDS) {
#pragma unroll
      for (int s = 0; s < kPasses; ++s) token[s] = ok[s] ? p.scatter[band + s * kRowsPerPass + lane / kLanesPerRow] : 0;
    }
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) ep[((lane >> 4) * 4 + r) * S::kPitch + j * 16 + (lane & 15)] = acc[i][j][r];
    float weight[kPasses];
    u32x4 resid[kPasses];
    if constexpr (FOLDS) {
#pragma unroll
      for (int s = 0; s < kPasses; ++s) {
        weight[s] = ok[s] && p.scale ? p.scale[token[s]] : 1.f;
        resid[s] = u32x4{0u, 0u, 0u, 0u};
        if (ok[s] && p.res) resid[s] = *(const u32x4*)(p.res + (long)token[s] * ldc + col);
      }
    }
#pragma unroll
    for (int s = 0; s < kPasses; ++s) {
      if (!ok[s]) continue;
      const float* row = ep + (s * kRowsPerPass + lane / kLanesPerRow) * S::kPitch + c0;
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = row[q];
      if constexpr (MODE == MODE_GATEUP) {
        float u[8], a_[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          u[q] = row[8 * WBN + q];
          a_[q] = silu_mul(v[q], u[q]);
        }
        *(u32x4*)(C0 + at[s]) = pack16<bf16_t>(v);
        *(u32x4*)(p.C1 + at[s]) = pack16<bf16_t>(u);
        *(u32x4*)(p.C2 + at[s]) = pack16<bf16_t>(a_);
      } else if constexpr (MODE == MODE_DA) {
        float g[8], u[8], a_[8], dg[8], du[8];
        unpack16<bf16_t>(g_[s], g);
        unpack16<bf16_t>(u_[s], u);
#pragma unroll
        for (int q = 0; q < 8; ++q) swiglu_bwd_bf16(v[q], g[q], u[q], &a_[q], &dg[q], &du[q]);
        *(u32x4*)(C0 + at[s]) = pack16<bf16_t>(dg);
        *(u32x4*)(p.C1 + at[s]) = pack16<bf16_t>(du);
        *(u32x4*)(p.C2 + at[s]) = pack16<bf16_t>(a_);
      } else {
        if (!FOLDS || C0) *(u32x4*)(C0 + at[s]) = pack16<bf16_t>(v);
        if constexpr (FOLDS) {
          float r[8];
          unpack16<bf16_t>(resid[s], r);
#pragma unroll
          for (int q = 0; q < 8; ++q) r[q] += weight[s] * v[q];
          *(u32x4*)(p.out + (long)token[s] * ldc + col) = pack16<bf16_t>(r);
        }
      }
    }
  }
}

template <int MODE, int WBM, int WBN>
static int32_t launch_tile(TileParams tp, int tiles, const ProfRoles& id, hipStream_t st) {
  tp.list = tile_list(tiles);
  if (tp.g.K % kTileK == 0) {
    DYNMO_TIMED_LAUNCH(id, st, ffn_tile_kernel<MODE, WBM, WBN, true><<<dim3(tp.list.blocks), dim3(kTileThreads), 0, st>>>(tp));
    return DYNMO_OK;
  }
  DYNMO_TIMED_LAUNCH(id, st, ffn_tile_kernel<MODE, WBM, WBN, false><<<dim3(tp.list.blocks), dim3(kTileThreads), 0, st>>>(tp));
  return DYNMO_OK;
}

template <int MODE>
static int32_t launch_shape(TileKind kind, const TileParams& tp, int tiles, const ProfRoles& id, hipStream_t st) {
  switch (kind) {
    case TILE_128x256:
      if constexpr (MODE == MODE_GATEUP) return DYNMO_EINVAL;  // never picked
      else return launch_tile<MODE, 4, 8>(tp, tiles, id, st);
    case TILE_128: return launch_tile<MODE, 4, 4>(tp, tiles, id, st);
    case TILE_64: return launch_tile<MODE, 2, 2>(tp, tiles, id, st);
    default: return DYNMO_EINVAL;
  }
}

static int rows_of(TileKind kind) { return kind == TILE_64 ? 64 : 128; }
static int cols_of(TileKind kind) { return kind == TILE_64 ? 64 : kind == TILE_128 ? 128 : 256; }

int32_t ffn_tile_rows(int mode, TileKind kind, const dynmo_desc* d, const GemmParams& p, KernelId id, hipStream_t st) {
  const int row_tiles = max_m_tiles(d, rows_of(kind));
  if (row_tiles <= 0) return DYNMO_OK;
  TileParams tp = {};
  tp.g = p;
  const int cols = cols_of(kind) / (mode == MODE_GATEUP ? 2 : 1);
  const int tiles = row_tiles * ((p.N + cols - 1) / cols);
  switch (mode) {
    case MODE_GATEUP: return launch_shape<MODE_GATEUP>(kind, tp, tiles, id, st);
    case MODE_DOWN: return launch_shape<MODE_DOWN>(kind, tp, tiles, id, st);
    case MODE_DOWN_FOLD: return launch_shape<MODE_DOWN_FOLD>(kind, tp, tiles, id, st);
    case MODE_DA: return launch_shape<MODE_DA>(kind, tp, tiles, id, st);
    case MODE_DX: return launch_shape<MODE_DX>(kind, tp, tiles, id, st);
    case MODE_DX_FOLD: return launch_shape<MODE_DX_FOLD>(kind, tp, tiles, id, st);
  }
  return DYNMO_EINVAL;
}

}  // namespace dynmo
