// Grouped SwiGLU FFN in fp32 on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands,
// fp32 accumulate, no conversion anywhere).
//
// One device routine serves the five products of the layer; an operand is described by how
// it lies in memory: K contiguous ([row][k]: activations and the forward's weights) or rows
// contiguous ([k][row]: the backward's weights and both operands of a weight gradient).
//
// Bound: the fp32 matrix rate is a sixteenth of the bf16 one (one 16x16x4 MFMA occupies its
// SIMD for 32 cycles and needs one dword per lane and operand), so neither LDS nor L2
// bandwidth is near its limit even for a 64x64 tile; what costs is latency.  Hence small
// tiles and several workgroups per compute unit (36 KB of LDS each): 64x64 outputs, four
// wavefronts of 32x32 (2x2 blocks), k in steps of 32 through two LDS stages, with two
// further k tiles on their way in registers; products of few such tiles take 32x32 outputs,
// a block per wavefront, with four k tiles on their way.  Vector fp32 instructions reach half of the
// MFMA rate at best.
//
// Measured against a 64x64 vector-ALU kernel with one k step of 16 in flight:
//   T=1500 H=516 F=1030 E=8 k=2   gate/up 275 -> 96 us, down 242 -> 61, dA 151 -> 61, dX 467 -> 105, dW 179 -> 50 each
//                                 (52 to 66 TFLOP/s; a large dense fp32 product of the vendor's library: 142)
//   T=256 H=128 F=256 E=4 k=2     gate/up 40 -> 8 us, down 37 -> 11, dA 26 -> 12, dX 74 -> 16, dW 31 -> 6 each
#include <type_traits>

#include "common.h"
#include "f32_grid.h"
#include "ffn.h"
#include "profile.h"

namespace dynmo {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int TK = 32;         // k step
constexpr int kThreads = 256;  // 2 x 2 wavefronts
// Output tiles of 32 NB x 32 NB: NB x NB blocks of 16 x 16 per wavefront, NB 16-byte chunks of either operand per thread and k step.
template <int NB>
constexpr int kTile = 32 * NB;
// k steps on their way in registers
template <int NB>
constexpr int kSets = NB == 1 ? 4 : 2;
// LDS layouts of an operand tile (64 rows x 32 k).  [row][k]: 36 floats per row, so that the
// 16-byte reads of sixteen rows fall into sixteen different bank groups (36 s mod 64).
// [k][row]: 68 floats per k-row, so that k-rows 4 apart -- the four lane groups of a fragment
// -- are 16 banks apart.  Share of the LDS cycles that are conflicts all the same: 32 % with two [row][k] operands, 16 %
// with one, 7 % in the gradients; the matrix units wait for little of it (busy 55 to 76 % of the cycles).
constexpr int kPitchRowK = TK + 4;
template <int NB>
constexpr int kPitchKRow = kTile<NB> + 4;
template <int NB>
constexpr int kOperandFloats = kTile<NB> * kPitchRowK > TK * kPitchKRow<NB> ? kTile<NB> * kPitchRowK : TK * kPitchKRow<NB>;
constexpr uint32_t kOutside = 0x80000000u;  // an offset beyond every record count: the load delivers zero

// A workgroup's place in its grid
struct Place {
  bool list;
  unsigned x, y, z, width;
  __device__ __forceinline__ static Place here(bool list) { return {list, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x}; }
};

// The row tile and column tile of a workgroup; false if it has none.  Lane e of every wavefront counts the tiles of
// expert e and a prefix sum and a ballot find the owner: one load latency, however many experts.
struct RowTile {
  int e, m0, m_end;
};
template <int NB>
__device__ __forceinline__ bool find_tile(const int32_t* __restrict__ seg, int E, const Place& w, int64_t cols, RowTile* t, int* col) {
  const int lane = threadIdx.x & 63;
  const int begin = lane < E ? seg[lane] : 0, end = lane < E ? seg[lane + 1] : 0;
  const int n = (end - begin + kTile<NB> - 1) / kTile<NB>;
  int upto = n;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(upto, d, 64);
    if (lane >= d) upto += o;
  }
  int row = 0;
  if (!tile_of_workgroup(w.list, w.x, w.y, w.z, w.width, __builtin_amdgcn_readlane(upto, 63), cols, &row, col)) return false;
  t->e = __builtin_ctzll(__ballot(upto > row));
  t->m0 = __builtin_amdgcn_readlane(begin, t->e) + (row - __builtin_amdgcn_readlane(upto - n, t->e)) * kTile<NB>;
  t->m_end = __builtin_amdgcn_readlane(end, t->e);
  return true;
}

// One operand of a product: the tile's rows by k.
//   KROW = false: element (row, k) at base + row * ld + k, with `rows` valid rows.  With `rowmap`, row r is row
//     rowmap[r] / rowdiv.  PAIR: LDS rows 0..31 are 32 rows of one matrix and rows 32..63 the same rows of
//     another one (`base2`): every thread's first chunk then belongs to the one and its second to the other.
//   KROW = true: element (row, k) at base + k * ld + row.
// VEC = floats per load: the largest of 4, 2, 1 that divides ld (and so every offset and limit).
// WIDE: a tile may span 2 GiB and more (64 rows of at least 2^23 floats), where the 32-bit offsets and the record
// count of a buffer load end; the loads are then ordinary ones from 64-bit addresses.
template <int NB, bool KROW, int VEC, bool WIDE, bool PAIR = false>
struct Operand {
  using offset_t = std::conditional_t<WIDE, long, uint32_t>;
  const float *base, *base2;  // (row 0, k 0) of the tile, wave-uniform
  long ld;
  offset_t off[NB];   // byte offsets of this thread's chunks of four floats, from (row 0, k 0 of the k tile)
  int kpos[NB];       // their k inside the k tile
  int left[NB];       // [k][row]: valid floats from there on (<= 0: none); [row][k]: valid row or not

  static constexpr int kFloats = kOperandFloats<NB>;
  static_assert(!PAIR || NB == 2, "every thread's first chunk belongs to one matrix of a pair and its second to the other");

  __device__ __forceinline__ void init(const float* b, long ld_, int rows, const float* b2 = nullptr,
                                       const int32_t* rowmap = nullptr, int rowdiv = 1) {
    base = b;
    base2 = b2;
    ld = ld_;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int c = threadIdx.x + i * kThreads;
      if constexpr (KROW) {
        kpos[i] = c / (kTile<NB> / 4);
        const int row = c % (kTile<NB> / 4) * 4;
        off[i] = (offset_t)(kpos[i] * ld + row) * 4;
        left[i] = rows - row;
      } else {
        kpos[i] = c % (TK / 4) * 4;
        int row = c / (TK / 4) - (PAIR && i ? kTile<NB> / 2 : 0);
        left[i] = row < rows;
        if (rowmap != nullptr) row = left[i] ? rowmap[row] / rowdiv : 0;
        off[i] = (offset_t)(row * ld + kpos[i]) * 4;
      }
    }
  }

  // the chunks of the k tile that starts at k0 (`k_left` valid k from there on); `shift`: floats to add to the base
  __device__ __forceinline__ void fetch(f32x4_t (&r)[NB], long k0, int k_left, long shift) const {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const float* p = (PAIR && i ? base2 : base) + shift + (KROW ? k0 * ld : k0);
      const bool ok = KROW ? kpos[i] < k_left : left[i] != 0;
      const int n = !ok ? 0 : KROW ? left[i] : k_left - kpos[i];  // valid floats of the chunk
      if constexpr (WIDE) {
        const float* q = (const float*)((const char*)p + off[i]);
        r[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if constexpr (VEC == 4) {
          if (n > 0) r[i] = *(const f32x4_t*)q;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (n > j) r[i][j] = q[j];
        }
        continue;
      }
      __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 0x7ffffffe, 0x00020000);
      if constexpr (VEC == 4) {
        r[i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(d, n > 0 ? off[i] : kOutside, 0, 0));
      } else if constexpr (VEC == 2) {
        const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(d, n > 0 ? off[i] : kOutside, 0, 0);
        const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(d, n > 2 ? off[i] + 8 : kOutside, 0, 0);
        r[i] = f32x4_t{__uint_as_float(lo.x), __uint_as_float(lo.y), __uint_as_float(hi.x), __uint_as_float(hi.y)};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          r[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(d, n > j ? off[i] + 4 * j : kOutside, 0, 0));
      }
    }
  }

  __device__ __forceinline__ void put(float* s, const f32x4_t (&r)[NB]) const {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int c = threadIdx.x + i * kThreads;
      const int at = KROW ? c / (kTile<NB> / 4) * kPitchKRow<NB> + c % (kTile<NB> / 4) * 4 : c / (TK / 4) * kPitchRowK + kpos[i];
      *(f32x4_t*)(s + at) = r[i];
    }
  }

  // The fragments of the 16-row block at `row16` for sixteen k from 16 kk on: lane l holds, for row l % 16, the
  // four k 4 (l / 16) .. + 3; MFMA j of the four that follow takes element j (both operands alike, so together
  // they cover the sixteen k, in an order that does not matter to the sum's terms).
  __device__ __forceinline__ static f32x4_t frag(const float* s, int row16, int kk) {
    const int lane = threadIdx.x & 63, row = row16 + (lane & 15), k = kk * 16 + (lane >> 4) * 4;
    if constexpr (!KROW) {
      return *(const f32x4_t*)(s + row * kPitchRowK + k);
    } else {
      f32x4_t f;
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = s[(k + j) * kPitchKRow<NB> + row];
      return f;
    }
  }
};

// acc[i][j] += sum over k of A(row block i) * B(row block j); the k range is `phases` stretches of K, the second
// one at (A + a_shift, B + b_shift).  Wavefront (wm, wn): A rows 32 wm + 16 i, B rows b_row[j].
template <int NA, int NB, typename OpA, typename OpB>
__device__ __forceinline__ void mac(f32x4_t (&acc)[NA][NB], const OpA& a, const OpB& b, int K, int phases, long a_shift,
                                    long b_shift, int a_row, const int (&b_row)[NB], float* lds) {
  constexpr int S = kSets<NA>, kStage = OpA::kFloats + OpB::kFloats;
  const int per_phase = (K + TK - 1) / TK, n_kt = per_phase * phases;
  if (n_kt == 0) return;
  f32x4_t ra[S][NA], rb[S][NB];  // k tiles on their way
  // past the last k tile nothing is fetched (zeros)
  auto fetch = [&](int kt, int set) {
    const bool second = kt >= per_phase && phases > 1;
    const int k0 = (second ? kt - per_phase : kt) * TK;
    const int k_left = kt < n_kt ? K - k0 : 0;
    a.fetch(ra[set], k0, k_left, second ? a_shift : 0);
    b.fetch(rb[set], k0, k_left, second ? b_shift : 0);
  };
  auto put = [&](int set, int stage) {
    a.put(lds + stage * kStage, ra[set]);
    b.put(lds + stage * kStage + OpA::kFloats, rb[set]);
  };
#pragma unroll
  for (int i = 0; i < S; ++i) fetch(i, i);
  put(0, 0);
  fetch(S, 0);
  __syncthreads();
  // k tile kt (= `at` modulo S) is in LDS stage kt % 2, tiles kt + 1 to kt + S are on their way
  auto step = [&](int kt, int at) {
    const int set = (at + 1) % S, stage = at % 2;
    put(set, 1 - stage);
    fetch(kt + 1 + S, set);
    __builtin_amdgcn_sched_barrier(0);  // the loads go out before the MFMAs, not when registers fall free
    const float* sa = lds + stage * kStage;
    const float* sb = sa + OpA::kFloats;
#pragma unroll
    for (int kk = 0; kk < TK / 16; ++kk) {
      f32x4_t fa[NA], fb[NB];
#pragma unroll
      for (int i = 0; i < NA; ++i) fa[i] = OpA::frag(sa, a_row + 16 * i, kk);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[j] = OpB::frag(sb, b_row[j], kk);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][q], fb[j][q], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  };
  int kt = 0;
  for (; kt + S <= n_kt; kt += S) {
#pragma unroll
    for (int i = 0; i < S; ++i) step(kt + i, i);
  }
#pragma unroll
  for (int i = 0; i < S - 1; ++i)
    if (kt + i < n_kt) step(kt + i, i);
}

// Position of this wavefront and lane in the output tile: block (i, j) holds rows row + 16 i + r, r = 0..3.
template <int NB>
struct OutPos {
  int wm, wn, row, col;
  __device__ __forceinline__ OutPos() {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wm = wave >> 1;
    wn = wave & 1;
    row = wm * 16 * NB + (lane >> 4) * 4;
    col = lane & 15;
  }
};

struct F32Params {
  const int32_t* seg;
  int E, H, F;
  const float *x, *dy, *G, *U, *A;  // inputs by name (A, dG, dU: written by one kernel, read by the next)
  const float *Wg, *Wu, *Wd;
  float *outG, *outU, *outA;        // GATEUP: G, U, A; DA: dG, dU, A
  float* C;                         // DOWN: y_p, DX: dx_p (may be nullptr when folded)
  const float *dG, *dU;
  float *dWg, *dWu, *dWd;
  const int32_t* gather;            // GATEUP: row p is x[gather[p] / gather_div], or nullptr
  int gather_div;
  FoldedCombine fold;               // scatter == nullptr: nothing folded
  bool list;                        // row products: the grid is a list (row_grid)
};

template <int NB>
__device__ __forceinline__ void store_row_product(const F32Params& p, const f32x4_t (&acc)[NB][NB], const RowTile& t, int n0,
                                                  int N) {
  const OutPos<NB> o;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = t.m0 + o.row + 16 * i + r;
      if (m >= t.m_end) continue;
      const int token = p.fold.scatter ? p.fold.scatter[m] : 0;
      const float scale = p.fold.scatter && p.fold.scale ? p.fold.scale[token] : 1.f;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = n0 + o.wn * 16 * NB + 16 * j + o.col;
        if (n >= N) continue;
        const float v = acc[i][j][r];
        if (p.C) p.C[(long)m * N + n] = v;
        if (p.fold.scatter) {
          const long at = (long)token * N + n;
          const float* res = (const float*)p.fold.res;
          ((float*)p.fold.out)[at] = (res ? res[at] : 0.f) + scale * v;
        }
      }
    }
}

constexpr int kPairCols = 32;  // columns of G and of U per tile
// G = X Wg^T, U = X Wu^T, A = silu(G) U: 32 NB rows x 32 columns of each.  LDS rows 0..31 of operand B are gate
// rows, 32..63 the matching up rows, and a wavefront takes sixteen of either.
template <int NB, bool WIDE>
__global__ __launch_bounds__(kThreads) void f32_gateup_kernel(const F32Params p) {
  __shared__ __attribute__((aligned(16))) float lds[2 * (kOperandFloats<NB> + kOperandFloats<2>)];
  RowTile t;
  int col = 0;
  if (!find_tile<NB>(p.seg, p.E, Place::here(p.list), tiles_of(p.F, kPairCols), &t, &col)) return;
  const int n0 = col * kPairCols;
  const long first = ((long)t.e * p.F + n0) * p.H;
  Operand<NB, false, 4, WIDE> a;
  Operand<2, false, 4, WIDE, true> b;
  if (p.gather) a.init(p.x, p.H, t.m_end - t.m0, nullptr, p.gather + t.m0, p.gather_div);
  else a.init(p.x + (long)t.m0 * p.H, p.H, t.m_end - t.m0);
  b.init(p.Wg + first, p.H, p.F - n0, p.Wu + first);
  f32x4_t acc[NB][2] = {};
  const OutPos<NB> o;
  const int b_row[2] = {o.wn * 16, 32 + o.wn * 16};
  mac(acc, a, b, p.H, 1, 0, 0, o.wm * 16 * NB, b_row, lds);
  const int n = n0 + o.wn * 16 + o.col;
  if (n >= p.F) return;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = t.m0 + o.row + 16 * i + r;
      if (m >= t.m_end) continue;
      const long at = (long)m * p.F + n;
      const float g = acc[i][0][r], u = acc[i][1][r];
      p.outG[at] = g;
      p.outU[at] = u;
      p.outA[at] = g * sigmoidf_(g) * u;
    }
}

// Y = A Wd^T
template <int NB, int VF, bool WIDE>
__global__ __launch_bounds__(kThreads) void f32_down_kernel(const F32Params p) {
  __shared__ __attribute__((aligned(16))) float lds[4 * kOperandFloats<NB>];
  RowTile t;
  int col = 0;
  if (!find_tile<NB>(p.seg, p.E, Place::here(p.list), tiles_of(p.H, kTile<NB>), &t, &col)) return;
  const int n0 = col * kTile<NB>;
  Operand<NB, false, VF, WIDE> a, b;
  a.init(p.A + (long)t.m0 * p.F, p.F, t.m_end - t.m0);
  b.init(p.Wd + ((long)t.e * p.H + n0) * p.F, p.F, p.H - n0);
  f32x4_t acc[NB][NB] = {};
  const OutPos<NB> o;
  int b_row[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) b_row[j] = o.wn * 16 * NB + 16 * j;
  mac(acc, a, b, p.F, 1, 0, 0, o.wm * 16 * NB, b_row, lds);
  store_row_product(p, acc, t, n0, p.H);
}

// dA = dY Wd; with the saved G, U: A, dG, dU
template <int NB, int VF, bool WIDE>
__global__ __launch_bounds__(kThreads) void f32_dA_kernel(const F32Params p) {
  __shared__ __attribute__((aligned(16))) float lds[4 * kOperandFloats<NB>];
  RowTile t;
  int col = 0;
  if (!find_tile<NB>(p.seg, p.E, Place::here(p.list), tiles_of(p.F, kTile<NB>), &t, &col)) return;
  const int n0 = col * kTile<NB>;
  Operand<NB, false, 4, WIDE> a;
  Operand<NB, true, VF, WIDE> b;
  a.init(p.dy + (long)t.m0 * p.H, p.H, t.m_end - t.m0);
  b.init(p.Wd + (long)t.e * p.H * p.F + n0, p.F, p.F - n0);
  f32x4_t acc[NB][NB] = {};
  const OutPos<NB> o;
  int b_row[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) b_row[j] = o.wn * 16 * NB + 16 * j;
  // what the stores need of G and U is on its way during the product (T=256 H=128 F=256: 12.4 -> 9.6 us)
  float g[NB][4][NB], u[NB][4][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int m = min(t.m0 + o.row + 16 * i + r, t.m_end - 1), n = min(n0 + b_row[j] + o.col, p.F - 1);
        g[i][r][j] = p.G[(long)m * p.F + n];
        u[i][r][j] = p.U[(long)m * p.F + n];
      }
  mac(acc, a, b, p.H, 1, 0, 0, o.wm * 16 * NB, b_row, lds);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = t.m0 + o.row + 16 * i + r;
      if (m >= t.m_end) continue;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = n0 + b_row[j] + o.col;
        if (n >= p.F) continue;
        const long at = (long)m * p.F + n;
        swiglu_bwd(acc[i][j][r], g[i][r][j], u[i][r][j], p.outA + at, p.outG + at, p.outU + at);
      }
    }
}

// dX = dG Wg + dU Wu, tile `tile` of the list (column tiles side by side)
template <int NB, int VF, bool WIDE>
__device__ __forceinline__ void input_grad(const F32Params& p, int tile, float* lds) {
  const unsigned th = (unsigned)tiles_of(p.H, kTile<NB>);
  RowTile t;
  int col = 0;
  const Place place = p.list ? Place{true, (unsigned)tile, 0, 0, 0} : Place{false, tile % th, tile / th, 0, th};
  if (!find_tile<NB>(p.seg, p.E, place, th, &t, &col)) return;
  const int n0 = col * kTile<NB>;
  Operand<NB, false, VF, WIDE> a;
  Operand<NB, true, 4, WIDE> b;
  a.init(p.dG + (long)t.m0 * p.F, p.F, t.m_end - t.m0);
  b.init(p.Wg + (long)t.e * p.F * p.H + n0, p.H, p.H - n0);
  f32x4_t acc[NB][NB] = {};
  const OutPos<NB> o;
  int b_row[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) b_row[j] = o.wn * 16 * NB + 16 * j;
  mac(acc, a, b, p.F, 2, p.dU - p.dG, p.Wu - p.Wg, o.wm * 16 * NB, b_row, lds);
  store_row_product(p, acc, t, n0, p.H);
}

// dW[m, n] = sum over the rows of an expert of P[row, m] Q[row, n]   (zeros if it has none)
template <int NB, int VM, int VN, bool WIDE>
__device__ __forceinline__ void weight_grad(const float* P, int M, const float* Q, int N, float* dW, int k_begin, int k_end,
                                            int m0, int n0, float* lds) {
  Operand<NB, true, VM, WIDE> a;
  Operand<NB, true, VN, WIDE> b;
  a.init(P + (long)k_begin * M + m0, M, M - m0);
  b.init(Q + (long)k_begin * N + n0, N, N - n0);
  f32x4_t acc[NB][NB] = {};
  const OutPos<NB> o;
  int b_row[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) b_row[j] = o.wn * 16 * NB + 16 * j;
  mac(acc, a, b, k_end - k_begin, 1, 0, 0, o.wm * 16 * NB, b_row, lds);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + o.row + 16 * i + r;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = n0 + b_row[j] + o.col;
        if (m < M && n < N) dW[(long)m * N + n] = acc[i][j][r];
      }
    }
}

// What follows dA, in one launch: nothing in it depends on anything else in it.  The list of tiles: dX, whose k ranges
// are long (2 F) and whose tiles are few, then dWd, dWg and dWu, which fill the compute units meanwhile.
//   T=1500 H=516 F=1030 E=8 k=2 (459 dX tiles, 3672 others):   four launches 242 us, one 204 (fp32 matrix rate: 131)
//   T=256 H=128 F=256 E=4 k=2 (24 and 96):                      36, 17
// This launch covers the list from `first` to `end`; `dx_tiles`, `dw_tiles`: tiles of dX and of each dW.
template <int NB, int VF, bool WIDE>
__global__ __launch_bounds__(kThreads) void f32_grads_kernel(const F32Params p, int first, int end, int dx_tiles, int dw_tiles) {
  __shared__ __attribute__((aligned(16))) float lds[4 * kOperandFloats<NB>];
  int r = first + (int)(blockIdx.y * gridDim.x + blockIdx.x);
  if (r >= end) return;
  if (r < dx_tiles) return input_grad<NB, VF, WIDE>(p, r, lds);
  r -= dx_tiles;
  const int which = r / dw_tiles;  // 0 = dWd (P = dY, Q = A), 1 = dWg (dG, x_p), 2 = dWu (dU, x_p)
  r -= which * dw_tiles;
  const int tf = (p.F + kTile<NB> - 1) / kTile<NB>, th = (p.H + kTile<NB> - 1) / kTile<NB>;
  const int e = r / (tf * th), tile = r - e * tf * th, width = which == 0 ? tf : th;
  const int m0 = tile / width * kTile<NB>, n0 = tile % width * kTile<NB>;
  const int k_begin = p.seg[e], k_end = p.seg[e + 1];
  const long FH = (long)p.F * p.H * e;
  if (which == 0) weight_grad<NB, 4, VF, WIDE>(p.dy, p.H, p.A, p.F, p.dWd + FH, k_begin, k_end, m0, n0, lds);
  else weight_grad<NB, VF, 4, WIDE>(which == 1 ? p.dG : p.dU, p.F, p.x, p.H, (which == 1 ? p.dWg : p.dWu) + FH, k_begin, k_end, m0, n0, lds);
}

// Which products go on tiles of 32 x 32 (gate/up: 32 rows), by how many tiles of 64 x 64 they have.  A k step of a 64 x 64 tile
// keeps its wavefronts' matrix units busy for 1024 cycles, and with few tiles that chain is the time of the product; with many the
// doubled traffic per flop weighs.  us on 64 / 32, tiles of 64 in brackets (T H F E k; times with the events around each launch):
//               256 128 256 4 2   303 256 768 5 3   1024 256 512 4 2   800 512 1024 4 2   1500 516 1030 8 2   2048 1024 1024 8 2
//   gate/up     10 /  8  (96)     19 / 17  (456)    25 / 22  (576)     47 / 42  (928)     88 /  90  (1782)   174 / 173  (2304)
//   down        13 /  8  (24)     24 / 12   (76)    19 / 15  (144)     31 / 26  (232)     58 /  55   (486)   102 /  87  (1152)
//   dA          11 /  7  (48)     14 / 13  (228)    20 / 16  (288)     30 / 28  (464)     59 /  60   (918)   103 /  97  (1152)
//   gradients   19 / 11 (120)     50 / 29  (796)    40 / 35  (528)     85 / 85 (1768)    183 / 217  (4158)   364 / 397  (7296)
constexpr int64_t kSmallGateup = 1024, kSmallDown = 1152, kSmallDA = 512, kSmallGrads = 1700;

static dim3 grid_of(F32Params& p, int64_t cols, int64_t rows) {
  const RowGrid g = row_grid(cols, rows);
  p.list = g.list;
  return dim3(g.x, g.y, g.z);
}

template <int NB, int VF, bool WIDE>
static int32_t gateup_f32(const dynmo_desc* d, F32Params p, hipStream_t st) {
  const dim3 grid = grid_of(p, tiles_of(d->F, kPairCols), max_m_tiles(d, kTile<NB>));
  DYNMO_TIMED_LAUNCH(K_FFN_GATEUP, st, f32_gateup_kernel<NB, WIDE><<<grid, dim3(kThreads), 0, st>>>(p));
  return DYNMO_OK;
}
template <int NB, int VF, bool WIDE>
static int32_t down_f32(const dynmo_desc* d, F32Params p, hipStream_t st) {
  const dim3 grid = grid_of(p, tiles_of(d->H, kTile<NB>), max_m_tiles(d, kTile<NB>));
  DYNMO_TIMED_LAUNCH(K_FFN_DOWN, st, f32_down_kernel<NB, VF, WIDE><<<grid, dim3(kThreads), 0, st>>>(p));
  return DYNMO_OK;
}
template <int NB, int VF, bool WIDE>
static int32_t dA_f32(const dynmo_desc* d, F32Params p, hipStream_t st) {
  const dim3 grid = grid_of(p, tiles_of(d->F, kTile<NB>), max_m_tiles(d, kTile<NB>));
  DYNMO_TIMED_LAUNCH(K_FFN_DA, st, f32_dA_kernel<NB, VF, WIDE><<<grid, dim3(kThreads), 0, st>>>(p));
  return DYNMO_OK;
}

template <int VF, bool WIDE>
static int32_t fwd_f32(const dynmo_desc* d, const F32Params& p, hipStream_t st) {
  const int64_t m_tiles = max_m_tiles(d, 64);
  if (m_tiles == 0) return DYNMO_OK;
  const bool small_g = !WIDE && m_tiles * tiles_of(d->F, kPairCols) <= kSmallGateup, small_d = !WIDE && m_tiles * tiles_of(d->H, 64) <= kSmallDown;
  const int32_t rc = small_g ? gateup_f32<1, VF, false>(d, p, st) : gateup_f32<2, VF, WIDE>(d, p, st);
  if (rc) return rc;
  return small_d ? down_f32<1, VF, false>(d, p, st) : down_f32<2, VF, WIDE>(d, p, st);
}

template <int NB, int VF, bool WIDE>
static int32_t grads_f32(const dynmo_desc* d, F32Params p, hipStream_t st) {
  const unsigned tf = (unsigned)tiles_of(d->F, kTile<NB>), th = (unsigned)tiles_of(d->H, kTile<NB>);
  // the weight gradients are written for every expert, rows or not
  int dx_tiles = (int)(th * max_m_tiles(d, kTile<NB>));
  const int dw_tiles = (int)(tf * th * d->E);
  p.list = dx_tiles <= kMaxList;
  if (p.list) dx_tiles = (dx_tiles + 7) / 8 * 8;
  auto launch = [&](const ProfRoles& roles, int first, int n) -> int32_t {
    if (n == 0) return DYNMO_OK;
    const int width = n < (int)kMaxWidth ? n : (int)kMaxWidth;
    DYNMO_TIMED_LAUNCH(roles, st, f32_grads_kernel<NB, VF, WIDE><<<dim3(width, (n + width - 1) / width), dim3(kThreads), 0, st>>>(
                                      p, first, first + n, dx_tiles, dw_tiles));
    return DYNMO_OK;
  };
  const KernelId ids[3] = {K_FFN_DWD, K_FFN_DWG, K_FFN_DWU};
  const size_t rows = (size_t)d->T * d->k * d->H * 4, tokens = (size_t)d->T * d->H * 4, weights = (size_t)d->E * d->F * d->H * 4;
  if (any_overlap({{p.dWd, weights}, {p.dWg, weights}, {p.dWu, weights}},
                  {{p.dy, rows}, {p.x, rows}, {p.Wg, weights}, {p.Wu, weights}, {p.fold.res, tokens}}) ||
      any_overlap({{p.C, rows}, {p.fold.out, tokens}}, {{p.dy, rows}, {p.x, rows}})) {
    // one after the other if one product's result is to be written over another's input
    int32_t rc = launch(K_FFN_DX, 0, dx_tiles);
    for (int s = 0; s < 3 && rc == DYNMO_OK; ++s) rc = launch(ids[s], dx_tiles + s * dw_tiles, dw_tiles);
    return rc;
  }
  ProfRoles roles;  // by flops
  if (dx_tiles > 0) roles.add(K_FFN_DX, 2.0);
  for (KernelId id : ids) roles.add(id, 1.0);
  return launch(roles, 0, dx_tiles + 3 * dw_tiles);
}

template <int VF, bool WIDE>
static int32_t bwd_f32(const dynmo_desc* d, const F32Params& p, hipStream_t st) {
  const int64_t m_tiles = max_m_tiles(d, 64), tf = tiles_of(d->F, 64), th = tiles_of(d->H, 64);
  if (m_tiles > 0) {
    const int32_t rc = !WIDE && m_tiles * tf <= kSmallDA ? dA_f32<1, VF, false>(d, p, st) : dA_f32<2, VF, WIDE>(d, p, st);
    if (rc) return rc;
  }
  return !WIDE && th * m_tiles + 3 * tf * th * d->E <= kSmallGrads ? grads_f32<1, VF, false>(d, p, st) : grads_f32<2, VF, WIDE>(d, p, st);
}

// Whether 64 rows of an operand can span 2 GiB (the rows of a gathered input as a whole stay below that)
static bool wide(const dynmo_desc* d) { return (d->H > d->F ? d->H : d->F) >= (1 << 23); }

static F32Params params_of(const dynmo_desc* d, const int32_t* seg, const void* Wg, const void* Wu, const void* Wd,
                           const FoldedCombine* fc) {
  F32Params p = {};
  p.seg = seg;
  p.E = d->E;
  p.H = d->H;
  p.F = d->F;
  p.Wg = (const float*)Wg;
  p.Wu = (const float*)Wu;
  p.Wd = (const float*)Wd;
  if (fc) p.fold = *fc;
  return p;
}

int32_t ffn_fwd_f32(const dynmo_desc* d, const void* x_p, const int32_t* gather, const int32_t* seg, const void* Wg,
                    const void* Wu, const void* Wd, void* y_p, void* G, void* U, void* A, const FoldedCombine* fc,
                    hipStream_t st) {
  F32Params p = params_of(d, seg, Wg, Wu, Wd, fc);
  p.x = (const float*)x_p;
  p.gather = gather;
  p.gather_div = d->k;
  p.outG = (float*)G;
  p.outU = (float*)U;
  p.outA = (float*)A;
  p.A = (const float*)A;
  p.C = (float*)y_p;
  // rows of length F can be loaded four, two or one float at a time, whichever divides F; H is a multiple of four
  if (wide(d)) return fwd_f32<1, true>(d, p, st);
  return d->F % 4 == 0 ? fwd_f32<4, false>(d, p, st) : d->F % 2 == 0 ? fwd_f32<2, false>(d, p, st) : fwd_f32<1, false>(d, p, st);
}

int32_t ffn_bwd_f32(const dynmo_desc* d, const void* dy_p, const void* x_p, const void* G, const void* U,
                    const int32_t* seg, const void* Wg, const void* Wu, const void* Wd, void* dx_p, void* dWg, void* dWu,
                    void* dWd, void* dG, void* dU, void* A, const FoldedCombine* fc, hipStream_t st) {
  F32Params p = params_of(d, seg, Wg, Wu, Wd, fc);
  p.x = (const float*)x_p;
  p.dy = (const float*)dy_p;
  p.G = (const float*)G;
  p.U = (const float*)U;
  p.outG = (float*)dG;
  p.outU = (float*)dU;
  p.outA = (float*)A;
  p.A = (const float*)A;
  p.dG = (const float*)dG;
  p.dU = (const float*)dU;
  p.C = (float*)dx_p;
  p.dWg = (float*)dWg;
  p.dWu = (float*)dWu;
  p.dWd = (float*)dWd;
  if (wide(d)) return bwd_f32<1, true>(d, p, st);
  return d->F % 4 == 0 ? bwd_f32<4, false>(d, p, st) : d->F % 2 == 0 ? bwd_f32<2, false>(d, p, st) : bwd_f32<1, false>(d, p, st);
}

}  // namespace dynmo
