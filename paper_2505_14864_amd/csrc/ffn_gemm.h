// What the bf16 grouped-GEMM kernels (ffn_mfma.hip, ffn_tile.hip, ffn_dw.hip, ffn_skinny.hip) share: the product's parameters, the global -> LDS
// loads, and the element-wise parts of their epilogues.
#pragma once

#include <type_traits>
#include <utility>

#include "common.h"
#include "ffn.h"
#include "profile.h"

namespace dynmo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;

// MODE_DOWN_FOLD is MODE_DOWN with the weighted combine of a one-slot layer in its stores;
// MODE_DX_FOLD is MODE_DX with the scatter back to token order (weight 1) in its stores
enum { MODE_GATEUP = 0, MODE_DOWN = 1, MODE_DA = 2, MODE_DX = 3, MODE_DW = 4, MODE_DOWN_FOLD = 5, MODE_DX_FOLD = 6 };

struct GemmParams {
  const int32_t* seg;
  int E;
  int M;  // rows of the output (MODE_DW only; the other modes take rows from seg)
  int N;  // columns of the output (for GATEUP: F, and a tile spans 128 of them twice)
  int K;  // contraction length per phase (MODE_DW: taken from seg)
  const bf16_t* A1;
  const bf16_t* A2;
  long lda;
  const bf16_t* B1;
  const bf16_t* B2;
  long ldb;
  long b_expert_stride;
  bf16_t* C0;
  bf16_t* C1;
  bf16_t* C2;
  long ldc;
  const bf16_t* G;
  const bf16_t* U;
  float* partial;     // kMaxPersistent fp32 partial tiles, then kSplitHdrInts ints (modes that may split k)
  const int32_t* gather;  // MODE_GATEUP: row p of operand A is row gather[p] / gather_div of A1, or nullptr
  int gather_div;
  // MODE_DOWN_FOLD / MODE_DX_FOLD (k = 1): row p also goes to row t = scatter[p] of out as
  // res[t] + scale[t] * value (res nullptr = 0; res may be out; scale nullptr = 1); C0 may then be nullptr
  const int32_t* scatter;
  const float* scale;
  const bf16_t* res;
  bf16_t* out;
};

constexpr uint32_t kOob = 0x80000000u;

// raw buffer descriptor (wave-uniform): base address, stride 0, record count in bytes
typedef uint32_t desc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ desc_t make_desc(const bf16_t* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  desc_t d;
  d.x = __builtin_amdgcn_readfirstlane((uint32_t)a);
  d.y = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
  d.z = __builtin_amdgcn_readfirstlane(bytes);
  d.w = 0x00020000u;
  return d;
}

// One piece: global -> LDS.  Written as assembly so that the compiler sees neither a
// load (it would count it against its own waits) nor an LDS write (it would make every
// transposed LDS read wait for all outstanding loads); the k loop waits for these loads
// itself, once per k tile.  The memory clobber keeps LDS reads from moving across it.
// The LDS destination is `lds_base` (wave-uniform, in a scalar register) + LDS_CONST.
template <int LDS_CONST>
__device__ __forceinline__ void load_to_lds(desc_t d, uint32_t lds_base, uint32_t global_offset) {
  asm volatile("s_add_i32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds_base), "v"(global_offset), "s"(d), "n"(LDS_CONST)
               : "memory", "scc");
}

template <int... Is, typename F>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), fully unrolled
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// The logistic function for results that are rounded to bf16: the hardware reciprocal (1 ulp) instead of a
// correctly rounded division, which is ten instructions per element in epilogues that are bound by their
// vector arithmetic.
__device__ __forceinline__ float sigmoid_bf16(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_mul(float g, float u) { return g * sigmoid_bf16(g) * u; }
// swiglu_bwd() of ffn.h with that reciprocal
__device__ __forceinline__ void swiglu_bwd_bf16(float dA, float g, float u, float* a, float* dg, float* du) {
  const float s = sigmoid_bf16(g);
  const float gs = g * s;
  *a = gs * u;
  *dg = dA * u * (s * (1.f + g * (1.f - s)));
  *du = dA * gs;
}

// ---- what ffn_tile.hip and ffn_dw.hip share: tiles whose k goes in steps of 32
constexpr int kTileK = 32;
constexpr int kChunkTiles = 4;  // row tiles that are walked together, column tile by column tile

// Waits until at most N of this wavefront's loads and stores, and none of its LDS reads, are outstanding.
template <int N>
__device__ __forceinline__ void wait_stage() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}

// Tile r of mt x nt tiles: row tiles in chunks of kChunkTiles, a chunk walked column tile by column tile.
__device__ __forceinline__ void tile_of(int r, int mt, int nt, int* mi, int* ni) {
  const int c = r / (kChunkTiles * nt);
  const int h = min(kChunkTiles, mt - c * kChunkTiles);
  r -= c * kChunkTiles * nt;
  *ni = r / h;
  *mi = c * kChunkTiles + r - *ni * h;
}

// An operand that lies [k][row] in memory: in LDS the k-row k of ROWS rows is ROWS / 32 blocks of 64 bytes; block b is stored as block
// b ^ (k & 3) (64 rows: b ^ ((k >> 1) & 1)), its two 32-byte halves swapped when bit 3 of k is set.
// where block `b` of k-row `k` is stored, and the other way round
template <int ROWS>
__device__ __forceinline__ int swizzled(int b, int k) {
  return ROWS == 64 ? b ^ ((k >> 1) & 1) : b ^ (k & 3);
}
// byte offset, from the tile's (row 0, k 0) element, of the 16 bytes that `lane` moves in piece q (1 KB); kOob outside the rows
template <int ROWS>
__device__ __forceinline__ uint32_t krow_piece(int q, int lane, uint32_t ld_bytes, int rows_left) {
  constexpr int kLanesPerK = ROWS * 2 / 16;
  const int k = q * (64 / kLanesPerK) + lane / kLanesPerK, slot = lane % kLanesPerK;
  const int blk = swizzled<ROWS>(slot >> 2, k);
  const int col = blk * 32 + ((slot & 3) ^ (((k >> 3) & 1) << 1)) * 8;
  return col < rows_left ? (uint32_t)k * ld_bytes + col * 2 : kOob;
}
// LDS byte offset (inside the operand's stage) from which `lane` reads its fragment of a 16-row block with ds_read_b64_tr_b16: lane
// l holds, for row l % 16 of the block, the eight k values (l / 16) * 8 .. + 7
template <int ROWS>
__device__ __forceinline__ uint32_t krow_frag(int lane, int block16) {
  const int s = lane & 15, g = lane >> 4;
  const int k = g * 8 + (s >> 2);
  const int blk = block16 >> 1, half = block16 & 1;
  return k * (ROWS * 2) + swizzled<ROWS>(blk, k) * 64 + (((g & 1) ^ half) << 5) + (s & 3) * 8;
}

// Which kernel takes a product (the DYNMO_KERNEL_* values of dynmo.h): ffn_mfma.hip, ffn_tile.hip with one of its tiles, ffn_skinny.hip
enum TileKind {
  TILE_256 = DYNMO_KERNEL_256x256,
  TILE_128x256 = DYNMO_KERNEL_128x256,
  TILE_128 = DYNMO_KERNEL_128x128,
  TILE_64 = DYNMO_KERNEL_64x64,
  FEW_ROWS = DYNMO_KERNEL_FEW_ROWS
};
// ffn_tile.hip: a row-segmented product (any mode but MODE_DW; MODE_GATEUP not on 128 x 256 tiles).
// DYNMO_EINVAL for a kind that is none of its tiles.
int32_t ffn_tile_rows(int mode, TileKind kind, const dynmo_desc* d, const GemmParams& p, KernelId id, hipStream_t st);
// ffn_dw.hip: the three weight gradients on the same tiles
int32_t ffn_dw_tiles(TileKind kind, const dynmo_desc* d, const int32_t* seg, const bf16_t* dy_p, const bf16_t* x_p,
                     const bf16_t* A, const bf16_t* dG, const bf16_t* dU, bf16_t* dWg, bf16_t* dWu, bf16_t* dWd, hipStream_t st);

// ffn_skinny.hip: MODE_GATEUP, MODE_DOWN or MODE_DOWN_FOLD with few rows per expert; at most `max_experts` experts have
// rows, none of them more than `max_rows` unless a token takes an expert twice (right in any case)
int32_t ffn_skinny_rows(int mode, const GemmParams& p, int max_experts, int max_rows, KernelId id, hipStream_t st);

}  // namespace dynmo
