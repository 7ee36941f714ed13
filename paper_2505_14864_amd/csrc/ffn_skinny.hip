// Grouped SwiGLU FFN forward on the gfx950 matrix cores (bf16 in, fp32 accumulate) for few rows per
// expert: decode steps and short prompts.
//
// Bound: reading the weights once.  There is next to no reuse of a weight inside a workgroup, so weights
// do not pass through LDS at all: a wavefront loads them from global memory straight into the MFMA
// operand layout, two or one k pieces ahead, and needs no barrier inside its k loop.  A workgroup of four
// wavefronts takes 16 CB weight rows of one expert; the wavefronts deal the k range among them in
// pieces of 64 (one 128-byte line of every weight row), so that together they stream 512 contiguous
// bytes per row and step, and add their fp32 sums in LDS at the end, in a fixed order: no split over
// workgroups, no second pass.  The rows of the expert are read from L1 / L2 in the same layout, 16, 32 or 64 at a
// time; every 64 rows of an expert are workgroups of their own, so that an expert that took many rows keeps as many
// workgroups busy as its rows need instead of walking its weights again and again.
//
// Measured, 64 rows over 8 experts, H=4096 F=14336: gate/up 446 us on 256-row tiles -> 330 (5.7 TB/s of weights), down
// 188 -> 159 (5.9 TB/s); 8 rows, H=1024 F=4096, down 20 -> 10.  Loading the two halves of a line with the lanes of one
// instruction or of two, and three instead of two workgroups per compute unit, measured the same.
#include "ffn_gemm.h"

namespace dynmo {

constexpr int kSkinnyThreads = 256;
constexpr int kSkinnyWaves = kSkinnyThreads / 64;
constexpr int kSkinnyRows = 64;  // rows that a workgroup takes at a time

// Whether grid y counts the experts that have rows (else all experts); `chunks`: row chunks on grid z
__host__ __device__ constexpr bool compacts(int mode, int chunks) { return mode != MODE_GATEUP && chunks == 1; }

template <int MODE, int CB>
__global__ __launch_bounds__(kSkinnyThreads, 2) void ffn_skinny_kernel(const GemmParams p) {
  __shared__ f32x4_t part[kSkinnyWaves][CB][64];
  constexpr int PAIRS = MODE == MODE_GATEUP ? CB / 2 : CB;  // gate/up: blocks 0 .. CB/2 - 1 are gate, the others the matching up columns
  const int n0 = blockIdx.x * 16 * PAIRS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Which expert.  The down products of one row chunk count only the experts that have rows, so that the workgroups
  // with work are the first ones and spread evenly over the compute units: they are few enough for that to matter
  // (4 experts, two of them empty, 4096 x 14336, 32 rows: 89 -> 59 us).  It costs gate/up, whose workgroups are many, more than it gives.
  int e = blockIdx.y, begin, end;
  if (compacts(MODE, gridDim.z) && p.E > 1) {
    const int first_row = p.seg[min(lane, p.E)], end_row = p.seg[min(lane + 1, p.E)];
    const unsigned long long used = __ballot(first_row < end_row);
    const unsigned long long mine = __ballot(first_row < end_row && __popcll(used & ((1ull << lane) - 1ull)) == e);
    if (mine == 0) return;
    e = __builtin_ctzll(mine);
    begin = __builtin_amdgcn_readlane(first_row, e);
    end = __builtin_amdgcn_readlane(end_row, e);
  } else {
    begin = p.seg[e];
    end = p.seg[e + 1];
  }
  if (begin + kSkinnyRows * (int)blockIdx.z >= end) return;
  const int s = lane & 15, g = lane >> 4;
  const int chunks = (p.K + 63) / 64;
  const int steps = (chunks + kSkinnyWaves - 1) / kSkinnyWaves;
  // Workgroups start at different places of the k range (and go round): started together at k = 0, with weight rows
  // a power of two apart, they would all ask the same few memory channels (H = 4096: gate/up 394 -> 333 us).
  const int first_step = (blockIdx.x + blockIdx.y) % steps;

  const bf16_t* w1 = p.B1 + (long)e * p.b_expert_stride;
  const bf16_t* w2 = MODE == MODE_GATEUP ? p.B2 + (long)e * p.b_expert_stride : w1;
  const bool gathered = MODE == MODE_GATEUP && p.gather != nullptr;
  const bf16_t* rows = gathered ? p.A1 : p.A1 + (long)begin * p.lda;
  // every offset below stays inside the operand: rows and columns past the end are the last ones again (their
  // results are dropped), k past the end is masked
  auto rsrc = [](const bf16_t* q) { return __builtin_amdgcn_make_buffer_rsrc((void*)q, 0, 0x7ffffffe, 0x00020000); };
  uint32_t b_off[CB];
#pragma unroll
  for (int j = 0; j < CB; ++j) b_off[j] = (uint32_t)min(n0 + (j % PAIRS) * 16 + s, p.N - 1) * (uint32_t)p.ldb * 2 + g * 16;

  auto pass = [&](int row0, auto RB_C) {
    constexpr int RB = decltype(RB_C)::value;
    constexpr int D = RB <= 2 ? 3 : 2;  // steps in registers
    uint32_t a_off[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      int r = min(row0 + i * 16 + s, end - begin - 1);
      if (gathered) r = p.gather[begin + r] / p.gather_div;
      a_off[i] = (uint32_t)r * (uint32_t)p.lda * 2 + g * 16;
    }
    u32x4 a[D][RB][2], b[D][CB][2];
    auto load = [&](int d, int step) {
      const int turn = step + first_step;  // past the last step: beyond K, nothing is loaded
      const int c = (step >= steps ? steps : turn < steps ? turn : turn - steps) * kSkinnyWaves + wave, k = c * 64 + g * 8;
      const uint32_t at = (uint32_t)c * 128;
#pragma unroll
      for (int j = 0; j < CB; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          b[d][j][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc(j < PAIRS ? w1 : w2),
                                                                                     k + h * 32 < p.K ? b_off[j] + at + h * 64 : kOob, 0, 0));
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          a[d][i][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc(rows), k + h * 32 < p.K ? a_off[i] + at + h * 64 : kOob, 0, 0));
      __builtin_amdgcn_sched_barrier(0);
    };
    f32x4_t acc[RB][CB] = {};
#pragma unroll
    for (int d = 0; d + 1 < D; ++d) load(d, d);
    for (int step = 0; step < steps; step += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load((d + D - 1) % D, step + d + D - 1);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int i = 0; i < RB; ++i)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[d][i][h]),
                                                                  __builtin_bit_cast(bf16x8_t, b[d][j][h]), acc[i][j], 0, 0, 0);
      }
    }
    // ---- the wavefronts' sums, added in their order; element r of block (i, j): row 16 i + 4 g + r, column 16 j + s
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < CB; ++j) part[wave][j][lane] = acc[i][j];
      __syncthreads();
      if (wave >= PAIRS) continue;
      f32x4_t v = part[0][wave][lane], u = {};
#pragma unroll
      for (int w = 1; w < kSkinnyWaves; ++w) v += part[w][wave][lane];
      if constexpr (MODE == MODE_GATEUP) {
        u = part[0][wave + PAIRS][lane];
#pragma unroll
        for (int w = 1; w < kSkinnyWaves; ++w) u += part[w][wave + PAIRS][lane];
      }
      const int n = n0 + wave * 16 + s;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = begin + row0 + i * 16 + g * 4 + r;
        if (m >= end || n >= p.N) continue;
        const long at = (long)m * p.ldc + n;
        if constexpr (MODE == MODE_GATEUP) {
          p.C0[at] = f32_to_bf16(v[r]);
          p.C1[at] = f32_to_bf16(u[r]);
          p.C2[at] = f32_to_bf16(silu_mul(v[r], u[r]));
        } else {
          if (MODE != MODE_DOWN_FOLD || p.C0) p.C0[at] = f32_to_bf16(v[r]);
          if constexpr (MODE == MODE_DOWN_FOLD) {
            const int token = p.scatter[m];
            const long to = (long)token * p.ldc + n;
            p.out[to] = f32_to_bf16((p.res ? bf16_to_f32(p.res[to]) : 0.f) + (p.scale ? p.scale[token] : 1.f) * v[r]);
          }
        }
      }
    }
  };
  for (int row0 = kSkinnyRows * blockIdx.z; row0 < end - begin; row0 += kSkinnyRows * gridDim.z) {
    const int left = end - begin - row0;
    if (left <= 16) pass(row0, std::integral_constant<int, 1>{});
    else if (left <= 32) pass(row0, std::integral_constant<int, 2>{});
    else pass(row0, std::integral_constant<int, 4>{});
  }
}

template <int MODE, int CB>
static int32_t launch_skinny(const GemmParams& p, int max_experts, int max_rows, KernelId id, hipStream_t st) {
  constexpr int cols = 16 * (MODE == MODE_GATEUP ? CB / 2 : CB);
  const int chunks = (max_rows + kSkinnyRows - 1) / kSkinnyRows;
  const dim3 grid((p.N + cols - 1) / cols, compacts(MODE, chunks) ? max_experts : p.E, chunks);
  DYNMO_TIMED_LAUNCH(id, st, ffn_skinny_kernel<MODE, CB><<<grid, dim3(kSkinnyThreads), 0, st>>>(p));
  return DYNMO_OK;
}

int32_t ffn_skinny_rows(int mode, const GemmParams& p, int max_experts, int max_rows, KernelId id, hipStream_t st) {
  if (max_experts <= 0) return DYNMO_OK;
  // 64 weight rows per workgroup, fewer where that would leave the chip (two workgroups per compute unit) short of work.
  // `blocks` assumes that every expert is in use.  When only few are, a down product with its long k is left with few
  // workgroups, so it keeps four times as many as it needs otherwise, at no cost to an even routing (8 experts, 4096 x
  // 14336, 16 rows on two of them / on all eight: 64 weight rows per workgroup 80 / 163 us, 32 49 / 159; 256-row tiles 59 / 188).
  const long blocks = (long)p.N * (mode == MODE_GATEUP ? 2 : 1) / 16 * max_experts;
  switch (mode) {
    case MODE_GATEUP:
      return blocks >= 4 * 512 ? launch_skinny<MODE_GATEUP, 4>(p, max_experts, max_rows, id, st)
                               : launch_skinny<MODE_GATEUP, 2>(p, max_experts, max_rows, id, st);
    case MODE_DOWN:
      return blocks >= 12 * 512  ? launch_skinny<MODE_DOWN, 4>(p, max_experts, max_rows, id, st)
             : blocks >= 2 * 512 ? launch_skinny<MODE_DOWN, 2>(p, max_experts, max_rows, id, st)
                                 : launch_skinny<MODE_DOWN, 1>(p, max_experts, max_rows, id, st);
    case MODE_DOWN_FOLD:
      return blocks >= 12 * 512  ? launch_skinny<MODE_DOWN_FOLD, 4>(p, max_experts, max_rows, id, st)
             : blocks >= 2 * 512 ? launch_skinny<MODE_DOWN_FOLD, 2>(p, max_experts, max_rows, id, st)
                                 : launch_skinny<MODE_DOWN_FOLD, 1>(p, max_experts, max_rows, id, st);
  }
  return DYNMO_EINVAL;
}

}  // namespace dynmo
