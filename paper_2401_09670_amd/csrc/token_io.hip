// The two ends of the token loop around the layer stack (Sec. 2.1: a prompt's tokens go in, the
// prefill pass produces the first new token, every decoding step one more): the embedding gather on
// the way in; on the way out the merge of the per-column-block maxima that the logits GEMM leaves.
#include <limits.h>

#include "common.h"
#include "kernels.h"

namespace ds {

// One workgroup per output row, 16-byte pieces.  Ids outside the tables are clamped into them (a
// wrong id must not become a wild read).  Up to 512 rows it is bound by latency: the T pieces of a lane are asked for
// together (past the end the last one again, not used).  5120 features with positions at 64 rows 2.73 -> 2.51 us, 12288
// 3.57 -> 3.15; with the merge below, which does the same, both ends of the token loop for 50272 x 5120 at 1 row 85.8 ->
// 84.7, at 64 rows 97.0 -> 95.3.  More rows, a prompt's, are bound by bandwidth: one piece at a time (1024 rows of 9216
// features without positions 5.8 us, 6.3 together).  A lane has no more pieces than its row, and there is no second table
// where none is given (4 pieces and two tables always: 8192 rows of 1024 features without positions 5.6 -> 8.0).
constexpr int kTogether = 4;
constexpr int kStreamedRows = 512;
// All of v is there from here on (or the compiler moves each load behind the branch before its use).
template <int T>
__device__ __forceinline__ void arrived(u32x4 (&v)[T]) {
  static_assert(T >= 1 && T <= 4);
  if constexpr (T == 1) asm volatile("" : "+v"(v[0]));
  if constexpr (T == 2) asm volatile("" : "+v"(v[0]), "+v"(v[1]));
  if constexpr (T == 3) asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]));
  if constexpr (T == 4) asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}
template <int T, bool POS>
__global__ __launch_bounds__(256) void embed_kernel(const int32_t* __restrict__ token_ids,
                                                    const int32_t* __restrict__ positions,
                                                    const uint16_t* __restrict__ tok_emb, int vocab,
                                                    const uint16_t* __restrict__ pos_emb, int n_pos, int h,
                                                    uint16_t* __restrict__ x) {
  const size_t row = blockIdx.x;
  const int id = min(max(token_ids[row], 0), vocab - 1);
  const uint16_t* te = tok_emb + (size_t)id * h;
  const uint16_t* pe = POS ? pos_emb + (size_t)min(max(positions[row], 0), n_pos - 1) * h : nullptr;
  uint16_t* xr = x + row * (size_t)h;
  const int pieces = h >> 3;
  for (int c0 = threadIdx.x; c0 < pieces; c0 += T * 256) {
    u32x4 a[T], b[T];
#pragma unroll
    for (int u = 0; u < T; ++u) {
      const int c = T == 1 ? c0 : min(c0 + 256 * u, pieces - 1);
      a[u] = ld16(te + c * 8);
      if constexpr (POS) b[u] = ld16(pe + c * 8);
    }
    if constexpr (POS) arrived(b);
    arrived(a);
#pragma unroll
    for (int u = 0; u < T; ++u) {
      if (c0 + 256 * u >= pieces) break;
      if constexpr (POS) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          a[u][j] = pack_bf16(bf16_lo(a[u][j]) + bf16_lo(b[u][j]), bf16_hi(a[u][j]) + bf16_hi(b[u][j]));
      }
      st16(xr + (c0 + 256 * u) * 8, a[u]);
    }
  }
}

template <int T>
static void launch_embed_pieces(const int32_t* token_ids, const int32_t* positions, const void* tok_emb, int vocab,
                                const void* pos_emb, int n_pos, int rows, int h, void* x, hipStream_t stream) {
  auto* kern = pos_emb ? embed_kernel<T, true> : embed_kernel<T, false>;
  hipLaunchKernelGGL(kern, dim3(rows), dim3(256), 0, stream, token_ids, positions, (const uint16_t*)tok_emb, vocab,
                     (const uint16_t*)pos_emb, n_pos, h, (uint16_t*)x);
}

hipError_t launch_embed(const int32_t* token_ids, const int32_t* positions, const void* tok_emb, int vocab,
                        const void* pos_emb, int n_pos, int rows, int h, void* x, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (h % 8 != 0 || vocab <= 0 || (pos_emb && (!positions || n_pos <= 0))) return hipErrorInvalidValue;
  const int turns = rows > kStreamedRows ? 1 : (h / 8 + 255) / 256;  // pieces of a lane at a time
  auto* launch = turns <= 1 ? launch_embed_pieces<1>
                            : (turns == 2 ? launch_embed_pieces<2>
                                          : (turns == 3 ? launch_embed_pieces<3> : launch_embed_pieces<kTogether>));
  launch(token_ids, positions, tok_emb, vocab, pos_emb, n_pos, rows, h, x, stream);
  return hipGetLastError();
}

// Merge the column blocks' candidates of one row: largest value, lowest column among equals.
// part_val / part_idx are [n_blocks][M].  A lane asks for kTogether candidates at a time (the last block's again past
// the end: a candidate does not win against itself).
__global__ __launch_bounds__(64) void argmax_merge_kernel(const float* __restrict__ part_val,
                                                          const int32_t* __restrict__ part_idx, int n_blocks,
                                                          int M, int32_t* __restrict__ next_token,
                                                          float* __restrict__ best_logit) {
  const int m = blockIdx.x;
  float bv = -INFINITY;
  int bi = INT_MAX;
  for (int b0 = threadIdx.x; b0 < n_blocks; b0 += kTogether * 64) {
    float v[kTogether];
    int i[kTogether];
#pragma unroll
    for (int u = 0; u < kTogether; ++u) {
      const size_t at = (size_t)min(b0 + 64 * u, n_blocks - 1) * M + m;
      v[u] = part_val[at];
      i[u] = part_idx[at];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kTogether; ++u)
      if (v[u] > bv || (v[u] == bv && i[u] < bi)) {
        bv = v[u];
        bi = i[u];
      }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float ov = __shfl_xor(bv, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    if (ov > bv || (ov == bv && oi < bi)) {
      bv = ov;
      bi = oi;
    }
  }
  if (threadIdx.x == 0) {
    next_token[m] = bi;
    if (best_logit) best_logit[m] = bv;
  }
}

hipError_t launch_argmax_merge(const float* part_val, const int32_t* part_idx, int n_blocks, int M,
                               int32_t* next_token, float* best_logit, hipStream_t stream) {
  hipLaunchKernelGGL(argmax_merge_kernel, dim3(M), dim3(64), 0, stream, part_val, part_idx, n_blocks, M,
                     next_token, best_logit);
  return hipGetLastError();
}

}  // namespace ds
