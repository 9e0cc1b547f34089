// Decode-phase GEMM: Y[M,N] = act(X[M,K] W[N,K]^T + bias) + residual for a handful of rows
// (ds_linear routes M <= 128 here, a layer M <= 64 and what is faster here up to 128; the kernels accept up to 256).
// The weights (N*K*2 bytes) are read once from HBM and dominate the traffic
// (App. A.3: 4h^2 + 2hm elements per layer), so the kernels are organised
// around streaming W at HBM rate while the matrix cores do the M x ... work.
//
// Two streaming kernels live here, one for products too short to stream, and the second passes of split-K:
//   * wring_gemm_kernel  - wave-private rings, no split of K over workgroups, no second launch;
//     taken for M <= 64 when N alone yields enough workgroups (described at the kernel).
//   * skinny_gemm_kernel - one ring per workgroup, K split over workgroups; everything else.
//   * short_wring_gemm_kernel - a layer's products of up to 8.5 MB of weights, optionally with the LayerNorm before it.
//   * skinny_reduce*_kernel - add the split partials in a fixed order and apply the epilogue,
//     optionally fused with the LayerNorm that follows or with the append to the paged KV cache;
//     also used by the tile GEMM when it splits K.
//
// What bounds the ring kernel on this chip is the number of bytes a CU can pull through
// its vector L1 per unit time, and the activation slabs count against that
// budget although they come from L2.  A workgroup therefore covers BN = 64,
// 128 or 256 weight rows (the X slab is fetched once per BN columns), and the
// K axis is split over workgroups until the chip is full; the launcher picks
// BN and the split count that minimise weight + activation + partial-sum
// bytes.
//
// grid = (N/BN, KSPLIT).  Workgroup = 8 waves: wave w owns the column tiles
// (16 weight rows each) of column group w & 3 and, of every 64-wide k slab,
// the 32-wide MFMA k-step w >> 2; the two k-halves are
// added through LDS at the end.  Both operands go global -> LDS directly (no
// registers, no ds_write) into a ring of S stages; a wave-level load fetches
// 8 rows x 128 contiguous bytes.  The tile is computed transposed (weights
// as MFMA row operand), so a lane ends up with 4 consecutive output columns
// of one row.  With KSPLIT > 1 each split writes fp32 partial sums and a
// second kernel adds them in a fixed order and applies the epilogue.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ds {

// Cache policy operand of the direct-to-LDS weight loads: 2 = non-temporal.  A weight byte is used once per
// launch, so it is not worth a line in L2 or the last-level cache (measured: 42.4 -> 41.3 us per decode GEMM
// at OPT-13B, batch 64); the activation slabs, re-read by every workgroup, keep the default policy.
constexpr int kWeightAux = 2;
constexpr int kSkThreads = 512;
constexpr int kSkWaves = kSkThreads / 64;
constexpr int kSkKS = 64;  // k elements per slab
// Granularity of K in plans and in the shapes these kernels are given.  Two slabs: the plan's constants were fitted to
// split counts of that grain, and other multiples of 64 go to the tile kernel.
constexpr int kSkPlanK = 128;

struct SkinnyParams {
  const uint16_t* X;
  const uint16_t* W;
  const uint16_t* bias;
  const uint16_t* residual;
  uint16_t* out[3];
  int seg_cols, seg_cols_kv;  // widths of the first and of the other two output segments
  int M, N, K;
  int relu;
  int splits = 1;  // gridDim.y
  float* partial;  // [KSPLIT][M][N] fp32 when splits > 1
  // Greedy-choice mode (unsplit launches only): nothing is written to `out`; per row the largest
  // accumulator of this workgroup's columns and its column go to amax_val / amax_idx [column block][M].
  float* amax_val = nullptr;
  int32_t* amax_idx = nullptr;
  // Unsplit launches only: with kv_k_cache set (decode QKV projection, N = (n + 2 n_kv) s) the K and V
  // parts of row m go to slot kv_ctx_lens[m] of the paged cache [num_blocks, n_kv, 16, s] instead of `out`.
  const int32_t* kv_ctx_lens = nullptr;
  const int32_t* kv_block_tables = nullptr;
  int kv_max_blocks = 0;
  uint16_t* kv_k_cache = nullptr;
  uint16_t* kv_v_cache = nullptr;
  int kv_n_heads = 0, kv_n_kv_heads = 0, kv_head_dim = 0;
  // short_wring_gemm_kernel<.., true> only: the rows of X are normalised first.
  const uint16_t* norm_gamma = nullptr;
  const uint16_t* norm_beta = nullptr;
  float norm_eps = 0.f;
};

template <int VM>
__device__ __forceinline__ void sk_wait_vmcnt() {
  // s_waitcnt with only vmcnt set: vmcnt[3:0] | expcnt=7 | lgkmcnt=15 | vmcnt[5:4] in bits 15:14
  __builtin_amdgcn_s_waitcnt((VM & 0xf) | (0x7 << 4) | (0xf << 8) | ((VM >> 4) << 14));
}

// Epilogue of the unsplit kernels, four columns n .. n+3 of a row at a time: bias, ReLU, residual, then into their output
// segment, or, in a decode QKV projection, this step's K / V row straight into its page.  Everything it reads is asked for
// while the product runs (Epilogue4): a load between two stores makes the second wait for the first to arrive, four to
// eight round trips in a row (prefill of 57 OPT-13B tokens 156.8 -> 154.7 us, a step at 64 rows 262.3 -> 261.2).  A wave
// finishes C column tiles of MT row tiles.
template <int C, int MT>
struct Epilogue4 {
  u32x2 bias[C], res[C][MT];
  int pos[MT], block[MT];  // slot of each row's sequence, and its page
  int first = 0;           // row of the first row tile
  // First column of tile c: col(c).  Rows and columns past the end are read inside the output, an absent operand from the
  // weights and not used: a branch around a load ends in a wait for all that are in flight.
  template <class Col>
  __device__ __forceinline__ void request(const SkinnyParams& p, int lane, Col&& col) {
    const uint16_t* bias_at = p.bias ? p.bias : p.W;
    const uint16_t* res_at = p.residual ? p.residual : p.W;
    const int ld_res = p.residual ? p.N : 0;
    const int32_t* pos_at = p.kv_k_cache ? p.kv_ctx_lens : reinterpret_cast<const int32_t*>(p.W);
    const int seqs = p.kv_k_cache ? ~0 : 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int n = min(col(c) + (lane >> 4) * 4, p.N - 4);
      bias[c] = *reinterpret_cast<const u32x2*>(bias_at + n);
#pragma unroll
      for (int t = 0; t < MT; ++t)
        res[c][t] = *reinterpret_cast<const u32x2*>(res_at + (size_t)row(p, lane, t) * ld_res + n);
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) pos[t] = pos_at[row(p, lane, t) & seqs];
  }
  __device__ __forceinline__ void pages(const SkinnyParams& p, int lane) {
    const int32_t* at = p.kv_k_cache ? p.kv_block_tables : reinterpret_cast<const int32_t*>(p.W);
    const size_t seqs = p.kv_k_cache ? ~(size_t)0 : 0;
#pragma unroll
    for (int t = 0; t < MT; ++t) block[t] = at[((size_t)row(p, lane, t) * p.kv_max_blocks + (pos[t] >> 4)) & seqs];
  }
  __device__ __forceinline__ int row(const SkinnyParams& p, int lane, int t) const {
    return min(first + 16 * t + (lane & 15), p.M - 1);
  }
  __device__ __forceinline__ void store(const SkinnyParams& p, const OutSegments& out, int c, int t, int m, int n,
                                        const floatx4& v) const {
    float r[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      r[j] = v[j];
      if (p.bias) r[j] += j & 1 ? bf16_hi(bias[c][j / 2]) : bf16_lo(bias[c][j / 2]);
      if (p.relu) r[j] = fmaxf(r[j], 0.f);
      if (p.residual) r[j] += j & 1 ? bf16_hi(res[c][t][j / 2]) : bf16_lo(res[c][t][j / 2]);
    }
    const u32x2 o{pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3])};
    const int hq = p.kv_n_heads * p.kv_head_dim, hkv = p.kv_n_kv_heads * p.kv_head_dim;
    if (p.kv_k_cache && n >= hq) {
      const int which = n >= hq + hkv;
      const int col = n - hq - which * hkv, shift = __builtin_ctz(p.kv_head_dim);  // 64 or 128
      const int head = col >> shift, d = col - (head << shift);
      const uint64_t k = (uint64_t)p.kv_k_cache, to_v = (uint64_t)p.kv_v_cache - k;
      st8((gmem_u16*)(k + (to_v & (uint64_t)(int64_t)-which) +
                      2 * ((((uint64_t)block[t] * p.kv_n_kv_heads + head) * 16 + (pos[t] & 15)) * p.kv_head_dim + d)), o);
      return;
    }
    st8(out.at(m, n), o);
  }
};

// Waits until at most `slabs` (0 .. MOST) slabs of G loads are in flight.
template <int MOST, int G>
__device__ __forceinline__ void sk_wait_slabs(int slabs) {
  if constexpr (MOST == 0) {
    sk_wait_vmcnt<0>();
  } else {
    if (slabs >= MOST) sk_wait_vmcnt<MOST * G>();
    else sk_wait_slabs<MOST - 1, G>(slabs);
  }
}

// Which of its ns slabs (slab_stride elements apart) a workgroup starts with; it goes round from there.  Where the row
// stride is a multiple of 4 KB, the pieces that all rows have at one position of K lie on few memory channels, and
// workgroups in lockstep wait for these (32768 x 8192, 48 rows: 123 us, 91 with this; 49152 x 12288, 64 rows: 218 and
// 214).  So each XCD (id % 8) starts at an eighth of its own, and its 32 workgroups are spread over as many slabs as
// their activations keep in the XCD's L2 (spread over all of K, 128 rows of 5120 x 20480 take 65 us, not 56).  Other
// strides spread by themselves, and rows in step share DRAM pages (5120 x 5120, 64 rows: 18.8 us in step, 20 spread).
// `rows` is the most rows the kernel takes (64, 128 or 256), never the batch's own: the start decides in which order K
// is added, and a sequence's result must not depend on how many others are in its step.  So a small batch is spread as a
// full one, and the window is all of the L2's 4 MB (half of it: 8192 x 32768 at 1 row 92.6 us, not 87.2, at 128 rows
// 112.4, not 107.2).
__device__ __forceinline__ int start_slab(unsigned id, int ns, int slab_stride, int rows, int K) {
  if (K % 2048 != 0) return 0;
  const int in_l2 = (1 << 21) / (rows * slab_stride);  // slabs whose activations take 4 MB
  const int window = in_l2 < ns ? in_l2 : ns;
  return (int)(((id & 7) * (unsigned)ns / 8 + ((id >> 3) & 31) * (unsigned)window / 32) % (unsigned)ns);
}

// MT = activation row tiles of 16 (1, 2, 4, 8, 16); NTW = most column tiles of a wave (1 to 4); S = LDS stages (prefetch
// distance D = S - 1); NT = column tiles of the workgroup: 4 * NTW, or for the greedy choice also 10, 13 and 14, dealt
// out in turn to the four column groups of waves.
//
// Stage layout: [MP rows of X | BN rows of W], every row 64 k-elements = 128 B = 8 chunks of
// 16 B, unpadded; chunk c of row r sits at position c ^ ((r >> 1) & 7), so the 16 consecutive rows a
// fragment read touches spread over all banks.  The swizzle is applied on the global
// side: lane l of a wave-level load fetches row 8g + l/8, chunk (l%8) ^ ((row >> 1) & 7).
//
// What bounds it: bytes on their way from HBM, so the ring holds as many small stages as the LDS has room for (160 KB of
// 16 to 40 KB each) and the loop never drains it - behind __syncthreads() the compiler waits for every load in
// flight, which with 128-element slabs in two or three stages left a gap per slab.  Nor does it ask for more slabs than
// there are: with the last one loaded again and again, so that the count of loads in flight stays the same, 512 x 128
// brought in nine slabs for two (1 row: 3.6 us, 3.2 without) and long products were 1-5 % slower.  Per product, reduce
// pass included, from 128-element slabs: 5120 x 5120 at 1 row 18.3 -> 14.0 us, at 64 rows 21.0 -> 19.5; 5120 x 20480 at
// 1 row 47.7 -> 39.5, at 64 rows 53.8 -> 46.4; 32768 x 8192 at 48 rows 128 -> 89 (6.0 TB/s of weights); 12288 x 49152 at
// 128 rows 301 -> 296.
template <int MT, int NTW, int S, int NT = 4 * NTW>
__global__ __launch_bounds__(kSkThreads) void skinny_gemm_kernel(const SkinnyParams p) {
  constexpr int MP = MT * 16;  // padded activation rows held in LDS
  constexpr int BN = 16 * NT;  // weight rows per workgroup
  constexpr int D = S - 1;      // slabs in flight ahead of the one being multiplied
  constexpr int STAGE_ELEMS = (MP + BN) * kSkKS;
  constexpr int GROUPS = (MP + BN) / 8;  // wave-level loads (8 rows each) per slab
  constexpr int XGROUPS = MP / 8, MORE = GROUPS % kSkWaves;  // the first MORE waves issue one load more than the others
  static_assert(XGROUPS % kSkWaves == 0 || XGROUPS < kSkWaves, "X rows: whole loads of all waves, or of some");
  static_assert(D >= 1 && (D - 1) * ((GROUPS + kSkWaves - 1) / kSkWaves) < 64, "vmcnt range");
  static_assert(NT <= 4 * NTW && NT > 4 * (NTW - 1), "column tiles of four groups of waves");
  extern __shared__ __attribute__((aligned(1024))) uint16_t lds[];  // [S][MP + BN][64]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int ng = wave & 3, kh = wave >> 2;  // column group, k half
  const int n0 = blockIdx.x * BN;
  const int split = blockIdx.y;
  const int n_splits = p.splits;
  // The K axis is dealt to the splits slab by slab: split s takes number s of every group of n_splits slabs.  With a
  // multiple of 4 splits it takes number (s + i) % n_splits of group i instead, or it would meet only every fourth
  // 128-byte piece of a row, a fraction of the memory channels (8192 x 32768, 48 rows, 8 splits: 118 -> 93 us; other
  // split counts meet all of them anyway and lose up to 10 % by the turning).
  // (The divisions are left out where there is nothing to divide: they are a tenth of a launch over few slabs.)
  const int slabs_total = p.K / kSkKS;
  const int turn_by = n_splits > 1 && (n_splits & 3) == 0 ? 1 : 0;
  int ns = slabs_total;  // >= 1: n_splits <= slabs_total
  if (n_splits > 1) {
    const int whole = slabs_total / n_splits;
    const int number = turn_by ? (split + whole) % n_splits : split;  // of this split in a last, partial group
    ns = whole + (number < slabs_total - whole * n_splits ? 1 : 0);
  }
  const int K = p.K;
  // Greedy choice: one order for all column blocks, so that equal vocabulary rows get equal logits, bit for bit, and the
  // tie goes to the lowest id.
  const int rot = p.amax_val ? 0
                             : start_slab(blockIdx.x + (p.N + BN - 1) / BN * split, ns, n_splits * kSkKS,
                                          MP < 64 ? 64 : MP, K);

  floatx4 acc[NTW][MT];
#pragma unroll
  for (int a = 0; a < NTW; ++a)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[a][t] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Column tile number a of this wave: its group's own range, or, where the groups have unequal numbers, every fourth.
  auto column_tile = [&](int a) __attribute__((always_inline)) { return NT == 4 * NTW ? ng * NTW + a : 4 * a + ng; };
  // fragment read offset of this wave's k-step: lane (row = lane%16, kq = lane/16) reads chunk 4*step + kq of its row
  const int fo = (lane & 15) * kSkKS + (((4 * kh + (lane >> 4)) ^ (((lane & 15) >> 1) & 7)) * 8);
  const int ngs = __builtin_amdgcn_readfirstlane(ng);
  auto multiply = [&](int st) __attribute__((always_inline)) {
    const uint16_t* sb = lds + st * STAGE_ELEMS;
    u32x4 xf[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) xf[t] = *reinterpret_cast<const u32x4*>(sb + t * 16 * kSkKS + fo);
#pragma unroll
    for (int a = 0; a < NTW; ++a) {
      if (NT < 4 * NTW && 4 * a + ngs >= NT) break;
      const u32x4 wf = *reinterpret_cast<const u32x4*>(sb + (MP + column_tile(a) * 16) * kSkKS + fo);
#pragma unroll
      for (int t = 0; t < MT; ++t)
        acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf),
                                                            __builtin_bit_cast(bf16x8, xf[t]), acc[a][t], 0, 0, 0);
    }
  };

  // The loop of a wave that issues G loads a slab: load j is row group g = j*8 + wave of the stage (8 rows), X rows
  // first, then W rows.
  auto run = [&](auto loads) __attribute__((always_inline)) {
    constexpr int G = decltype(loads)::value;
    const int lr = lane >> 3;
    const uint16_t* src[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int r = 8 * (j * kSkWaves + wave) + lr;  // stage row
      const int sw = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
      if (r < MP) src[j] = p.X + (size_t)min(r, p.M - 1) * K + sw;
      else src[j] = p.W + (size_t)min(n0 + r - MP, p.N - 1) * K + sw;
    }
    // requests the next slab of this split into stage `st`
    int group = rot, turn = turn_by && rot ? (split + rot) % n_splits : split;
    auto request = [&](int st) __attribute__((always_inline)) {
      const int ofs = (group * n_splits + turn) * kSkKS;
      turn = turn + turn_by == n_splits ? 0 : turn + turn_by;
      if (++group == ns) group = 0, turn = split;
      uint16_t* dst = lds + st * STAGE_ELEMS + wave_s * 512;  // one wave-load = 8 rows = 1 KB = 512 elements
#pragma unroll
      for (int j = 0; j < G; ++j) {
        if (j < XGROUPS / kSkWaves || (j == 0 && wave_s < XGROUPS))  // activation rows
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + ofs),
                                           (__attribute__((address_space(3))) void*)(dst + j * kSkWaves * 512), 16,
                                           0, 0);
        else
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + ofs),
                                           (__attribute__((address_space(3))) void*)(dst + j * kSkWaves * 512), 16,
                                           0, kWeightAux);
      }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < ns) request(d);

    int st = 0;      // stage of slab i
    int st_req = D;  // stage slab i+D goes to (= the stage slab i-1 used)
    int i = 0;
    for (; i + D < ns; ++i) {
      sk_wait_vmcnt<(D - 1) * G>();  // this wave's part of slab i has landed
      lds_barrier();                 // slab i visible to all waves; everyone is done with slab i-1
      request(st_req);
      multiply(st);
      st_req = st;
      st = (st + 1 == S) ? 0 : st + 1;
    }
    // The last D slabs, all requested: ns - 1 - i younger ones may still be in flight.
    for (; i < ns; ++i) {
      sk_wait_slabs<D - 1, G>(ns - 1 - i);
      lds_barrier();
      multiply(st);
      st = (st + 1 == S) ? 0 : st + 1;
    }
  };
  if constexpr (MORE == 0) {
    run(std::integral_constant<int, GROUPS / kSkWaves>{});
  } else {
    if (wave_s < MORE) run(std::integral_constant<int, GROUPS / kSkWaves + 1>{});
    else run(std::integral_constant<int, GROUPS / kSkWaves>{});
  }
  Epilogue4<NTW, MT> epi;
  if (n_splits == 1 && !p.amax_val && kh == 0) {  // (before the loop these loads held up the split launches, 1 %)
    epi.request(p, lane, [&](int a) { return n0 + column_tile(a) * 16; });
    epi.pages(p, lane);
  }
  sk_wait_vmcnt<0>();  // no global->LDS write of this workgroup may still be in flight ...
  __syncthreads();     // ... and nobody reads the stages any more: reuse them to add the two k-halves
  {
    floatx4* red = reinterpret_cast<floatx4*>(lds);  // [4 column groups][NTW][MT][64 lanes]
    if (kh == 1) {
#pragma unroll
      for (int a = 0; a < NTW; ++a)
#pragma unroll
        for (int t = 0; t < MT; ++t) red[((ng * NTW + a) * MT + t) * 64 + lane] = acc[a][t];
    }
    __syncthreads();
    if (kh == 1) return;
#pragma unroll
    for (int a = 0; a < NTW; ++a)
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[a][t] += red[((ng * NTW + a) * MT + t) * 64 + lane];
  }

  // acc[a][t][r]: row m = 16t + lane%16, column n = n0 + 16*column_tile(a) + 4*(lane/16) + r
  if (p.amax_val) {
    // candidates of this lane per row tile, then across the 4 lanes that share a row (lane/16), then
    // across the 4 column-group waves through LDS (behind the k-half buffer, which may still be read)
    constexpr int RED_FLOATS = 4 * NTW * MT * 64 * 4;
    float* cv = reinterpret_cast<float*>(lds) + RED_FLOATS;  // [4 waves][MT][16]
    int32_t* ci = reinterpret_cast<int32_t*>(cv + 4 * MT * 16);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      float bv = -INFINITY;
      int bi = 0x7fffffff;
#pragma unroll
      for (int a = 0; a < NTW; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int n = n0 + column_tile(a) * 16 + (lane >> 4) * 4 + r;
          const float v = acc[a][t][r];
          if (column_tile(a) < NT && n < p.N && (v > bv || (v == bv && n < bi))) {
            bv = v;
            bi = n;
          }
        }
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {
        const float ov = __shfl_xor(bv, off, 64);
        const int oi = __shfl_xor(bi, off, 64);
        if (ov > bv || (ov == bv && oi < bi)) {
          bv = ov;
          bi = oi;
        }
      }
      if (lane < 16) {
        cv[(ng * MT + t) * 16 + lane] = bv;
        ci[(ng * MT + t) * 16 + lane] = bi;
      }
    }
    __syncthreads();  // the four remaining waves (the k-half-1 waves have left)
    if (ng == 0) {
      for (int e = lane; e < MT * 16; e += 64) {  // e = 16 t + row-in-tile = row m
        float bv = cv[e];
        int bi = ci[e];
#pragma unroll
        for (int g = 1; g < 4; ++g) {
          const float ov = cv[g * MT * 16 + e];
          const int oi = ci[g * MT * 16 + e];
          if (ov > bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
          }
        }
        if (e < p.M) {
          p.amax_val[(size_t)blockIdx.x * p.M + e] = bv;
          p.amax_idx[(size_t)blockIdx.x * p.M + e] = bi;
        }
      }
    }
    return;
  }
  const OutSegments out = out_segments(p, p.seg_cols);
#pragma unroll
  for (int a = 0; a < NTW; ++a) {
    const int n = n0 + column_tile(a) * 16 + (lane >> 4) * 4;
    if (column_tile(a) >= NT || n >= p.N) continue;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int m = t * 16 + (lane & 15);
      if (m >= p.M) continue;
      if (n_splits > 1) {
        *reinterpret_cast<floatx4*>(p.partial + ((size_t)split * p.M + m) * p.N + n) = acc[a][t];
        continue;
      }
      epi.store(p, out, a, t, m, n, acc[a][t]);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Wave-private rings (up to 64 rows, wide N): the shape for which the ring kernel above needs
// split-K only to find 256 workgroups, and then pays for it twice (≈ 5 us of partial-sum stores at
// the end of every workgroup at once, ≈ 5 us for the reduce launch).  Measured on this chip: what a
// streaming kernel needs is not many bytes in flight per CU but several streams per CU that do not
// stall together - two independent 16 KB streams per CU reach 5.7 TB/s, one 64 KB stream 5.3.
//
// So: a workgroup (4 waves; 3 for batches above 64 rows) owns 64 or 80 output columns over the whole K; its waves split
// K between them 64-wide slab by slab (wave w takes slabs w, w+4, ...) and each wave runs its OWN two- or three-stage
// direct-to-LDS ring [16, 32 or 64 activation rows | 64 or 80 weight rows] x 128 bytes, waiting on nothing but its
// own loads - no barrier in the loop, four desynchronised streams per CU.  The four waves' 64 x 64
// fp32 tiles are added through LDS at the end (fixed order) and wave w finishes column tile w.
// grid = N / 64 workgroups, no partial sums in global memory, no second launch.
// ---------------------------------------------------------------------------------------------
constexpr int kWrKS = 64;  // k elements per slab

// NT = weight row tiles of 16 per workgroup (4 or 5: 64 or 80 output columns, whichever tiles N into
// fewer rounds of 256 workgroups); MT = activation row tiles of 16 (1, 2 or 4: batches of up to 16, 32 or
// 64 sequences - a small batch does not pay for 64 activation rows per slab: worth 2 us of a 158 us step at
// OPT-13B, the rest of such a step is weight bytes and per-launch ramps); S = stages of a wave's ring (the
// smaller stages of small batches leave room for a third: two slabs in flight per wave); NW = waves per
// workgroup (4; 3 for batches of 65..128 sequences, whose stages of 128 activation rows fit the LDS three times
// two, not four times two).
template <int NT, int MT, int S, int NW>
__global__ __launch_bounds__(64 * NW) void wring_gemm_kernel(const SkinnyParams p) {
  constexpr int kWrBN = 16 * NT, kWrBM = 16 * MT;
  constexpr int kWrStageElems = (kWrBM + kWrBN) * kWrKS;  // [BM X rows | BN W rows] x 64 k
  constexpr int kWrLoads = (kWrBM + kWrBN) / 8;           // wave-level loads (8 rows x 128 B) per slab
  static_assert((S - 1) * kWrLoads < 64, "vmcnt range");
  extern __shared__ __attribute__((aligned(1024))) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * kWrBN;
  const int K = p.K;
  const int slabs_total = K / kWrKS;
  const int ns = (slabs_total - wave + NW - 1) / NW;  // this wave's slabs: wave, wave + NW, ...  (>= 1: K >= 256)
  const int rot = start_slab(blockIdx.x, ns, NW * kWrKS, MT <= 4 ? 64 : 128, K);

  // load j of a slab covers stage rows 8j .. 8j+7 (rows 0..BM-1 = X, then W); lane: row 8j + lane/8,
  // 16-byte chunk (lane%8) ^ ((row >> 1) & 7) - the swizzle that makes the fragment reads conflict-free
  const uint16_t* src[kWrLoads];
#pragma unroll
  for (int j = 0; j < kWrLoads; ++j) {
    const int r = 8 * j + (lane >> 3);
    const int sw = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    if (r < kWrBM) src[j] = p.X + (size_t)min(r, p.M - 1) * K + (size_t)wave * kWrKS + sw;
    else src[j] = p.W + (size_t)min(n0 + r - kWrBM, p.N - 1) * K + (size_t)wave * kWrKS + sw;
  }
  uint16_t* ring = lds + wave * S * kWrStageElems;
  auto request = [&](int i, int st) {  // this wave's slab i (clamped: a harmless re-load) into its stage st
    const int at = min(i, ns - 1) + rot;
    const int ofs = (at < ns ? at : at - ns) * NW * kWrKS;
    uint16_t* dst = ring + st * kWrStageElems;
#pragma unroll
    for (int j = 0; j < kWrLoads; ++j) {
      if (j < kWrBM / 8)  // activation rows
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + ofs),
                                         (__attribute__((address_space(3))) void*)(dst + j * 512), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + ofs),
                                         (__attribute__((address_space(3))) void*)(dst + j * 512), 16, 0, kWeightAux);
    }
  };

  floatx4 acc[NT][MT];  // [weight row tile a][activation row tile t]
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[a][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  // fragment of k-step s (32 k): lane (row r = lane%16 of a 16-row tile, quarter q = lane/16) reads chunk 4s+q
  int fo[2];
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2)
    fo[s2] = (lane & 15) * kWrKS + (((4 * s2 + (lane >> 4)) ^ (((lane & 15) >> 1) & 7)) * 8);

  constexpr int MINE = (NT + NW - 1) / NW;  // weight row tiles a wave finishes
  Epilogue4<MINE, MT> epi;
  epi.request(p, lane, [&](int i) { return n0 + 16 * (wave + i * NW); });
#pragma unroll
  for (int i = 0; i < S - 1; ++i) request(i, i);
  int st = 0, st_in = S - 1;  // stage read in this iteration; stage the newest request goes into
  for (int i = 0; i < ns; ++i) {
    request(i + S - 1, st_in);            // that stage was last read in iteration i-1
    sk_wait_vmcnt<(S - 1) * kWrLoads>();  // slab i has landed (the S-1 younger ones may still fly)
    const uint16_t* sb = ring + st * kWrStageElems;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      u32x4 xf[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) xf[t] = *reinterpret_cast<const u32x4*>(sb + t * 16 * kWrKS + fo[s2]);
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        const u32x4 wf = *reinterpret_cast<const u32x4*>(sb + (kWrBM + a * 16) * kWrKS + fo[s2]);
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf),
                                                              __builtin_bit_cast(bf16x8, xf[t]), acc[a][t], 0, 0, 0);
      }
    }
    st = st + 1 == S ? 0 : st + 1;
    st_in = st_in + 1 == S ? 0 : st_in + 1;
  }
  epi.pages(p, lane);
  sk_wait_vmcnt<0>();  // the clamped re-load of the last iteration must not land in the reduction area
  __syncthreads();     // every wave is done with its ring: reuse the LDS to add the four waves' tiles
  {
    floatx4* red = reinterpret_cast<floatx4*>(lds);  // [wave][a][t][64 lanes]
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
      for (int t = 0; t < MT; ++t) red[((wave * NT + a) * MT + t) * 64 + lane] = acc[a][t];
    __syncthreads();
  }
  // wave w finishes weight row tiles a = w (and w + 4): the four waves' tiles are added in wave order.
  // Lane: row m = 16t + lane%16, columns n = n0 + 16a + 4*(lane/16) + 0..3.
  const floatx4* red = reinterpret_cast<const floatx4*>(lds);
  const OutSegments out = out_segments(p, p.seg_cols);
#pragma unroll
  for (int i = 0; i < MINE; ++i) {
    const int a = wave + i * NW;
    const int n = n0 + 16 * a + (lane >> 4) * 4;
    if (a >= NT || n >= p.N) continue;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int m = t * 16 + (lane & 15);
      if (m >= p.M) continue;
      floatx4 v = red[((0 * NT + a) * MT + t) * 64 + lane];
#pragma unroll
      for (int w2 = 1; w2 < NW; ++w2) v += red[((w2 * NT + a) * MT + t) * 64 + lane];
      epi.store(p, out, i, t, m, n, v);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Short products (up to 64 rows, up to some MB of weights: layers of 256 to 1024 features).  Such a launch is
// its own start, one memory latency and its end; what made it longer were the bytes of a workgroup (64 columns and 64
// rows of X, most of them copies, through a single compute unit) and a ring that takes them one barrier after another.
// So the waves split K among themselves as above, but a workgroup owns 16 columns and there is no ring: a lane asks for
// all pieces of its wave's share at once, straight into the registers that the matrix instructions read.
//
// With LN the rows of X are normalised on the way (norm_gamma, norm_beta): every workgroup computes the rows' mean and
// variance for itself, as layernorm_kernel does for rows of up to 512 elements, sum by sum in the same order, and
// each lane normalises the pieces it multiplies, so the bits are those of a launch of its own.
//
// NT = 1 column tile a workgroup (the first parameter as at wring_gemm_kernel: what ran is read off the kernels' names); MT
// row tiles (blockIdx.y: which); C = slabs of 64 a wave asks for at once, K is a multiple of that many for
// every wave, or C = 1.
// ---------------------------------------------------------------------------------------------
constexpr int kShortWaves = 4;
constexpr int kShortNormK = 512;  // one 16-byte piece of a row per lane

template <int NT, int MT, int C, bool LN>
__global__ __launch_bounds__(64 * kShortWaves) void short_wring_gemm_kernel(const SkinnyParams p) {
  static_assert(NT == 1, "16 columns a workgroup");
  constexpr int NW = kShortWaves, BM = 16 * MT, ROWS = LN ? BM / NW : 1;
  __shared__ floatx4 red[NW][MT][64];
  __shared__ float mean_s[BM], rstd_s[BM];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, q = lane >> 4;  // row of a fragment, its quarter of 32 k
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * BM, K = p.K, slabs = K / kWrKS;
  const uint16_t* wrow = p.W + (size_t)min(n0 + r, p.N - 1) * K + 8 * q;
  const uint16_t* xrow[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) xrow[t] = p.X + (size_t)min(m0 + 16 * t + r, p.M - 1) * K + 8 * q;

  // whole rows for their statistics: wave w has rows w, w + NW, ...
  u32x4 raw[ROWS];
  if constexpr (LN) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
      raw[i] = ld16(p.X + (size_t)min(m0 + wave + NW * i, p.M - 1) * K + min(lane, K / 8 - 1) * 8);
  }
  Epilogue4<1, 1> epi;  // wave w finishes row tile w
  epi.first = m0 + 16 * min(wave, MT - 1);
  floatx4 acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  float mean[MT], rstd[MT];
  for (int s0 = wave; s0 < slabs; s0 += NW * C) {
    u32x4 wf[C][2], xf[C][2][MT], gf[C][2], bf[C][2];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int k0 = (s0 + NW * c) * kWrKS;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        wf[c][h] = ld16(wrow + k0 + 32 * h);
#pragma unroll
        for (int t = 0; t < MT; ++t) xf[c][h][t] = ld16(xrow[t] + k0 + 32 * h);
        if constexpr (LN) {
          gf[c][h] = ld16(p.norm_gamma + k0 + 32 * h + 8 * q);
          bf[c][h] = ld16(p.norm_beta + k0 + 32 * h + 8 * q);
        }
      }
    }
    if (s0 == wave) epi.request(p, lane, [&](int) { return n0; });
    __builtin_amdgcn_sched_barrier(0);  // all of them on their way before the first is waited for
    if constexpr (LN) {
      if (s0 == wave) {  // statistics first; every wave comes here once (slabs >= NW)
        const bool live = lane < K / 8;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
          if (i > 0 && m0 + NW * i >= p.M) break;  // no such rows (256 features, step of 1 row 16.0 -> 14.4 us)
          float v[8], sum = 0.f, sq = 0.f;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            v[2 * j] = bf16_lo(raw[i][j]);
            v[2 * j + 1] = bf16_hi(raw[i][j]);
            sum += live ? v[2 * j] + v[2 * j + 1] : 0.f;
          }
          const float mu = wave_sum(sum) / (float)K;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float d = v[j] - mu;
            sq += live ? d * d : 0.f;
          }
          const float rs = rsqrtf(wave_sum(sq) / (float)K + p.norm_eps);
          if (lane == 0) {
            mean_s[wave + NW * i] = mu;
            rstd_s[wave + NW * i] = rs;
          }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          mean[t] = mean_s[16 * t + r];
          rstd[t] = rstd_s[16 * t + r];
        }
      }
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int t = 0; t < MT; ++t) {
            u32x4& x = xf[c][h][t];
#pragma unroll
            for (int j = 0; j < 4; ++j)
              x[j] = pack_bf16((bf16_lo(x[j]) - mean[t]) * rstd[t] * bf16_lo(gf[c][h][j]) + bf16_lo(bf[c][h][j]),
                               (bf16_hi(x[j]) - mean[t]) * rstd[t] * bf16_hi(gf[c][h][j]) + bf16_hi(bf[c][h][j]));
          }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[c][h]),
                                                           __builtin_bit_cast(bf16x8, xf[c][h][t]), acc[t], 0, 0, 0);
    }
  }
  epi.pages(p, lane);
  // the waves' parts are added in wave order
  const int n = n0 + q * 4;
#pragma unroll
  for (int t = 0; t < MT; ++t) red[wave][t][lane] = acc[t];
  __syncthreads();
  if (wave >= MT || n >= p.N) return;
  const int m = m0 + 16 * wave + r;
  if (m >= p.M) return;
  floatx4 v = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < NW; ++w) v += red[w][wave][lane];
  epi.store(p, out_segments(p, p.seg_cols), 0, 0, m, n, v);
}

// Sum of the split partials of 8 consecutive columns of row m, added in split order.  The reduce passes are bound by
// latency, one round trip after another: the loads of up to U splits are issued together, and what the epilogue needs
// besides is requested before them (epi_load) instead of after the sum.  64 rows of 5120: 4.7 -> 4.5 us, with
// LayerNorm 5.7 -> 5.2; decode step of OPT-13B at 1 row 130.7 -> 129.8, at 64 rows 268.9 -> 267.3.
template <int U>
__device__ __forceinline__ void sum_partials8_by(const SkinnyParams& p, int n_splits, int m, int n, float v[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = 0.f;
  for (int s0 = 0; s0 < n_splits; s0 += U) {
    floatx4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float* src = p.partial + ((size_t)min(s0 + u, n_splits - 1) * p.M + m) * p.N + n;
      a[u] = *reinterpret_cast<const floatx4*>(src);
      b[u] = *reinterpret_cast<const floatx4*>(src + 4);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < n_splits) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] += a[u][j];
          v[4 + j] += b[u][j];
        }
      }
    }
  }
}

__device__ __forceinline__ void sum_partials8(const SkinnyParams& p, int n_splits, int m, int n, float v[8]) {
  if (n_splits <= 4) sum_partials8_by<4>(p, n_splits, m, n, v);
  else sum_partials8_by<8>(p, n_splits, m, n, v);
}

// Bias and residual of 8 columns.  An absent operand is read from the partials instead and not used: a branch around
// the load would end in a wait for it.
struct EpiPieces {
  u32x4 bias, res;
};
__device__ __forceinline__ EpiPieces epi_load(const SkinnyParams& p, int m, int n) {
  const uint16_t* any = reinterpret_cast<const uint16_t*>(p.partial);
  EpiPieces e;
  e.bias = ld16((p.bias ? p.bias : any) + n);
  e.res = ld16((p.residual ? p.residual : any) + (size_t)m * p.N + n);
  return e;
}
__device__ __forceinline__ void epi_apply(const SkinnyParams& p, const EpiPieces& e, float v[8]) {
  if (p.bias) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] += bf16_lo(e.bias[j]);
      v[2 * j + 1] += bf16_hi(e.bias[j]);
    }
  }
  if (p.relu) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = fmaxf(v[j], 0.f);
  }
  if (p.residual) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] += bf16_lo(e.res[j]);
      v[2 * j + 1] += bf16_hi(e.res[j]);
    }
  }
}

// Sum the split partials in split order, then bias / ReLU / residual, 8 columns per thread.
__global__ __launch_bounds__(256) void skinny_reduce_kernel(const SkinnyParams p, int n_splits) {
  const int chunks_per_row = p.N >> 3;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)p.M * chunks_per_row) return;
  const int m = (int)(idx / chunks_per_row);
  const int n = (int)(idx % chunks_per_row) * 8;
  const EpiPieces e = epi_load(p, m, n);
  float v[8];
  sum_partials8(p, n_splits, m, n, v);
  epi_apply(p, e, v);
  u32x4 ov;
#pragma unroll
  for (int j = 0; j < 4; ++j) ov[j] = pack_bf16(v[2 * j], v[2 * j + 1]);
  st16(out_segments(p, p.seg_cols).at(m, n), ov);
}

// The same reduction, one workgroup per output row, followed by LayerNorm of that row: writes
// out[0][m,:] = act(sum + bias) + residual (bf16) and ln_out[m,:] = LN(out[m,:]) (statistics in
// fp32 over the bf16-rounded row, exactly what the stand-alone LayerNorm kernel would see).
// 1024 threads per row so that a 5120-wide row is one 8-column piece per thread and all partial loads of a
// row are in flight together (the kernel is pure latency: 64 rows, a few hundred KB each).
constexpr int kRedLnThreads = 1024;
constexpr int kRedLnMaxChunks = 2;  // 2 pieces x 8 columns x 1024 threads = 16384 columns
template <int NCH>
__global__ __launch_bounds__(kRedLnThreads) void skinny_reduce_ln_kernel(const SkinnyParams p, int n_splits,
                                                                         const uint16_t* __restrict__ gamma,
                                                                         const uint16_t* __restrict__ beta, float eps,
                                                                         uint16_t* __restrict__ ln_out) {
  __shared__ float red[kRedLnThreads / 64];
  const int m = blockIdx.x;
  const int nchunk = p.N >> 3;
  EpiPieces e[NCH];
  u32x4 gam[NCH], bet[NCH];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = min((int)threadIdx.x + i * kRedLnThreads, nchunk - 1);
    e[i] = epi_load(p, m, c * 8);
    gam[i] = ld16(gamma + c * 8);
    bet[i] = ld16(beta + c * 8);
  }
  float vals[NCH][8];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = threadIdx.x + i * kRedLnThreads;
    if (c < nchunk) {
      const int n = c * 8;
      float v[8];
      sum_partials8(p, n_splits, m, n, v);
      epi_apply(p, e[i], v);
      u32x4 ov;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ov[j] = pack_bf16(v[2 * j], v[2 * j + 1]);
        vals[i][2 * j] = bf16_lo(ov[j]);
        vals[i][2 * j + 1] = bf16_hi(ov[j]);
        sum += vals[i][2 * j] + vals[i][2 * j + 1];
      }
      st16(p.out[0] + (size_t)m * p.N + n, ov);
    }
  }
  auto block_sum = [&](float v) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kRedLnThreads / 64; ++w) t += red[w];
    return t;
  };
  const float mean = block_sum(sum) / (float)p.N;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = threadIdx.x + i * kRedLnThreads;
    if (c < nchunk) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float d = vals[i][j] - mean;
        sq += d * d;
      }
    }
  }
  const float rstd = rsqrtf(block_sum(sq) / (float)p.N + eps);
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = threadIdx.x + i * kRedLnThreads;
    if (c < nchunk) {
      u32x4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float lo = (vals[i][2 * j] - mean) * rstd * bf16_lo(gam[i][j]) + bf16_lo(bet[i][j]);
        const float hi = (vals[i][2 * j + 1] - mean) * rstd * bf16_hi(gam[i][j]) + bf16_hi(bet[i][j]);
        o[j] = pack_bf16(lo, hi);
      }
      st16(ln_out + (size_t)m * p.N + c * 8, o);
    }
  }
}

// The same reduction for the decode QKV projection (N = (n + 2 n_kv) s, one output buffer with row stride N):
// the Q part is written to out[0]; the K and V parts are this step's new cache rows and go to
// slot ctx_lens[m] of the paged cache [num_blocks, n_kv, 16, s].
__global__ __launch_bounds__(256) void skinny_reduce_kv_kernel(const SkinnyParams p, int n_splits,
                                                               const int32_t* __restrict__ ctx_lens,
                                                               const int32_t* __restrict__ block_tables,
                                                               int max_blocks, uint16_t* __restrict__ k_cache,
                                                               uint16_t* __restrict__ v_cache, int n_heads,
                                                               int n_kv_heads, int head_dim) {
  const int chunks_per_row = p.N >> 3;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)p.M * chunks_per_row) return;
  const int m = (int)(idx / chunks_per_row);
  const int n = (int)(idx % chunks_per_row) * 8;
  const EpiPieces e = epi_load(p, m, n);
  const int pos = ctx_lens[m];
  const int blk = block_tables[(size_t)m * max_blocks + pos / 16];
  float v[8];
  sum_partials8(p, n_splits, m, n, v);
  epi_apply(p, e, v);
  u32x4 ov;
#pragma unroll
  for (int j = 0; j < 4; ++j) ov[j] = pack_bf16(v[2 * j], v[2 * j + 1]);
  const int h = n_heads * head_dim, hkv = n_kv_heads * head_dim;
  if (n < h) {
    st16(p.out[0] + (size_t)m * p.N + n, ov);
    return;
  }
  const int which = n >= h + hkv;
  const int col = n - h - which * hkv;
  const int head = col / head_dim, d = col - head * head_dim;
  uint16_t* dst = (which ? v_cache : k_cache) + (((size_t)blk * n_kv_heads + head) * 16 + (pos % 16)) * head_dim + d;
  st16(dst, ov);
}

DS_SWITCH(g_skinny_force_ntw, 0);  // 0 = byte model
DS_SWITCH(g_skinny_force_splits, 0);

struct SkinnyPlan {
  int ntw;     // column tiles per wave: BN = 64 * ntw
  int splits;  // K splits over workgroups
};

constexpr double kReduceBytes = 57e6;  // what a reduce launch costs, in bytes of the chip's stream (4 us)

// Measured on MI355X: a CU sustains about one workgroup's worth of streaming whatever the LDS would
// allow, and a second round of workgroups costs a full round.  So a plan must fit one round
// (<= 256 workgroups) and should fill it; among such plans take the fewest bytes through the CUs' L1:
//   weights + (N/BN) * X (each column block re-reads the activations) + partial sums written and
//   read back.
static SkinnyPlan skinny_plan(int M, int N, int K, bool allow_split = true, double* cost_out = nullptr) {
  const int slabs = K / kSkPlanK;
  const int mp = M <= 64 ? 64 : (M <= 128 ? 128 : 256);
  SkinnyPlan best{1, 1};
  double best_cost = 1e300;
  for (int ntw = 1; ntw <= 4; ntw *= 2) {
    if (g_skinny_force_ntw > 0 && ntw != g_skinny_force_ntw) continue;
    const int bn = 64 * ntw;
    // Wider tiles than these are not instantiated: four stages of 256 + 128 or of 128 + 256 rows do not fit the LDS.
    // (Three do, 144 KB; not tried.  More than 128 rows come here for the greedy choice only.)
    if (mp == 256 && ntw > 1) continue;
    if (mp == 128 && ntw > 2) continue;
    const int wgs_n = (N + bn - 1) / bn;
    for (int splits = 1; splits <= slabs && splits <= 64; ++splits) {
      if (!allow_split && splits > 1) break;
      if (allow_split && g_skinny_force_splits > 0 && splits != g_skinny_force_splits) continue;
      const double wgs = (double)wgs_n * splits;
      const bool forced = g_skinny_force_splits > 0;
      if (wgs > 256.0 && splits > 1 && !forced) break;        // never split into a second round
      const double rounds = wgs <= 256.0 ? 1.0 : ceil(wgs / 256.0);  // unsplit but larger than the chip: whole rounds
      const double fill = wgs >= 256.0 ? 1.0 : 256.0 / wgs;    // idle CUs stretch the time
      // partial sums are charged four times their bytes: they are stored by every workgroup at once at
      // the end of the launch and read back by a second, latency-bound launch (measured: 6 splits of
      // 128 columns beat 12 splits of 256 on the FFN-out shape although they stream more activations; charged
      // for the padded row count, since a workgroup's partial-tile epilogue costs the same at 16 rows as at 64)
      const double bytes = 2.0 * N * K + 2.0 * wgs_n * (double)mp * K +
                           (splits > 1 ? 4.0 * 2.0 * 4.0 * splits * (double)mp * N : 0.0);
      const double cost = bytes * fill * rounds;
      if (cost < best_cost) {
        best_cost = cost;
        best = SkinnyPlan{ntw, splits};
      }
    }
  }
  if (cost_out) *cost_out = best_cost + (best.splits > 1 ? kReduceBytes : 0.0);
  return best;
}

// What the unsplit ring kernel with 64 columns a workgroup costs, in the same bytes; rows that only repeat the last one
// are left out (they come from one line).
static double unsplit_bytes(int M, int N, int K) {
  const int wgs = (N + 63) / 64, rows = (M + 15) / 16 * 16;
  return (2.0 * N * K + 2.0 * wgs * rows * (double)K) * (wgs >= 256 ? (wgs + 255) / 256 : 256.0 / wgs);
}

size_t skinny_workspace_bytes(int M, int N, int K) {
  if (K % kSkPlanK != 0 || M > 256) return 0;
  const SkinnyPlan pl = skinny_plan(M, N, K);  // (also covers the shapes the unsplit kernel takes)
  return pl.splits > 1 ? (size_t)pl.splits * M * N * sizeof(float) : 0;
}

// Stages of 16 MT + 16 NT rows that the LDS has room for (more than eight gain nothing).
constexpr int ring_stages(int MT, int NT) {
  const int fit = 160 * 1024 / ((MT + NT) * 16 * kSkKS * 2);
  return fit < 8 ? fit : 8;
}
template <int MT, int NTW, int NT = 4 * NTW>
static hipError_t launch_skinny_cfg(SkinnyParams p, int splits, hipStream_t stream) {
  p.splits = splits;
  constexpr int BN = 16 * NT, S = ring_stages(MT, NT);
  constexpr size_t lds_bytes = (size_t)S * (MT * 16 + BN) * kSkKS * sizeof(uint16_t);
  static_assert(lds_bytes <= 160 * 1024, "LDS");
  static_assert((size_t)4 * NTW * MT * 64 * 16 + (size_t)4 * MT * 16 * 8 <= lds_bytes,
                "k-half reduction (and the greedy-choice candidates behind it) fit the stages");
  constexpr auto kern = skinny_gemm_kernel<MT, NTW, S, NT>;
  (void)KernelAttrReg<kern, (int)lds_bytes>::done;
  hipLaunchKernelGGL(kern, dim3((p.N + BN - 1) / BN, splits), dim3(kSkThreads), lds_bytes, stream, p);
  return hipGetLastError();
}

template <int NT, int MT, int S, int NW>
static hipError_t launch_wring_cfg(const SkinnyParams& p, hipStream_t stream) {
  constexpr size_t lds_bytes = (size_t)NW * S * (16 * MT + 16 * NT) * kWrKS * sizeof(uint16_t);  // NW waves x S stages
  static_assert(lds_bytes <= 160 * 1024 && (size_t)NW * NT * MT * 1024 <= lds_bytes, "LDS");
  constexpr auto kern = wring_gemm_kernel<NT, MT, S, NW>;
  (void)KernelAttrReg<kern, (int)lds_bytes>::done;
  hipLaunchKernelGGL(kern, dim3((p.N + 16 * NT - 1) / (16 * NT)), dim3(64 * NW), lds_bytes, stream, p);
  return hipGetLastError();
}

// The instantiation for NT column tiles and the batch's row count.
static hipError_t launch_wring(int nt, const SkinnyParams& p, hipStream_t stream) {
  const int M = p.M;
  if (nt == 5) {
    if (M <= 16) return launch_wring_cfg<5, 1, 3, 4>(p, stream);  // 144 KB
    if (M <= 32) return launch_wring_cfg<5, 2, 2, 4>(p, stream);  // 112 KB
    if (M <= 64) return launch_wring_cfg<5, 4, 2, 4>(p, stream);  // 144 KB
    return launch_wring_cfg<5, 8, 2, 3>(p, stream);               // 156 KB
  }
  if (M <= 16) return launch_wring_cfg<4, 1, 3, 4>(p, stream);    // 120 KB
  if (M <= 32) return launch_wring_cfg<4, 2, 3, 4>(p, stream);    // 144 KB
  return launch_wring_cfg<4, 4, 2, 4>(p, stream);                 // 128 KB (wring_tiles: at most 64 rows)
}

template <int MT, int C>
static hipError_t launch_short_cfg(const SkinnyParams& p, hipStream_t stream) {
  const dim3 grid((p.N + 15) / 16, (p.M + 16 * MT - 1) / (16 * MT)), block(64 * kShortWaves);
  if constexpr (MT == 1 && C * kShortWaves * kWrKS <= kShortNormK)
    if (p.norm_gamma) {
      hipLaunchKernelGGL((short_wring_gemm_kernel<1, MT, C, true>), grid, block, 0, stream, p);
      return hipGetLastError();
    }
  hipLaunchKernelGGL((short_wring_gemm_kernel<1, MT, C, false>), grid, block, 0, stream, p);
  return hipGetLastError();
}
template <int MT>
static hipError_t launch_short_rows(const SkinnyParams& p, hipStream_t stream) {
  constexpr int kAll = kShortWaves * kWrKS;
  if (p.K % (4 * kAll) == 0) return launch_short_cfg<MT, 4>(p, stream);
  if (p.K % (2 * kAll) == 0) return launch_short_cfg<MT, 2>(p, stream);
  return launch_short_cfg<MT, 1>(p, stream);
}

// Whether a product of a layer is short: up to 1024 of K, so that a lane holds its whole share, and 8.5 MB of weights.  A
// decoding step (us, of a graph of 24) by the former kernels, with short products, with those that normalise too:
//   256 x 1024 features, 1 row 24.7, 17.1, 14.4; 16 rows 25.3, 19.1, 17.0; 64 rows 31.1, 19.9, 17.5
//   512 x 2048            1 row 29.3, 21.0, 18.2; 16 rows 30.9, 23.9, 21.7; 64 rows 38.6, 28.6, 27.2
//   1024 x 4096           1 row 32.8, 26.1, -;    64 rows 48.8, 41.4, -
// 1024 x 8192 (17 MB): 1 row 32.2 without it, 32.4 with; 64 rows 52.4 and 53.7.  K = 2048 -> 512 features: 1 row 24.1
// and 22.0, 64 rows 48.3 and 51.3; K = 4096 -> 1024: 29.8 and 30.1, 47.6 and 58.1.  (One line for all row counts, so that a
// row's bits do not depend on them.)
DS_SWITCH(g_skinny_short_k, 1024);   // longest K
DS_SWITCH(g_skinny_short_kb, 8500);  // most weights (KB)
static bool short_product(int M, int N, int K) {
  return M <= 64 && K >= kShortWaves * kWrKS && K % kWrKS == 0 && K <= g_skinny_short_k && 2e-3 * N * K <= g_skinny_short_kb;
}
// Whether each 16 rows of a short product have workgroups of their own, which read the weights again: as long as that
// is no more than a short product may have of them.  Many small workgroups start their loads together where one that
// holds all rows is one load path for 64 rows of X: steps at 64 rows of 256 features 25.1 -> 19.9 us, of 512 31.0 ->
// 28.6, of 1024 44.2 -> 41.4 (32 rows 35.4 -> 34.4; its QKV and FFN-in, 25 and 34 MB that way for 6.3 and 8.4, apart
// too: 45.0 and 36.2).
static bool short_rows_apart(int M, int N, int K) { return 2e-3 * N * K * ((M + 15) / 16) <= g_skinny_short_kb; }
// Rows are normalised where they lie apart, every workgroup of theirs for itself (all 64 rows' statistics in each
// workgroup cost more than the launch that is saved): 19.9 -> 17.5 us at 64 rows of 256, 28.6 -> 27.2 of 512.
bool skinny_norms_input(int M, int N, int K) {
  return K <= kShortNormK && short_product(M, N, K) && short_rows_apart(M, N, K);
}
static hipError_t launch_short(const SkinnyParams& p, hipStream_t stream) {
  if (p.M <= 16 || short_rows_apart(p.M, p.N, p.K)) return launch_short_rows<1>(p, stream);
  if (p.M <= 32) return launch_short_rows<2>(p, stream);
  return launch_short_rows<4>(p, stream);
}

// Column-tile width (in 16-row tiles) for the wave-private-ring kernel, or 0 if the shape is not one it
// is good at: K a multiple of 256 and enough column tiles to occupy most of the chip without splitting K.
// Up to 64 rows it takes both widths; for 65..128 rows only the 80-column one, where a workgroup re-reads 1.6
// activation bytes per weight byte rather than 2 (measured at 128 rows against the ring kernel: FFN-in of OPT-13B 55 us
// and 64, of OPT-66B 166 and 201, QKV of OPT-175B 217 and 268; every 64-column shape was equal or up to 20 % slower).
DS_SWITCH(g_skinny_wring, 1);  // 0 = never use the wave-private-ring kernel, 2 = also where it needs several rounds
static int wring_tiles(int M, int N, int K) {
  if (!g_skinny_wring || M > 128 || K < 256 || K % 256 != 0) return 0;
  const int t4 = (N + 63) / 64, t5 = (N + 79) / 80;
  const int r4 = (t4 + 255) / 256, r5 = (t5 + 255) / 256;
  const int nt = r5 < r4 ? 5 : 4;
  const int tiles = nt == 5 ? t5 : t4;
  if (M > 64 && nt != 5) return 0;
  if (tiles < 160) return 0;
  // Several rounds of workgroups: each of them streams the activation slab again beside its 64 or 80 weight
  // rows, and from 32 rows up that is as many bytes through a compute unit's load path as the weights.  The
  // split-K ring kernel with 256-column tiles reads a quarter of that and stays within one round; it wins where
  // its bytes (in skinny_plan's terms, reduce launch included) are clearly fewer.  Measured at 64 rows: FFN-in of
  // OPT-175B 219 -> 203 us, QKV of OPT-66B 107 -> 93 us; QKV of OPT-175B and FFN-in of OPT-66B (two rounds of 80
  // columns against 144 workgroups of 256) stay here, 171 against 184 and 134 against 137.
  // A single round that leaves a fifth of the chip idle is compared the same way: 12288 x 49152 on 192 workgroups at
  // 17, 32 and 64 rows 200, 218 and 260 us, 48 x 5 split 185, 187 and 194; 12288 x 12288 at 48 and 64 rows 71 and 76,
  // split 58 and 58; 10240 x 8192 on 160 at 48 and 64 rows 46 and 48, split 37 and 37.5.  15360 x 5120 on 240 is not:
  // 32.5 and 34.9 at 48 rows, 34.6 and 37.4 at 64.
  const int rounds = nt == 5 ? r5 : r4;
  if ((rounds > 1 || tiles < 208) && M > 16 && g_skinny_wring != 2) {
    const double rows = M <= 32 ? 32 : (M <= 64 ? 64 : 128);
    const double wring_cost = rounds * 256.0 * (16.0 * nt + rows) * K * 2.0;
    double ring_cost;
    skinny_plan(M, N, K, true, &ring_cost);
    if (ring_cost < 0.95 * wring_cost) return 0;
  }
  return nt;
}

// Activation rows of a stage: the batch's, up to 16, 32 or 64 (the last row again makes up the rest; with 64 for every
// batch the token loop's two ends took 91.8 us at 1 row; 85.8 with these and the tiles of `greedy_tiles`).
template <int NTW, int NT = 4 * NTW>
static hipError_t dispatch_skinny_rows(const SkinnyParams& p, int splits, hipStream_t stream) {
  if (p.M <= 16) return launch_skinny_cfg<1, NTW, NT>(p, splits, stream);
  if (p.M <= 32) return launch_skinny_cfg<2, NTW, NT>(p, splits, stream);
  return launch_skinny_cfg<4, NTW, NT>(p, splits, stream);
}
static hipError_t dispatch_skinny(const SkinnyParams& p, const SkinnyPlan& pl, hipStream_t stream) {
  if (p.M <= 64) {
    if (pl.ntw == 4) return dispatch_skinny_rows<4>(p, pl.splits, stream);
    if (pl.ntw == 2) return dispatch_skinny_rows<2>(p, pl.splits, stream);
    return dispatch_skinny_rows<1>(p, pl.splits, stream);
  }
  if (p.M <= 128) {
    if (pl.ntw == 2) return launch_skinny_cfg<8, 2>(p, pl.splits, stream);
    return launch_skinny_cfg<8, 1>(p, pl.splits, stream);
  }
  return launch_skinny_cfg<16, 1>(p, pl.splits, stream);
}

hipError_t launch_argmax_merge(const float* part_val, const int32_t* part_idx, int n_blocks, int M,
                               int32_t* next_token, float* best_logit, hipStream_t stream);

// Tiles of 16 columns that a workgroup of the greedy choice takes: what one CU streams over all rounds of workgroups is
// smallest.  The launch is not split, so with 64, 128 and 256 columns alone 50272 x 5120 left 59 of the 256 CUs idle (197
// tiles of 256); a CU has only so much in flight, and 242 tiles of 208 bring 515 MB in faster: with the embedding and
// the LayerNorm 104.1 -> 97.0 us at 64 rows.  Reckoned for 64 rows whatever the batch has, so that a workspace for
// many rows is enough for fewer.  Other vocabularies (5120 features, with the LayerNorm, at 1 and 64 rows, from 64, 128
// and 256 columns alone): 32000 ids 57.9 -> 54.7 and 65.9 -> 64.7, 65024 107 -> 102 and 113 -> 112, 100352 178 -> 157 and
// 194 -> 175, 128256 202 -> 194 and level, 152064 270 -> 233 and 290 -> 259; none slower, at 1024 to 12288 features.  Of
// the widths on offer the rule takes the fastest there, or one within 2 %.  Where rows are a power of two apart it can miss
// (the channels of the memory count then): 4096 features, 65024 ids at 1 row 123 with its 256 columns, 98 with 64.
static int greedy_tiles(int M, int N, int K) {
  int best = 4 * skinny_plan(M, N, K, false).ntw;
  if (M > 64 || g_skinny_force_ntw > 0) return best;
  double best_cost = 1e300;
  for (int nt : {4, 8, 10, 12, 13, 14, 16}) {
    const int wgs = (N + 16 * nt - 1) / (16 * nt);
    const double cost = ((wgs + 255) / 256) * (16.0 * nt + 64);
    if (cost < best_cost) best_cost = cost, best = nt;
  }
  return best;
}

static size_t candidate_bytes(int M, int N, int tiles) {
  const size_t blocks = (size_t)(N + 16 * tiles - 1) / (16 * tiles);
  return blocks * M * (sizeof(float) + sizeof(int32_t));
}
size_t skinny_argmax_workspace_bytes(int M, int N, int K) {
  if (K % kSkPlanK != 0 || M > 256 || M <= 0 || N <= 0) return 0;
  return candidate_bytes(M, N, greedy_tiles(M, N, K));
}
// With the 64, 128 or 256 columns of the product's own plan, taken where a workspace has no room for the candidates of
// the tiles above (the same values in either).
size_t skinny_argmax_least_bytes(int M, int N, int K) {
  if (K % kSkPlanK != 0 || M > 256 || M <= 0 || N <= 0) return 0;
  return std::min(skinny_argmax_workspace_bytes(M, N, K), candidate_bytes(M, N, 4 * skinny_plan(M, N, K, false).ntw));
}

hipError_t launch_skinny_argmax(const void* X, const void* W, int M, int N, int K, void* workspace, size_t workspace_bytes,
                                int32_t* next_token, float* best_logit, hipStream_t stream) {
  if (M <= 0 || M > 256 || N <= 0 || K % kSkPlanK != 0 || !workspace || !next_token ||
      workspace_bytes < skinny_argmax_least_bytes(M, N, K))
    return hipErrorInvalidValue;
  const bool fits = workspace_bytes >= skinny_argmax_workspace_bytes(M, N, K);
  const int tiles = fits ? greedy_tiles(M, N, K) : 4 * skinny_plan(M, N, K, false).ntw;
  const int blocks = (N + 16 * tiles - 1) / (16 * tiles);
  SkinnyParams p;
  p.X = (const uint16_t*)X;
  p.W = (const uint16_t*)W;
  p.bias = nullptr;
  p.residual = nullptr;
  for (int i = 0; i < 3; ++i) p.out[i] = nullptr;
  p.seg_cols = N;
  p.seg_cols_kv = N;
  p.M = M; p.N = N; p.K = K;
  p.relu = 0;
  p.partial = nullptr;
  p.amax_val = (float*)workspace;
  p.amax_idx = (int32_t*)(p.amax_val + (size_t)blocks * M);
  hipError_t e;
  switch (tiles) {
    case 10: e = dispatch_skinny_rows<3, 10>(p, 1, stream); break;
    case 12: e = dispatch_skinny_rows<3>(p, 1, stream); break;
    case 13: e = dispatch_skinny_rows<4, 13>(p, 1, stream); break;
    case 14: e = dispatch_skinny_rows<4, 14>(p, 1, stream); break;
    default: e = dispatch_skinny(p, SkinnyPlan{tiles / 4, 1}, stream);
  }
  if (e != hipSuccess) return e;
  return launch_argmax_merge(p.amax_val, p.amax_idx, blocks, M, next_token, best_logit, stream);
}

// Second pass of any split-K product: partial [splits][M][N] fp32 -> epilogue, optionally with the
// LayerNorm or KV-append work folded in (reported through *fused_done).
hipError_t launch_splitk_reduce(const float* partial, int splits, int M, int N, const Epilogue& ep,
                                const SkinnyFused* fused, bool* fused_done, hipStream_t stream) {
  if (fused_done) *fused_done = false;
  if (N % 8 != 0 || ep.seg_cols <= 0 || ep.seg_cols % 8 != 0 || ep.seg_cols_kv < 0 || ep.seg_cols_kv % 8 != 0)
    return hipErrorInvalidValue;
  SkinnyParams p;
  p.X = nullptr;
  p.W = nullptr;
  p.bias = (const uint16_t*)ep.bias;
  p.residual = (const uint16_t*)ep.residual;
  for (int i = 0; i < 3; ++i) p.out[i] = (uint16_t*)ep.out[i];
  p.seg_cols = ep.seg_cols;
  p.seg_cols_kv = ep.seg_cols_kv > 0 ? ep.seg_cols_kv : ep.seg_cols;
  p.M = M; p.N = N; p.K = 0;
  p.relu = ep.relu;
  p.partial = const_cast<float*>(partial);
  const long items = (long)M * (N / 8);
  const unsigned blocks = (unsigned)((items + 255) / 256);
  if (fused && fused->kind == SkinnyFused::kLayerNorm && ep.seg_cols == N &&
      N <= kRedLnThreads * 8 * kRedLnMaxChunks) {
    if (N <= kRedLnThreads * 8)
      hipLaunchKernelGGL(skinny_reduce_ln_kernel<1>, dim3(M), dim3(kRedLnThreads), 0, stream, p, splits,
                         (const uint16_t*)fused->ln_gamma, (const uint16_t*)fused->ln_beta, fused->ln_eps,
                         (uint16_t*)fused->ln_out);
    else
      hipLaunchKernelGGL(skinny_reduce_ln_kernel<2>, dim3(M), dim3(kRedLnThreads), 0, stream, p, splits,
                         (const uint16_t*)fused->ln_gamma, (const uint16_t*)fused->ln_beta, fused->ln_eps,
                         (uint16_t*)fused->ln_out);
    if (fused_done) *fused_done = true;
  } else if (fused && fused->kind == SkinnyFused::kKvAppend && ep.seg_cols == N && !ep.relu && !ep.residual &&
             N == (fused->n_heads + 2 * fused->n_kv_heads) * fused->head_dim) {
    hipLaunchKernelGGL(skinny_reduce_kv_kernel, dim3(blocks), dim3(256), 0, stream, p, splits, fused->ctx_lens,
                       fused->block_tables, fused->max_blocks, (uint16_t*)fused->k_cache,
                       (uint16_t*)fused->v_cache, fused->n_heads, fused->n_kv_heads, fused->head_dim);
    if (fused_done) *fused_done = true;
  } else {
    hipLaunchKernelGGL(skinny_reduce_kernel, dim3(blocks), dim3(256), 0, stream, p, splits);
  }
  return hipGetLastError();
}

// Which kernel takes a product: the one with wave-private rings (wring: 16-row tiles of W a workgroup, unsplit; 1: the
// one for short products), or, with wring = 0, the ring kernel by `plan`.  own_epilogue: no LayerNorm wants a reduce pass
// to ride in.
struct SkinnyRoute {
  int wring;
  SkinnyPlan plan;
};
static SkinnyRoute skinny_route(int M, int N, int K, bool own_epilogue, bool weigh_reduce) {
  if (weigh_reduce && short_product(M, N, K)) return SkinnyRoute{1, {1, 1}};
  SkinnyRoute r{own_epilogue ? wring_tiles(M, N, K) : 0, {1, 1}};
  if (r.wring > 0) return r;
  double split;
  r.plan = skinny_plan(M, N, K, true, &split);
  if (weigh_reduce && own_epilogue && r.plan.splits > 1 && unsplit_bytes(M, N, K) < split - kReduceBytes + 24e6)
    r.plan = SkinnyPlan{1, 1};
  return r;
}

void skinny_describe(int M, int N, int K, int* tile_cols, int* splits, bool own_epilogue, bool weigh_reduce) {
  const SkinnyRoute r = skinny_route(M, N, K, own_epilogue, weigh_reduce);
  *tile_cols = r.wring > 0 ? 16 * r.wring : 64 * r.plan.ntw;
  *splits = r.plan.splits;
}

// By the bytes the plans go by, fitted to 16 products at 65, 96 and 128 rows (within 10 %; 12288 x 49152 left out: two
// rounds of 128 columns, where it is a third too long).
double skinny_us(int M, int N, int K) {
  const int nt = wring_tiles(M, N, K);
  double bytes;
  if (nt > 0) {
    const int tiles = (N + 16 * nt - 1) / (16 * nt);
    bytes = (tiles + 255) / 256 * 256.0 * (16.0 * nt + (M <= 64 ? 64 : 128)) * K * 2.0;
  } else {
    skinny_plan(M, N, K, true, &bytes);
  }
  return 7.5 + (nt > 0 ? 0.0760e-6 : 0.0734e-6) * bytes * (1.0 + 0.088 * (M - 96) / 32.0);
}

hipError_t launch_skinny_gemm(const void* X, const void* W, int M, int N, int K, const Epilogue& ep,
                              void* workspace, hipStream_t stream, const SkinnyFused* fused, bool* fused_done,
                              bool weigh_reduce, const InputNorm* norm) {
  if (fused_done) *fused_done = false;
  if (M <= 0 || N <= 0) return hipSuccess;
  if (M > 256 || K % kSkPlanK != 0 || N % 8 != 0 || ep.seg_cols <= 0 || ep.seg_cols % 8 != 0 || ep.seg_cols_kv < 0 ||
      ep.seg_cols_kv % 8 != 0)
    return hipErrorInvalidValue;
  if (ep.residual && ep.seg_cols != N) return hipErrorInvalidValue;
  if (ep.x_ld != 0 || ep.out_ld != 0) return hipErrorInvalidValue;  // dense rows only
  SkinnyParams p;
  p.X = (const uint16_t*)X;
  p.W = (const uint16_t*)W;
  p.bias = (const uint16_t*)ep.bias;
  p.residual = (const uint16_t*)ep.residual;
  for (int i = 0; i < 3; ++i) p.out[i] = (uint16_t*)ep.out[i];
  p.seg_cols = ep.seg_cols;
  p.seg_cols_kv = ep.seg_cols_kv > 0 ? ep.seg_cols_kv : ep.seg_cols;
  p.M = M; p.N = N; p.K = K;
  p.relu = ep.relu;
  // wide N, few rows: unsplit, wave-private rings, K/V scatter in its own epilogue
  const bool plain = !fused || fused->kind == SkinnyFused::kNone;
  const bool want_kv = fused && fused->kind == SkinnyFused::kKvAppend && ep.seg_cols == N && !ep.relu &&
                       !ep.residual && N == (fused->n_heads + 2 * fused->n_kv_heads) * fused->head_dim &&
                       fused->head_dim % 4 == 0;
  const SkinnyRoute route = skinny_route(M, N, K, plain || want_kv, weigh_reduce);
  const SkinnyPlan pl = route.plan;
  if (want_kv && pl.splits == 1) {
    p.kv_ctx_lens = fused->ctx_lens; p.kv_block_tables = fused->block_tables; p.kv_max_blocks = fused->max_blocks;
    p.kv_k_cache = (uint16_t*)fused->k_cache; p.kv_v_cache = (uint16_t*)fused->v_cache;
    p.kv_n_heads = fused->n_heads; p.kv_n_kv_heads = fused->n_kv_heads; p.kv_head_dim = fused->head_dim;
    if (fused_done) *fused_done = true;
  }
  if (norm) {
    if (!weigh_reduce || !skinny_norms_input(M, N, K)) return hipErrorInvalidValue;
    p.norm_gamma = (const uint16_t*)norm->gamma;
    p.norm_beta = (const uint16_t*)norm->beta;
    p.norm_eps = norm->eps;
  }
  if (route.wring > 0) {
    p.partial = nullptr;
    if (route.wring == 1) return launch_short(p, stream);
    return launch_wring(route.wring, p, stream);
  }
  p.partial = (float*)workspace;
  if (pl.splits > 1 && workspace == nullptr) return hipErrorInvalidValue;
  hipError_t e = dispatch_skinny(p, pl, stream);
  if (e != hipSuccess) return e;
  if (pl.splits > 1) e = launch_splitk_reduce(p.partial, pl.splits, M, N, ep, fused, fused_done, stream);
  return e;
}

}  // namespace ds
