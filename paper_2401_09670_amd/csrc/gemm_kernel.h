// The MFMA tile kernel (template), its tiles and the launch of one: included by the sources that instantiate them.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace ds {

constexpr int kBK = 64;

// LDS a workgroup asks for: its ring of operand stages - or the whole 160 KB of the compute unit once the ring
// alone is more than half of it (a second workgroup could not move in anyway), which gives the epilogue a
// larger staging area: more columns per pass, longer contiguous row pieces in the output stores.
constexpr int gemm_lds_bytes(int BM, int BN, int XS, int WS) {
  const int ring = (XS * BM + WS * BN) * kBK * 2;
  return ring > 80 * 1024 ? 160 * 1024 : ring;
}

struct GemmParams {
  const uint16_t* X;
  const uint16_t* W;
  const uint16_t* bias;
  const uint16_t* residual;
  uint16_t* out[3];
  int seg_cols, seg_cols_kv;  // widths of the first and of the other two output segments
  int M, N, K;
  int relu;
  int tiles_m, tiles_n;
  int ldx;     // row stride of X in elements (>= K)
  int ld_out;  // row stride of out[0]
  int ld_res;  // row stride of residual
  int n_base;  // first output column of this launch (a launch may cover the columns [n_base, N) only)
  int spread;  // workgroups start at different places of K
  int splits;
  // Split-K (splits = gridDim.y = S > 1): split s multiplies k-tiles s, s + S, ... and stores its fp32
  // accumulators to partial[s][M][N]; the epilogue then belongs to whoever adds the partials.
  float* partial;
  // Decode QKV projection (N = (n_heads + 2 n_kv_heads) head_dim): with k_cache set, the K and V parts of
  // row m go to slot ctx_lens[m] of the paged cache [num_blocks, n_kv_heads, 16, head_dim] instead of `out`.
  const int32_t* ctx_lens;
  const int32_t* block_tables;
  int max_blocks;
  uint16_t* k_cache;
  uint16_t* v_cache;
  int n_heads, n_kv_heads, head_dim;
#ifdef DS_DEV_STAMPS
  unsigned long long* dbg;  // timing harness builds only: 4 wall-clock stamps per workgroup
#endif
};

#ifdef DS_DEV_STAMPS
inline unsigned long long* g_gemm_dbg = nullptr;
#define DS_STAMP(i)                                                                         \
  do {                                                                                      \
    if (p.dbg && threadIdx.x == 0) p.dbg[(size_t)(blockIdx.x + gridDim.x * blockIdx.y) * 4 + (i)] = __builtin_amdgcn_s_memrealtime(); \
  } while (0)
#else
#define DS_STAMP(i)
#endif

// Tile order.  Workgroup ids are dealt round-robin to the 8 XCDs (each with a private L2).  With one
// contiguous m-fastest range of tiles per XCD and many row tiles (long prefill batches), the 32 workgroups an
// XCD runs at a time share one weight tile and read 32 different activation tiles, and the eight XCDs sit in
// far-apart parts of the output, so every column tile re-streams the whole activation matrix from HBM.
// Instead, the 256 workgroups that run together (32 per XCD, ids dealt round-robin) take one patch of up to
// 16 x 16 output tiles, and inside it every XCD a block of 8 x 4: 16 + 16 operand tiles from HBM per 256 output
// tiles, 8 + 4 through each L2 per 32.  (A strip of 16 x 2 per XCD - 16 + 2 through each L2 - cost 1-3 % at 16384
// rows; with 8 row tiles the plain m-fastest order inside a chunk is the 8 x 4 block.)
constexpr int kXcd = 8, kPerXcd = 32, kChunk = kXcd * kPerXcd, kGroupM = 16;
__host__ __device__ constexpr void patch_tile(int pid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int full = total / kChunk * kChunk;
  int v = pid;
  if (pid < full) {
    const int xcd = pid % kXcd, slot = pid / kXcd;
    const int s = slot % kPerXcd;
    // the chunk's tiles are numbered m-fastest in groups of 16 rows: (row, column) = (number % 16, number / 16)
    v = slot / kPerXcd * kChunk + (tiles_m >= kGroupM ? ((xcd >> 1) * 4 + (s >> 3)) * kGroupM + (xcd & 1) * 8 + (s & 7)
                                                      : xcd * kPerXcd + s);
  } else {
    const int per = (total - full) / kXcd, q = pid - full;  // last, partial chunk: equal contiguous shares
    if (q < per * kXcd) v = full + (q % kXcd) * per + q / kXcd;
  }
  const int per_group = kGroupM * tiles_n;
  const int g = v / per_group;
  const int left = tiles_m - g * kGroupM, gsz = left < kGroupM ? left : kGroupM;
  const int r = v - g * per_group;
  tm = g * kGroupM + r % gsz;
  tn = r / gsz;
}

// The XCD whose workgroup takes row tile 0 of column tile tn (fewer than kGroupM row tiles).
__host__ __device__ constexpr int column_xcd(int tn, int tiles_m, int tiles_n) {
  const int total = tiles_m * tiles_n, full = total / kChunk * kChunk, v = tn * tiles_m;
  if (v < full) return v % kChunk / kPerXcd;
  const int per = (total - full) / kXcd;
  return v - full < per * kXcd ? (v - full) / per : (v - full) % kXcd;
}
constexpr bool column_xcd_follows_patch_tile(int tiles_m, int tiles_n) {
  for (int pid = 0; pid < tiles_m * tiles_n; ++pid) {
    int tm = 0, tn = 0;
    patch_tile(pid, tiles_m, tiles_n, tm, tn);
    if (tm == 0 && column_xcd(tn, tiles_m, tiles_n) != pid % kXcd) return false;
  }
  return true;
}
static_assert(column_xcd_follows_patch_tile(1, 5) && column_xcd_follows_patch_tile(1, 27) &&
              column_xcd_follows_patch_tile(1, 260) && column_xcd_follows_patch_tile(2, 129) &&
              column_xcd_follows_patch_tile(3, 171) && column_xcd_follows_patch_tile(7, 75) &&
              column_xcd_follows_patch_tile(8, 64), "spread starts");

// ---------------------------------------------------------------------------
// Direct global->LDS loads (no register staging, no ds_write):
// each wave-level load instruction drops 64 x 16 bytes = 8 rows x 128 bytes
// into a contiguous 1 KB of LDS.  Rows are unpadded; bank conflicts are
// avoided by an XOR swizzle applied on the *global* side: LDS row r holds
// 16-byte chunk c at position c ^ ((r >> 1) & 7).  Rows are 128 bytes = half
// of the 64 banks, so even/odd rows use different halves and any 16
// consecutive rows read at the same chunk index cover all 64 banks once.  The operands have rings of their own, of
// XS and WS >= XS stages: the loads of X k-tile kt+XS and W k-tile kt+WS are issued while k-tile kt is multiplied.
// ---------------------------------------------------------------------------
template <int VM>
__device__ __forceinline__ void wait_vmcnt() {
  // s_waitcnt with only vmcnt set: vmcnt[3:0] | expcnt=7 | lgkmcnt=15 | vmcnt[5:4] in bits 15:14
  __builtin_amdgcn_s_waitcnt((VM & 0xf) | (0x7 << 4) | (0xf << 8) | ((VM >> 4) << 14));
}

// acc += W-fragment x X-fragment, in place in the accumulator registers.  As the builtin, with 64 accumulators of
// four registers - all 256 accumulator registers - the compiler gave results other registers than inputs and
// moved 100 to 400 registers per k-tile.  What it cannot see here: an accumulator may be moved or read only 8 wait
// states after the instruction, and used as input 2 after it was moved.  PADDED carries these waits along, for code
// around which the compiler does move accumulators (all but the main loop, whose body is free of moves: that is the
// register allocator's choice, and tests/test_gemm_wait_states_cpu.py reads it off the compiled kernels).
template <bool PADDED>
__device__ __forceinline__ void mfma_acc(floatx4& acc, const u32x4& w, const u32x4& x) {
  if constexpr (PADDED)
    asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 7" : "+a"(acc) : "v"(w), "v"(x));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}

// EPI selects the epilogue at compile time, so the plain prefill instantiation carries none of the
// decode-side code: 0 = bias / ReLU / residual -> bf16 segments; 1 = split-K, raw fp32 partials;
// 2 = as 0, but the K and V thirds go into the paged cache.
enum { kEpiPlain = 0, kEpiPartial = 1, kEpiKvScatter = 2 };

// Which k-tiles a workgroup multiplies, in order, and where in K (bytes) they lie.  `first` is the one to start with; the
// walk goes round from there and stays on its last tile, so that the loads in the loop's tail, into stages nobody reads,
// hit the caches.  (Going round once more they brought in weights again: up to 16 % on 28 tiles a split.)
template <bool SPREAD>
struct KWalk {
  int tiles, first, at;
  __device__ __forceinline__ KWalk(int n) : tiles(n), first(0), at(0) {}
  __device__ __forceinline__ int count() const { return tiles; }
  __device__ __forceinline__ void start(int f) { first = f; }
  __device__ __forceinline__ uint32_t offset() const {
    uint32_t t = at < tiles ? at : tiles - 1;
    if (SPREAD) {
      t += first;
      t = min(t, t - tiles);  // unsigned: t - tiles where that is no wrap
    }
    return t * (kBK * 2);
  }
  __device__ __forceinline__ void next() { ++at; }
};

// The same for split-K: K is dealt to S splits round-robin, split s takes one tile of every group of S.  With a multiple
// of four splits it takes number (s + i) % S of group i instead of s, or it would meet only every fourth 128-byte piece
// of a row, a fraction of the memory channels (128 x 8192 x 32768 on 8 splits 140 us, 112 turned).
struct KSplitWalk {
  int splits, split, groups, turn_by, group, turn, left;
  __device__ __forceinline__ KSplitWalk(int tiles, int s, int n) : splits(n), split(s), group(0), turn(s) {
    turn_by = (n & 3) == 0 ? 1 : 0;
    const int whole = tiles / n;
    const int number = turn_by ? (s + whole) % n : s;  // of this split in a last, partial group
    groups = whole + (number < tiles - whole * n ? 1 : 0);
    left = groups - 1;
  }
  __device__ __forceinline__ int count() const { return groups; }
  __device__ __forceinline__ void start(int f) {
    group = f;
    turn = turn_by ? (split + f) % splits : split;
  }
  __device__ __forceinline__ uint32_t offset() const { return (uint32_t)(group * splits + turn) * (kBK * 2); }
  __device__ __forceinline__ void next() {  // (no branches: the loop stays one block)
    const int step = left > 0 ? 1 : 0;
    left -= step;
    group += step;
    turn += step ? turn_by : 0;
    turn = turn == splits ? 0 : turn;
    turn = group == groups ? split : turn;
    group = group == groups ? 0 : group;
  }
};

// NT: the weight loads carry the non-temporal hint, and p.spread is heeded.
template <int BM, int BN, int WAVES_M, int WAVES_N, int XS, int WS, int EPI, bool NT>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_dl_kernel(const GemmParams p) {
  // One wave per SIMD.  (Eight waves - two per SIMD, 128 accumulator registers each - were measured on the
  // 256x256 tile: equal as 4x2 waves of 64x128, 7 % slower as 2x4 of 128x64; the loop is not latency-bound.)
  constexpr int NW = WAVES_M * WAVES_N;
  static_assert(NW == 4, "4 waves");
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int TM = WTM / 16, TN = WTN / 16;   // 16x16 result tiles of a wave
  static_assert(WTM % 16 == 0 && WTN % 32 == 0, "the epilogue stages 32 columns of a wave tile at a time");
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "a wave-level load covers 8 rows");
  constexpr int ROW_BYTES = kBK * 2;                      // 128
  constexpr int W_RING = XS * BM * kBK;                   // the weight ring starts behind the activation ring (elements)
  constexpr int XL = BM / (8 * NW);                       // X loads per wave per stage
  constexpr int WL = BN / (8 * NW);                       // W loads per wave per stage
  constexpr int LPS = XL + WL;
  static_assert(XS >= 2 && WS >= XS && (XS - 1) * LPS + WL < 64, "rings, vmcnt range");

  extern __shared__ __attribute__((aligned(1024))) uint16_t lds[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;

  DS_STAMP(0);
  int tile_m, tile_n;
  patch_tile(blockIdx.x, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM;
  const int n0 = p.n_base + tile_n * BN;
  const int K = p.K;
  auto walk = [&] {
    if constexpr (EPI == kEpiPartial) return KSplitWalk(K / kBK, blockIdx.y, p.splits);
    else return KWalk<NT>(K / kBK);
  };
  auto xk = walk();
  const int KT = xk.count();  // >= 1: splits <= K / 64
  // Spread starts: each XCD (id % 8) begins at an eighth of its own, where the row stride puts the pieces that all rows
  // have at one position of K on few memory channels.  Where the row tiles of a column lie on two XCDs, all of them begin
  // where the first does: equal rows have equal sums, whatever their place in the batch.
  if (NT && p.spread) {
    const unsigned xcd = column_xcd(tile_n, p.tiles_m, p.tiles_n) + p.tiles_m * p.tiles_n * blockIdx.y;
    xk.start((int)((xcd & 7) * (unsigned)KT / 8));
  }
  auto wk = xk;

  // per-lane source offsets (bytes, from the tile's first row) of this wave's loads; load j covers rows
  // 8*(NW*j+wave) .. +7.  With the tile origin and the k position in a scalar base, the lane part is a 32-bit
  // value that never changes, and a load needs no vector arithmetic at all.
  const int lrow = lane >> 3;
  const int lchunk = (lane & 7) ^ (4 * (wave & 1) + (lane >> 4));  // key = (row >> 1) & 7, row = 8*(NW*j+wave) + lane/8
  const char* xbase = reinterpret_cast<const char*>(p.X + (size_t)m0 * p.ldx);
  const char* wbase = reinterpret_cast<const char*>(p.W + (size_t)n0 * K);
  uint32_t xoff[XL], woff[WL];
#pragma unroll
  for (int j = 0; j < XL; ++j) {
    const int row = min(8 * (NW * j + wave) + lrow, p.M - 1 - m0);
    xoff[j] = ((uint32_t)row * (uint32_t)p.ldx + lchunk * 8) * 2u;
  }
#pragma unroll
  for (int j = 0; j < WL; ++j) {
    const int row = min(8 * (NW * j + wave) + lrow, p.N - 1 - n0);
    woff[j] = ((uint32_t)row * (uint32_t)K + lchunk * 8) * 2u;
  }
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);  // keep LDS destinations in scalar registers
  // Load number j of an iteration, in [0, LPS): of an X tile first, into X stage `xst`, then of a W tile, into W stage
  // `wst`; xofs and wofs are the tiles' places in K.
  auto issue_one = [&](int xst, int wst, uint32_t xofs, uint32_t wofs, int j) {
    // (the empty asm keeps the 32-bit lane offset a value of this basic block: hoisted out of the loop as a
    // 64-bit pair it costs a 64-bit vector add per load instead of riding in the instruction's offset operand)
    uint32_t& off = j < XL ? xoff[j < XL ? j : 0] : woff[j < XL ? 0 : j - XL];
    asm volatile("" : "+v"(off));
    // a wave-level load fills 512 elements = 1 KB
    if (j < XL)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(xbase + xofs + off),
          (__attribute__((address_space(3))) void*)(lds + xst * BM * kBK + (j * NW + wave_s) * 512), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(wbase + wofs + off),
          (__attribute__((address_space(3))) void*)(lds + W_RING + wst * BN * kBK + ((j - XL) * NW + wave_s) * 512), 16, 0,
          NT ? 2 : 0);
  };

  floatx4 acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

  // swizzled fragment offsets (elements) inside a row, one per 32-deep k-step: lane (row = lane % 16, quarter =
  // lane / 16) reads chunk 4 * step + quarter
  // Kept in registers across the k loop, one per k-step and operand (the empty asm stops the compiler from
  // recomputing them in the loop): a fragment read is then one add of the stage's base plus an immediate.
  const int frag_row = lane & 15;
  int xfrag[kBK / 32], wfrag[kBK / 32];
#pragma unroll
  for (int ks = 0; ks < kBK / 32; ++ks) {
    const int koff = ((4 * ks + (lane >> 4)) ^ ((lane >> 1) & 7)) * 8;
    xfrag[ks] = (wm * WTM + frag_row) * kBK + koff;
    wfrag[ks] = W_RING + (wn * WTN + frag_row) * kBK + koff;
    asm volatile("" : "+v"(xfrag[ks]), "+v"(wfrag[ks]));
  }

  // A k-tile is multiplied in two halves of one 32-deep k-step each.  The fragments of the next half are fetched
  // while the current half is multiplied, so two fragment sets of TN + TM registers x 4 exist.
  // (held as integer vectors: bf16 vectors carried around the loop get re-packed by the compiler)
  struct Frags {
    u32x4 w[TN];
    u32x4 x[TM];
  };
  Frags fa, fb;
  constexpr int NR = TN + TM;  // fragment reads per half
  // read number r of k-step ks of the stage buffers sb
  struct Bufs {
    const uint16_t *x, *w;
  };
  auto bufs = [&](int xst, int wst) { return Bufs{lds + xst * BM * kBK, lds + wst * BN * kBK}; };
  auto frag_read = [&](Frags& f, const Bufs& sb, int ks, int r) {
    if (r == 0) f.w[0] = *reinterpret_cast<const u32x4*>(sb.w + wfrag[ks]);
    else if (r <= TM) f.x[r - 1] = *reinterpret_cast<const u32x4*>(sb.x + xfrag[ks] + (r - 1) * 16 * kBK);
    else f.w[r - TM] = *reinterpret_cast<const u32x4*>(sb.w + wfrag[ks] + (r - TM) * 16 * kBK);
  };

  // One half.  The 16x16x32 instruction, not 32x32x16: under the chip's power limit it sustains 13 % more with
  // N(0,1)-like operands (registers only: 1.98 against 1.75 PFLOP/s; with zeros 2.43 and 2.47), and the tiles are
  // walked back and forth so that consecutive instructions share an operand.  It also leaves only 16 cycles between
  // two of them, room for about three other instructions, so the next half's fragment reads and (in the second half
  // of a tile) the global->LDS loads of a later tile are dealt out one at a time, never at the same place: in
  // clumps after every four matrix instructions the 256x256 kernel was 2 % slower.  The reads come first needed
  // first and end three quarters into the half, so that the barrier (or the next half) does not wait for the last.
  // A scheduling fence after every group keeps that interleaving.  (256x256 prefers groups of one, the rest of two.)
  // `last` marks the last k-tile.  `mem(j)` is called for j = 0 .. JN-1: it issues the j-th direct-to-LDS load.
  auto half = [&](auto jn, auto last, const Frags& fc, Frags& fn, const Bufs& sb_next, int ks_next, auto&& mem) {
    constexpr int NM = TM * TN, GRP = NM >= 64 ? 1 : 2, NG = NM / GRP, NGR = NG > 4 ? NG * 3 / 4 : NG;
    static_assert(NM % GRP == 0, "whole groups");
    constexpr int JN = decltype(jn)::value;
    auto reads_by = [](int g) { return (g < NGR ? g : NGR) * NR / NGR; };           // fragment reads due before group g
    auto loads_by = [](int g) { return (g + 2 < NG ? (g > 0 ? g + 2 : 0) : NG) * JN / NG; };
#pragma unroll
    for (int g = 0; g < NG; ++g) {
#pragma unroll
      for (int q = g * GRP; q < (g + 1) * GRP; ++q) {
        const int a = q / TM, b = (a & 1) ? TM - 1 - q % TM : q % TM;
        if constexpr (NM >= 64)
          mfma_acc<decltype(last)::value>(acc[a][b], fc.w[a], fc.x[b]);
        else
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fc.w[a]),
                                                              __builtin_bit_cast(bf16x8, fc.x[b]), acc[a][b], 0, 0, 0);
      }
#pragma unroll
      for (int r = reads_by(g); r < reads_by(g + 1); ++r) frag_read(fn, sb_next, ks_next, r);
#pragma unroll
      for (int j = loads_by(g); j < loads_by(g + 1); ++j) mem(j);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NM >= 64 && !decltype(last)::value) asm volatile("s_nop 7");   // moves at the loop's exit (mfma_acc)
  };
  using none = std::integral_constant<int, 0>;
  using all_loads = std::integral_constant<int, LPS>;
  auto no_mem = [](int) {};

  // ---- epilogue set-up (used after the k-loop; the first pass's loads are issued inside it) ----
  // Each wave stages its own WTM x (GA*32) fp32 block (GA column tiles per pass) in LDS that the
  // k-loop no longer needs; rows are padded by 4 floats so the 16-byte transposing writes of 16
  // lanes fall into distinct banks.
  constexpr int LDS_FLOATS = gemm_lds_bytes(BM, BN, XS, WS) / 4;
  constexpr int GA_FIT = (LDS_FLOATS / (NW * WTM) - 4) / 32;
  constexpr int TG = WTN / 32;  // groups of 32 columns of a wave tile
  // (three groups a pass only where they are all: 12 pieces a row, of which no whole number is a wave's)
  constexpr int GA = GA_FIT >= TG ? TG : (GA_FIT == 3 ? 2 : GA_FIT);
  static_assert(GA >= 1, "no room to stage the epilogue");
  constexpr int RSTR = GA * 32 + 4;  // staging row stride in floats
  constexpr int MAX_ITERS = WTM * GA * 4 / 64;
  constexpr int NPASS = (TG + GA - 1) / GA;
  const int row_base = m0 + wm * WTM;
  const int col_base = n0 + wn * WTN;
  // Pass `a0/GA` covers column tiles a0 .. a0+ga-1; after the LDS transposition lane `idx = it*64+lane`
  // owns row idx / cpr, 8-column chunk idx % cpr (cpr = 4*ga chunks per row).
  u32x4 epi_res[2][MAX_ITERS], epi_bias[2][MAX_ITERS];
  auto epi_prefetch = [&](int a0, u32x4* resv, u32x4* biasv) {
    const int ga = (TG - a0) < GA ? (TG - a0) : GA;
    const int cpr = ga * 4;
    const int iters = WTM * cpr / 64;
#pragma unroll
    for (int it = 0; it < MAX_ITERS; ++it) {
      if (it >= iters) break;
      const int idx = it * 64 + lane;
      const int r = idx / cpr, ch = idx - r * cpr;
      const int row = row_base + r, n = col_base + a0 * 32 + ch * 8;
      const bool ok = row < p.M && n < p.N;
      resv[it] = u32x4{0, 0, 0, 0};
      biasv[it] = u32x4{0, 0, 0, 0};
      if (EPI == kEpiPartial) continue;
      if (ok && p.residual) resv[it] = ld16(p.residual + (size_t)row * p.ld_res + n);
      // when cpr divides 64 the chunk (hence the bias piece) is the same for every `it`
      if (ok && p.bias && (it == 0 || 64 % cpr != 0)) biasv[it] = ld16(p.bias + n);
    }
  };

  {
    // Direct-to-LDS schedule (one ring per operand, ONE barrier per k-tile):
    //   iteration kt:  first half of tile kt (fetching the fragments of its second half)
    //                  wait until this wave's part of tile kt+1 has landed (later ones may still fly)
    //                  barrier: tile kt+1 is visible to all, and nobody reads the buffers of tile kt any more
    //                           (the second half's fragments are already in registers)
    //                  second half of tile kt, issuing the loads of X tile kt+XS, then of W tile kt+WS, into the
    //                  buffers of tile kt, and fetching the first-half fragments of tile kt+1
    // Loads land in the order of their issue, so with WS > XS the weights asked for right behind X tile kt+1 may still
    // fly at iteration kt's barrier: they have a k-tile longer than with WS = XS.  256x256 has room for two stages of
    // both (128 KB) or for a third one of weights (160 KB), which the kernels that wait for weights need most.  From two
    // stages each: 4096 x 12288 x 49152 4.05 -> 3.37 ms (rows of X 96 KB apart), 256 x 49152 x 12288 371 -> 350 us,
    // 1536 x 20480 x 5120 254 -> 232, 2985 x 15360 x 5120 371 -> 357, 16384 x 12288 x 12288 3.36 -> 3.32 ms.  (256x160
    // and 128x256 tiles with two and four stages instead of three each: between 4 % faster and 8 % slower.)
    // the loads of iterations -WS to -1, as far as they are of tiles from 0 on
#pragma unroll
    for (int i = -WS; i < 0; ++i) {
#pragma unroll
      for (int j = 0; j < LPS; ++j)
        if (j >= XL || i >= -XS) issue_one(i + XS, i + WS, xk.offset(), wk.offset(), j);
      if (i >= -XS) xk.next();
      wk.next();
    }
    constexpr int IN_FLIGHT = (XS - 2) * LPS + (WS > XS ? WL : 0);  // loads issued after the last of tile kt+1
    wait_vmcnt<IN_FLIGHT + LPS>();
    lds_barrier();
    DS_STAMP(1);
#pragma unroll
    for (int r = 0; r < NR; ++r) frag_read(fa, bufs(0, 0), 0, r);

    int xst = 0, wst = 0;  // buffers of tile kt
    for (int kt = 0; kt < KT - 1; ++kt) {
      const Bufs sb = bufs(xst, wst);
      const int nx = xst + 1 == XS ? 0 : xst + 1, nw = wst + 1 == WS ? 0 : wst + 1;
      const Bufs sbn = bufs(nx, nw);
      __builtin_amdgcn_sched_barrier(0);
      half(none{}, std::false_type{}, fa, fb, sb, 1, no_mem);
      wait_vmcnt<IN_FLIGHT>();
      lds_barrier();
      const uint32_t xofs = xk.offset(), wofs = wk.offset();
      half(all_loads{}, std::false_type{}, fb, fa, sbn, 0, [&](int j) { issue_one(xst, wst, xofs, wofs, j); });
      xk.next();
      wk.next();
      xst = nx;
      wst = nw;
    }
    // Last k-tile (already in LDS and visible since the previous iteration's barrier): no loads, no
    // waits.  The residual and bias pieces of the first epilogue pass are requested before it, so
    // their memory latency passes while the matrix pipe still has work.
    // (only where the register file has room for them next to the accumulators and both fragment sets)
    constexpr bool EARLY_EPI = TM * TN <= 40;
    if (EARLY_EPI) epi_prefetch(0, epi_res[0], epi_bias[0]);
    {
      const Bufs sb = bufs(xst, wst);
      __builtin_amdgcn_sched_barrier(0);
      half(none{}, std::true_type{}, fa, fb, sb, 1, no_mem);
      // (the fragment fetch of this half reads a buffer of clamped re-loads; the values are never used)
      half(none{}, std::true_type{}, fb, fa, sb, 0, no_mem);
    }
    if (!EARLY_EPI) epi_prefetch(0, epi_res[0], epi_bias[0]);
    wait_vmcnt<0>();  // the clamped re-loads of the loop tail must not land in the epilogue's staging area
  }

  // ---- epilogue through LDS: every lane ends up with 8 consecutive columns of one row, so bias,
  // residual and output move as 16-byte pieces that are contiguous along rows. ----
  // Each wave stages its own WTM x (GA*32) fp32 block (GA column tiles per pass) in LDS that the
  // k-loop no longer needs; rows are padded by 4 floats so the 16-byte transposing writes of 16
  // lanes fall into distinct banks.
  __syncthreads();                 // every wave has finished reading the k-loop buffers
  DS_STAMP(2);
  float* stg = reinterpret_cast<float*>(lds) + wave * (WTM * RSTR);
  const OutSegments out = out_segments(p, p.ld_out);
#pragma unroll
  for (int pass = 0; pass < NPASS; ++pass) {
    const int a0 = pass * GA;
    const int ga = (TG - a0) < GA ? (TG - a0) : GA;  // column tiles in this pass (compile-time after unrolling)
    u32x4* resv = epi_res[pass & 1];
    u32x4* biasv = epi_bias[pass & 1];
    // the next pass's residual / bias pieces travel while this pass is transposed and stored
    if (pass + 1 < NPASS) epi_prefetch(a0 + GA, epi_res[(pass + 1) & 1], epi_bias[(pass + 1) & 1]);
    // 1. accumulators -> LDS (transposing): lane holds row 16 b + lane%16, columns 16 a + 4*(lane/16) + 0..3
#pragma unroll
    for (int a = 0; a < 2 * GA; ++a) {
      if (a >= 2 * ga) break;
#pragma unroll
      for (int b = 0; b < TM; ++b)
        *reinterpret_cast<floatx4*>(stg + (b * 16 + (lane & 15)) * RSTR + a * 16 + (lane >> 4) * 4) = acc[2 * a0 + a][b];
    }
    // 2. read back row-contiguous: chunk = 8 columns; cpr chunks per row
    const int cpr = ga * 4;
    const int iters = WTM * cpr / 64;
#pragma unroll
    for (int it = 0; it < MAX_ITERS; ++it) {
      if (it >= iters) break;
      const int idx = it * 64 + lane;
      const int r = idx / cpr, ch = idx - r * cpr;
      const int row = row_base + r, n = col_base + a0 * 32 + ch * 8;
      const floatx4 lo = *reinterpret_cast<const floatx4*>(stg + r * RSTR + ch * 8);
      const floatx4 hi = *reinterpret_cast<const floatx4*>(stg + r * RSTR + ch * 8 + 4);
      if (EPI == kEpiPartial) {  // split-K: raw fp32 sums, row-contiguous
        if (row < p.M && n < p.N) {
          float* dst = p.partial + ((size_t)blockIdx.y * p.M + row) * p.N + n;
          *reinterpret_cast<floatx4*>(dst) = lo;
          *reinterpret_cast<floatx4*>(dst + 4) = hi;
        }
        continue;
      }
      const u32x4 bv = biasv[(64 % cpr != 0) ? it : 0];
      float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      u32x4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float e0 = v[2 * j] + bf16_lo(bv[j]);
        float e1 = v[2 * j + 1] + bf16_hi(bv[j]);
        if (p.relu) {
          e0 = fmaxf(e0, 0.f);
          e1 = fmaxf(e1, 0.f);
        }
        e0 += bf16_lo(resv[it][j]);
        e1 += bf16_hi(resv[it][j]);
        o[j] = pack_bf16(e0, e1);
      }
      if (row < p.M && n < p.N) {
        const int hq = p.n_heads * p.head_dim, hkv = p.n_kv_heads * p.head_dim;
        if (EPI == kEpiKvScatter && n >= hq) {  // this step's new K / V row of sequence `row`: straight into its page
          const int which = n >= hq + hkv;
          const int col = n - hq - which * hkv;
          const int head = col / p.head_dim, d = col - head * p.head_dim;
          const int pos = p.ctx_lens[row];
          const int blk = p.block_tables[(size_t)row * p.max_blocks + pos / 16];
          st16((which ? p.v_cache : p.k_cache) + (((size_t)blk * p.n_kv_heads + head) * 16 + (pos % 16)) * p.head_dim + d, o);
        } else {
          st16(out.at(row, n), o);
        }
      }
    }
  }
  DS_STAMP(3);
}

// The tiles there are, numbered from 1 (the numbers are what g_gemm_variant forces): rows x columns, waves along each,
// stages of X and W, what it may be used for, and what the time model (layer_plan) knows of it.  Larger tiles than
// these do not fit the registers (256 accumulator registers of a wave) or the LDS with two stages.
struct Tile {
  int bm, bn, wm, wn, xs, ws;
  bool tail;           // may take the columns behind a cut
  bool kv;             // also with the K/V scatter of a decoding step
  double k_us, t0_us;  // of a k-tile, of prologue and epilogue
};
constexpr Tile kTiles[] = {
    {0, 0, 0, 0, 0, 0, false, false, 0, 0},
    {256, 160, 4, 1, 3, 3, true, true, 0.929, 2.95},
    {128, 128, 2, 2, 3, 3, true, true, 0.556, 3.48},
    {256, 256, 2, 2, 2, 3, true, false, 1.355, 6.16},
    {64, 128, 1, 4, 3, 3, false, true, 0.47, 0.5},
    {128, 256, 2, 2, 3, 3, true, false, 0.835, 7.0},
    {256, 128, 2, 2, 3, 3, true, true, 0.808, 2.83},
    {256, 192, 2, 2, 2, 3, true, true, 1.062, 2.91},
    {96, 192, 2, 2, 4, 4, false, true, 0.702, 3.69},
    {128, 192, 2, 2, 3, 4, false, true, 0.738, 4.7},
    {160, 192, 2, 2, 3, 3, false, true, 0.807, 3.52},
    {192, 192, 2, 2, 3, 3, false, true, 0.874, 3.22},
    {192, 128, 2, 2, 3, 3, false, false, 0.677, 3.3},
    {192, 256, 2, 2, 2, 3, false, false, 1.073, 5.32},
    {160, 256, 2, 2, 2, 3, false, false, 0.959, 5.53},
    {224, 192, 2, 2, 3, 3, false, true, 0.953, 2.94},
    {288, 192, 2, 2, 2, 3, false, false, 1.191, 1.92},
    {320, 192, 2, 2, 2, 3, false, false, 1.307, 1.94},
    {384, 160, 4, 1, 2, 3, false, false, 1.308, 2.18},
    {384, 128, 2, 2, 2, 4, false, false, 1.115, 2.58},
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
template <int T, int EPI, bool NT>
inline hipError_t launch_kernel(const GemmParams& p, int splits, hipStream_t stream) {
  constexpr Tile t = kTiles[T];
  constexpr size_t lds_bytes = gemm_lds_bytes(t.bm, t.bn, t.xs, t.ws);
  static_assert((size_t)(t.xs * t.bm + t.ws * t.bn) * kBK * sizeof(uint16_t) <= lds_bytes && lds_bytes <= 160 * 1024, "LDS");
  constexpr auto kern = gemm_dl_kernel<t.bm, t.bn, t.wm, t.wn, t.xs, t.ws, EPI, NT>;
  (void)KernelAttrReg<kern, (int)lds_bytes>::done;
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n, splits), dim3(64 * t.wm * t.wn), lds_bytes, stream, p);
  return hipGetLastError();
}

// One launch of tile T.
template <int T, bool NT>
inline hipError_t launch_one(const GemmParams& p, int splits, hipStream_t stream) {
  if (splits > 1) return launch_kernel<T, kEpiPartial, NT>(p, splits, stream);
  if constexpr (kTiles[T].kv)
    if (p.k_cache) return launch_kernel<T, kEpiKvScatter, NT>(p, 1, stream);
  return launch_kernel<T, kEpiPlain, NT>(p, 1, stream);
}
template <int FIRST, int... T>
inline hipError_t launch_any(int tile, const GemmParams& p, bool nt, int splits, hipStream_t stream,
                             std::integer_sequence<int, T...>) {
  hipError_t e = hipErrorInvalidValue;
  (void)((tile == FIRST + T && ((e = nt ? launch_one<FIRST + T, true>(p, splits, stream)
                                          : launch_one<FIRST + T, false>(p, splits, stream)), true)) || ...);
  return e;
}

// The tiles from number kFirstLayerTile on, which only products of a layer take (gemm_tiles.hip).
constexpr int kFirstLayerTile = 8;
hipError_t launch_layer_tile(int tile, const GemmParams& p, bool nt, int splits, hipStream_t stream);

}  // namespace ds
