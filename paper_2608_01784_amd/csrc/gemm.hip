// SwiGLU experts over expert-sorted rows on bf16 MFMA (gfx950).
//
// Expert e (Eq. (2)) is E_e(x) = W_down[e] (SiLU(W_gate[e] x) * (W_up[e] x)), the
// two input projections and one output projection counted in Appendix A.  Two
// grouped GEMMs do the work, both "NT" (both operands K-contiguous):
//   up:   act[j, :] = SiLU(x_j W_gate[e]^T) * (x_j W_up[e]^T),  x_j = h[sorted_token[j]]
//   down: y[j, :]   = act[j, :] W_down[e]^T
// Rows of one expert are contiguous after the permutation; each workgroup counts the
// experts' M tiles itself from expert_offsets, so no launch shape depends on the
// device-resident per-expert counts.  One more expert may follow the routed ones, the
// always-on one: every token is one of its rows, in token order.
//
// In the up GEMM the first half of a tile's weight rows are gate rows and the second
// half the matching up rows, so gate and up of one output column meet in the same
// lane and register and SiLU(g) * u is formed before the single bf16 rounding of
// the activation.  A partial last N tile clamps its weight rows and skips the
// stores past N.
//
// Data movement: operands go from global memory straight into LDS (16 bytes per lane,
// no register staging) through rings of 64-wide K slices.  LDS rows are 128 bytes
// (8 chunks of 16 bytes) with chunk c of row r stored in slot c ^ ((r / 2) % 8).  The
// LDS has 64 four-byte banks and serves a 16-byte read for 16 lanes at a time, i.e. 16
// rows of one fragment: their (row parity, slot) pairs are all distinct, so fragment
// reads are conflict-free, while a wave's copy still writes 1 KB (8 whole rows)
// contiguously.
//
// Scheduling: a persistent grid (as many workgroups as the LDS admits: one per CU of the
// large tiles, two and four of the small ones) walks a flattened
// sequence of (tile, K-slice) steps, so prefetching continues across tile
// boundaries.  Tiles are dealt to the 8 XCDs in contiguous runs (workgroup b
// runs on XCD b % 8), so one expert's tiles share that XCD's L2.  Within an
// expert the N tiles of one M tile are adjacent, so the workgroups of an XCD
// working at the same time share each gathered input slice and each weight slice.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace rfx {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int GM_XCDS = 8;

// s_waitcnt vmcnt(N) with expcnt and lgkmcnt left at their maxima (gfx9 encoding:
// vmcnt in bits [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8]).
template <int N>
__device__ __forceinline__ void waitcnt_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}

// Cache policy of the copies: sc0 (work-group scope).  Each copied line is read once
// per workgroup, so nothing is gained from keeping it in the CU's vector L1; measured
// 1-2 % less grouped-GEMM time on the tall-tile layers than the default policy (the
// non-temporal hint, which lets L2 drop the lines early, was 35-40 % slower: the
// weight lines it evicts are the ones the other M tiles of the expert read next).
constexpr int kDmaPolicy = 1;

// One wave's 1 KB copy: 16 bytes per lane from `src` straight into LDS at `dst`
// (the wave-uniform base; lane L lands at dst + 16 L bytes).  Kept out of line of
// the kernel's lambdas so that the host-side pass of the kernel stays valid.
__device__ __forceinline__ void lds_dma(const uint16_t* src, uint16_t* dst) {
  __builtin_amdgcn_global_load_lds(src, dst, 16, 0, kDmaPolicy);
}

// Workgroup barrier without the release/acquire fences of __syncthreads(): those
// would drain every outstanding vector-memory op (the in-flight LDS-DMA slices
// included) at each step.  The explicit vmcnt wait before it already makes this
// wave's DMA writes complete; lgkmcnt(0) makes this wave's earlier LDS reads
// complete before any wave refills the slice they read; the memory clobber keeps
// the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Epilogue of one 32 x 32 output block of a wave: rows row_base + (0..31), columns
// col_base + (0..31), from the fp32 accumulators (weights as the MFMA's A operand) to
// bf16 rows of `out`; UP: SiLU(g) u from the gate and up accumulators of the same
// columns.  Lane l, register r holds output row l % 32 (a pair row) and column
// 8 (r/4) + 4 (l/32) + r%4.  Stored as it lies, one instruction would write 8 bytes to
// each of 32 rows; instead the block goes through the wave's staging buffer in LDS and
// comes back with 4 lanes per row, so each store instruction writes 16 rows of 64
// contiguous bytes (a quarter of the write requests).  Rows at or past row_end are
// skipped; N is a multiple of 64, so a group of 8 columns is wholly inside a partial
// last N tile or wholly past it.
//
// The staging accesses are inline assembly: the compiler cannot tell that the buffer
// does not alias the ring the direct-to-LDS copies write, and would wait for the next
// slice's copies (issued before the epilogue) before touching it.
constexpr int ST_LD = 40;                 // staging row pitch (elements): 80 B, 16 B aligned
constexpr int ST_ELEMS = 32 * ST_LD;      // one wave's staging buffer
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

template <bool UP>
__device__ __forceinline__ void store_block(const f32x16_t& g, const f32x16_t& u, int row_base,
                                            int col_base, int row_end, int N_out,
                                            uint16_t* __restrict__ out, uint16_t* stage) {
  const int lane = threadIdx.x & 63;
  const uint32_t base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(stage));
  const uint32_t wr = base + ((lane & 31) * ST_LD + 4 * (lane >> 5)) * 2;
  const uint32_t rd = base + ((lane >> 2) * ST_LD + 8 * (lane & 3)) * 2;
  u32x2_t v[4];
#pragma unroll
  for (int gi = 0; gi < 4; ++gi) {
    float a4[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      if (UP) {
        const float gg = g[4 * gi + h], uu = u[4 * gi + h];
        const float en = __builtin_amdgcn_exp2f(gg * -1.4426950408889634f);
        a4[h] = gg * __builtin_amdgcn_rcpf(1.0f + en) * uu;
      } else {
        a4[h] = g[4 * gi + h];
      }
    }
    v[gi] = u32x2_t{pack_bf16x2(a4[0], a4[1]), pack_bf16x2(a4[2], a4[3])};
  }
  u32x4_t r0, r1;
  asm volatile(
      "ds_write_b64 %2, %4\n\t"
      "ds_write_b64 %2, %5 offset:16\n\t"
      "ds_write_b64 %2, %6 offset:32\n\t"
      "ds_write_b64 %2, %7 offset:48\n\t"
      "ds_read_b128 %0, %3\n\t"
      "ds_read_b128 %1, %3 offset:1280\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r0), "=&v"(r1)
      : "v"(wr), "v"(rd), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3])
      : "memory");
  const int rbase = row_base + (lane >> 2);
  const int col = col_base + 8 * (lane & 3);
  if (col < N_out) {
    if (rbase < row_end) *reinterpret_cast<u32x4_t*>(out + static_cast<size_t>(rbase) * N_out + col) = r0;
    if (rbase + 16 < row_end)
      *reinterpret_cast<u32x4_t*>(out + static_cast<size_t>(rbase + 16) * N_out + col) = r1;
  }
}

// ---- the tile kernel: waves that all load and multiply -------------------------------
//
// The main shape is 256 pair rows x 256 weight rows x 64 (K) by 8 waves on
// v_mfma_f32_32x32x16_bf16 with fp32 accumulators.  Experts with hundreds of rows are bound
// by the MFMAs, those with few by the weight stream; one kernel serves both, because copies and
// MFMAs of absent rows are skipped and an expert of up to 256 rows then reads its weights
// once.  (128-row tiles with dedicated copier waves, which launches with fewer than 512 rows
// per expert at pair capacity used before: LLaDA-MoE shape, up + down GEMM at 6 / 80 / 160 /
// 188 / 375 rows per expert 151 / 166 / 231 / 241 / 391 us against 147 / 166 / 183 / 191 / 320
// us here; LLaDA2.0-mini shape at 164 rows 500 against 388 us.)
//
// Two waves share each SIMD.  The waves form 2 (pair rows) x 4 (weight rows): wave
// (wm, wn) multiplies the 32-row pair blocks wm, wm + 2, wm + 4, wm + 6 by 64
// weight rows (UP: the 32 gate rows and the 32 matching up rows of activation columns
// n0 + 32 wn ..; DOWN: weight rows 64 wn ..).  Waves w and w + 4 share a SIMD, so each
// SIMD holds one wave of each wm: an expert's last tile, whose rows end early, shortens
// the MFMA stream of all four SIMDs, and of both their waves, alike (row blocks past the
// expert's end are skipped), instead of idling some while the others run a full tile.  The K
// loop is instantiated per count of active row blocks, so the common full tile runs
// straight-line code with no per-block branches.  Every wave issues its share of the
// global->LDS copies of the next input-row slice and of the weight slice two steps
// ahead into the ring slots the previous step has just released, one copy between
// every two MFMAs of the first two K sub-steps: issued all at once after the barrier,
// the 64 copies of a step queue up in the texture path and stall both waves of each
// SIMD until they drain.
//
// A tile shape: WAVES waves, of which the first WM x WN multiply, MI 32-row pair blocks by 64
// weight rows each (the others only copy); the input-row and weight rings have A_SLOTS and
// B_SLOTS slices and are copied A_SLOTS - 1 and B_SLOTS - 1 K steps ahead.
template <int MI_, int WM_, int WN_, int WAVES_, int A_SLOTS_, int B_SLOTS_>
struct Shape {
  static constexpr int MI = MI_, WM = WM_, WN = WN_, WAVES = WAVES_, A_SLOTS = A_SLOTS_,
                       B_SLOTS = B_SLOTS_;
};
constexpr int TL_BK = 64;
constexpr int TL_NJ = 2;                         // 32-row weight blocks per wave
constexpr int TL_CH = TL_BK / 8;
constexpr int TL_ROWS_PER_OP = 64 / TL_CH;
constexpr int TL_RG = 16 / TL_CH;

template <class S>
struct Geometry {
  static constexpr int THREADS = 64 * S::WAVES;
  static constexpr int BM = 32 * S::MI * S::WM, BROWS = 64 * S::WN;     // pair and weight rows of a tile
  static constexpr int UP_BN = BROWS / 2, DOWN_BN = BROWS;              // output columns of a tile
  static constexpr int A_ELEMS = BM * TL_BK, B_ELEMS = BROWS * TL_BK;   // one slice
  static constexpr int A_OPS = BM / TL_ROWS_PER_OP / S::WAVES;          // copies per wave and step
  static constexpr int B_OPS = BROWS / TL_ROWS_PER_OP / S::WAVES;
  static constexpr int B_WROWS = BROWS / S::WAVES;                      // weight rows a wave copies
  static constexpr int RING = S::A_SLOTS * A_ELEMS + S::B_SLOTS * B_ELEMS;
  static constexpr bool STAGE_IN_A = S::WM * S::WN * ST_ELEMS <= A_ELEMS;     // else in a weight slot
  static constexpr size_t LDS = 2 * size_t(RING);
  static_assert(S::WM * S::WN * ST_ELEMS <= (STAGE_IN_A ? A_ELEMS : B_ELEMS), "staging fits a slot");
  // Copies that may still be in flight when a K step starts: those issued after its own input
  // rows (A_SLOTS - 1 steps ago) and weights (no later than the rows).
  static constexpr int IN_FLIGHT = (S::B_SLOTS > S::A_SLOTS ? B_OPS : 0) + (S::A_SLOTS - 2) * (A_OPS + B_OPS);
  static_assert(S::WM * S::WN <= S::WAVES && S::A_SLOTS >= 2 && S::B_SLOTS >= S::A_SLOTS, "shape");
  static_assert(A_OPS * TL_ROWS_PER_OP * S::WAVES == BM && B_OPS * TL_ROWS_PER_OP * S::WAVES == BROWS,
                "whole copies");
  static_assert(B_WROWS == 16 || B_WROWS == 32, "a wave's weight rows are all gate or all up rows");
  static_assert(4 * (REFLEX_MAX_EXPERTS + 1) <= 2 * RING, "start-up scratch in the rings");
  static_assert(LDS <= 160 * 1024 && IN_FLIGHT < 64, "LDS and vmcnt range");
};

// BIG: input rows are addressed with 64-bit pointers (operands of 2^30 elements or more,
// beyond the reach of a buffer resource's 32-bit byte offset).
//
// The always-on expert: sh_rows rows (0: none), in order the rows 0 .. sh_rows - 1 of h (UP)
// or rows sh_row0 .. of x (DOWN), to rows sh_row0 .. of `out`, with weights sw0 / sw1.
template <bool UP, class S, bool BIG>
__global__ __launch_bounds__(Geometry<S>::THREADS) void swiglu_gemm_kernel(
    const uint16_t* __restrict__ x, const int32_t* __restrict__ gather,
    const int32_t* __restrict__ expert_offsets, int E, const uint16_t* __restrict__ w0,
    const uint16_t* __restrict__ w1, size_t w_expert_stride, const uint16_t* __restrict__ sw0,
    const uint16_t* __restrict__ sw1, int sh_row0, int sh_rows, int K, int N_out, int x_rows,
    int out_rows, uint16_t* __restrict__ out) {
  // The LDS holds the two rings (256-row tiles: all 160 KB, input-row slices in slots 0-1,
  // weight slices in the three slots after them).  The weight lines mostly come from HBM (the
  // input rows mostly hit in L2), so they are copied further ahead and the copies of the next
  // weight slices stay in flight across each step's barrier.  The tile tables live in
  // registers, and the epilogue stages its stores in the input-row slot the tile's last K
  // step has read (in the weight slot it has read where that one is too small).
  using G = Geometry<S>;
  constexpr int TL_BM = G::BM, TL_A_ELEMS = G::A_ELEMS, TL_B_ELEMS = G::B_ELEMS;
  constexpr int TL_A_OPS = G::A_OPS, TL_B_OPS = G::B_OPS, TL_A_SLOTS = S::A_SLOTS, TL_B_SLOTS = S::B_SLOTS;
  constexpr int TL_MI = S::MI;
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  uint16_t* const a_ring = smem;
  uint16_t* const b_ring = smem + TL_A_SLOTS * TL_A_ELEMS;
  constexpr int BN = UP ? G::UP_BN : G::DOWN_BN;
  const int n_tiles = (N_out + BN - 1) / BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // ---- expert row offsets and the per-expert prefix of M tiles, kept in registers: lane l
  // holds the entries of experts l, l + 64, l + 128, l + 192.  The offsets are read once per
  // workgroup into LDS (scratch: the rings are empty until the first copies; every wave
  // reading them from memory would queue up at the same few cache lines), the prefix is four
  // wave scans that every wave does for itself.
  int toff_r[4], eo_r[4], eo_E = 0, m_total = 0, bm_log = __builtin_ctz(TL_BM);
  {
    int* s_eo = reinterpret_cast<int*>(smem);
    for (int e = tid; e <= E; e += G::THREADS) s_eo[e] = E > 0 ? expert_offsets[e] : 0;
    __syncthreads();
    int n[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane + 64 * q;
      eo_r[q] = s_eo[e < E ? e : E];
      n[q] = s_eo[e < E ? e + 1 : E] - eo_r[q];
    }
    eo_E = __builtin_amdgcn_readfirstlane(s_eo[E]);
    // Rows per tile (2^bm_log): 256-row tiles are cut to 128 rows where few, far larger experts
    // would outlast all others by a tile: the largest has over four times the mean of the
    // experts with pairs, and the cut adds at most a quarter to the tiles (Zipf-skewed
    // experts, forward at T = 256 / 512 / 1024: 164 / 159 / 171 us uncut, 155 / 146 / 159 cut;
    // T = 2048, where the cut adds more: 200 us uncut, 215 cut).  Cutting evenly filled experts
    // only reads their weights twice (LLaDA-MoE, 110 rows each: 200 us uncut, 222 cut).  The
    // always-on expert by itself: up to 4096 rows, to have more tiles beside the routing
    // (LLaDA2.0-mini, T = 4096: forward 422 us uncut, 415 cut; T = 8192: 508 and 541), while
    // the cut tiles still run in one round (d = 2176, 8 experts, always-on width 3456: T = 1500 /
    // 2083 / 4000 162 / 194 / 338 us cut, 140 / 174 / 255 uncut); past 4096 rows where the whole
    // tiles take an eighth of the CUs or less, the down GEMM of a narrow layer (d = 128, width 3776,
    // T = 4874: 133 us uncut, 112 cut).
    auto prefix = [&]() {
      m_total = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tiles = n[q] < 0 ? 0 : (n[q] + (1 << bm_log) - 1) >> bm_log;
        const int incl = wave_inclusive_scan_i32(tiles, lane);
        // (scaled to tiles; lanes past E: never at or before a tile)
        toff_r[q] = lane + 64 * q < E ? (m_total + incl - tiles) * n_tiles : INT32_MAX;
        m_total += __builtin_amdgcn_readlane(incl, 63);
      }
    };
    prefix();
    if constexpr (TL_BM == 256) {
      int used = 0;
      uint64_t far = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) used += __popcll(__ballot(n[q] > 0));
      const float mean4 = 4.0f * static_cast<float>(eo_E) / static_cast<float>(max(used, 1));
#pragma unroll
      for (int q = 0; q < 4; ++q) far |= __ballot(static_cast<float>(n[q]) > mean4);
      if (far != 0) {
        int more = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) more += n[q] <= 0 ? 0 : ((n[q] + 127) >> 7) - ((n[q] + 255) >> 8);
        if (__builtin_amdgcn_readfirstlane(wave_sum_i32(more)) <= m_total / 4) {
          bm_log = 7;
          prefix();
        }
      }
      const int whole = ((sh_rows + 255) >> 8) * n_tiles;
      if (E == 0 && (sh_rows <= 4096 ? 2 : 8) * whole <= static_cast<int>(gridDim.x)) bm_log = 7;
    }
    __syncthreads();     // all scratch reads done before the first copies land
  }
  // entry e (< 256) of a per-lane table, uniform e
  auto table_at = [&](const int (&r)[4], int e) {
    const int q = e >> 6;
    const int v = q == 0 ? r[0] : (q == 1 ? r[1] : (q == 2 ? r[2] : r[3]));
    return __builtin_amdgcn_readlane(v, e & 63);
  };
  // Logical tile L -> tile: experts in order, the M tile outer and the N tile inner; the
  // expert is found in one round (four ballots count the experts whose first tile lies at or
  // before L).  rot: the tile's K rotation (below).
  struct TT {
    int expert, row0, row_end, n0, rot;
  };
  const int nk = K / TL_BK;
  const int routed_tiles = m_total * n_tiles;
  // local / n_tiles by a multiplication with the rounded-up reciprocal, at most one too large
  const uint32_t recip = n_tiles > 1 ? 0xffffffffu / static_cast<uint32_t>(n_tiles) + 1u : 0u;
  auto split = [&](int local, int& m, int& n) {
    m = n_tiles > 1 ? static_cast<int>(__umulhi(static_cast<uint32_t>(local), recip)) : local;
    n = local - m * n_tiles;
    if (n < 0) {
      --m;
      n += n_tiles;
    }
  };
  auto decode = [&](bool always_on, int L) {
    TT t;
    int m, n;
    if (always_on) {
      split(L, m, n);
      t.expert = E;
      t.n0 = n * BN;
      t.row0 = sh_row0 + (m << bm_log);
      t.row_end = min(sh_row0 + sh_rows, t.row0 + (1 << bm_log));
      t.rot = n % nk;
      return t;
    }
    int lo = -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) lo += __popcll(__ballot(toff_r[q] <= L));
    lo = lo < 0 ? 0 : lo;
    split(L - table_at(toff_r, lo), m, n);
    const int er0 = table_at(eo_r, lo);
    const int er1 = lo + 1 < E ? table_at(eo_r, lo + 1) : eo_E;
    t.expert = lo;
    t.n0 = n * BN;
    // Tiles of one height, in whole 64-row steps (a block for each wm): an expert just over a
    // multiple of the tile otherwise leaves a tile of few rows, whose K steps take far more
    // than their share (copies, barriers, fewer MFMAs per LDS read).  LLaDA-MoE, forward at
    // 272 / 314 / 375 / 544 rows per expert: 354 / 362 / 377 / 543 us full tiles first, 340 /
    // 323 / 354 / 527 even ones; 448 / 826 rows, which hardly move: 418 / 744, 421 / 742.
    int height = 1 << bm_log;
    if constexpr (TL_BM > 64) {
      const int tiles = (er1 - er0 + height - 1) >> bm_log;
      if (tiles > 1) height = ((er1 - er0 + tiles - 1) / tiles + 63) & ~63;
    }
    t.row0 = er0 + m * height;
    t.row_end = min(min(er1, out_rows), t.row0 + height);
    if (t.row0 < 0 || t.row0 >= t.row_end) t.row_end = t.row0;   // inconsistent offsets: no rows
    // K rotation: tile (M tile m of expert e, N tile n) walks its K slices starting at
    // slice n mod nk (down) or (n mod 2 + 5 e) mod nk (up).  The tiles sharing an input-row
    // slice (same e and m) then request it a step apart instead of all at once (5 % less
    // GEMM time on the 16-layer stack, 3 % on the skewed layer, against no rotation), while
    // the M tiles sharing a weight slice (same e and n) read it in the same step, so it
    // comes from HBM once for all of them (1 % less time than a rotation of 2 m + n, which
    // spread them two steps apart).  In the up GEMM the 8 N tiles sharing a gathered-row
    // slice stay within two steps, so fewer of its lines leave L2 before the last of them
    // reads it (1 % less up-GEMM time than n mod nk; the same in the down GEMM made it 2-4 %
    // slower).  The expert term spreads the tiles that stream weights at the same time over
    // the offsets within their 4 KB weight rows (d = 2048): without it the 256 concurrent
    // tiles of a weight-bound up GEMM read only two distinct slices (LLaDA-MoE shape, 6 / 80 /
    // 160 rows per expert: 112 / 139 / 146 us without, 94 / 106 / 112 us with it; 4 e instead
    // of 5 e, which leaves out three offsets in four: 104 / 118 / 127 us; even from 300 rows
    // up and in the down GEMM).  Only the order of the fp32 sums over K changes.
    t.rot = (UP ? n % 2 + 5 * lo : n) % nk;
    return t;
  };
  // This workgroup's tiles: a contiguous run of the routed tiles per XCD, strided over the
  // XCD's workgroups; ahead of the run the XCD's share of the always-on expert's tiles (full
  // ones, so they go first), dealt one by one.
  const int xcd = blockIdx.x % GM_XCDS;
  const int per_xcd = gridDim.x / GM_XCDS;
  const int j0 = blockIdx.x / GM_XCDS;
  const int sh_tiles = ((sh_rows + (1 << bm_log) - 1) >> bm_log) * n_tiles;
  const int sh_mine = (max(sh_tiles - xcd, 0) + GM_XCDS - 1) / GM_XCDS;
  const int chunk = (routed_tiles + GM_XCDS - 1) / GM_XCDS;
  const int r_begin = xcd * chunk, r_mine = max(min(routed_tiles - r_begin, chunk), 0);
  if (j0 >= sh_mine + r_mine) return;
  const int n_my = (sh_mine + r_mine - j0 + per_xcd - 1) / per_xcd;
  // multiplying waves: (wm, wn); wm >= WM: a wave that only copies
  const int wm = wave / S::WN, wn = wave % S::WN;

  // ---- copies: op q of the step fills rows ROWS_PER_OP q ..; lane L writes row
  // r = ROWS_PER_OP q + L / CH at slot L % CH, holding chunk (L % CH) ^ ((r / RG) % CH)
  auto lane_row = [&](int q) { return q * TL_ROWS_PER_OP + lane / TL_CH; };
  auto lane_chunk = [&](int q) { return ((lane % TL_CH) ^ ((lane_row(q) / TL_RG) % TL_CH)) * 8; };
  // The copies are buffer loads into LDS.  Input rows go through a resource of the
  // operand's size, and a copy that is skipped (wholly past the expert's last row) gets
  // an offset past that size, which the hardware's range check turns into no memory
  // access, so the step has no branch: a branch splits the step into several basic
  // blocks, and the instruction order pinned below then holds only within each (16-layer
  // stack and skewed layer: 2-3 % less GEMM time than a branch around each copy,
  // identical output; traced in one process).  (BIG: nothing is skipped, absent rows read
  // the tile's first row again.)  Weight rows go through a resource of the
  // wave's 32 rows of the tile: with global_load_lds copies the compiler made each
  // sub-step's MFMAs wait for all of the step's LDS reads, not only their own (2-3 %
  // less GEMM time with the buffer form).  Copy sources are 32-bit element offsets (BIG:
  // 64-bit).
  //
  // Each loader (input rows, weights) has a current tile and K slice, and holds the next
  // tile's setup ready: a tile's K loop takes every loader across exactly one tile boundary,
  // so both setups are made from one decode before the K loop and the K step only moves them
  // over (decoding a tile inside the step, for each loader by itself, made the step 290
  // instead of 175 instructions long and the kernel half as large again).
  //
  // Input rows: rotation, the copies that hold rows of the tile, and copy j's offset into x;
  // of the next tile the row numbers n_row (UP: of the expert-sorted list, replaced by the
  // token's row of h in the K loop's first step, so that the loader does not wait for the
  // gather: a wait for the newest load is a wait for every copy in flight).
  using Off = typename std::conditional<BIG, size_t, uint32_t>::type;
  int a_tile = -1, a_k = nk, a_rot = 0, a_ops = 0, n_rot = 0, n_ops = 0;
  bool n_ready = false, n_gather = false;
  Off a_off[TL_A_OPS];
  int n_row[TL_A_OPS];
  auto set_a = [&](const TT& t) {
    const int rows_valid = t.row_end - t.row0;
    // Input-row copy q holds rows ROWS_PER_OP q ..; copies wholly past the expert's last
    // row are not issued.  The multiply reads whole 32-row blocks up to the one holding the
    // last row, so it may read up to three groups of 8 rows that were not copied: whatever
    // the slot held before.  Each of them enters only its own row of the product, and rows
    // past row_end are not stored (16-layer stack and skewed layer: 1-2 % less GEMM time,
    // identical output; traced in one process).
    int n = (rows_valid + TL_ROWS_PER_OP - 1) / TL_ROWS_PER_OP - TL_A_OPS * wave;
    n = n < 0 ? 0 : (n > TL_A_OPS ? TL_A_OPS : n);
    n_ops = __builtin_amdgcn_readfirstlane(n);
    n_rot = t.rot;
    n_gather = UP && t.expert != E;
#pragma unroll
    for (int j = 0; j < TL_A_OPS; ++j) {
      const int r = lane_row(TL_A_OPS * wave + j);
      int src = t.row0 + (r < rows_valid ? r : 0);     // rows past the expert reuse row0
      if (rows_valid <= 0) src = 0;
      if (UP && !n_gather) src -= sh_row0;
      n_row[j] = src;
    }
  };
  auto gather_a = [&]() {
    if (UP && n_ready && n_gather) {
#pragma unroll
      for (int j = 0; j < TL_A_OPS; ++j) n_row[j] = gather[n_row[j]];
    }
  };
  // Weights: rotation and the address of the wave's B_WROWS weight rows: tile rows B_WROWS
  // wave .. (UP: of the gate rows in the first half of the waves, of the up rows in the
  // second).  N is a multiple of 64 and the rows start at a multiple of B_WROWS, so in a
  // partial last N tile they are all valid or all past N; past N they are replaced by the
  // last rows (the columns past N are not stored).  Copies j and j + 2 are 16 rows apart and
  // share the chunk swizzle: copy j reads 16 K (j / 2) + b_off[j % 2].
  int b_tile = -1, b_k = nk, b_rot = 0, nb_rot = 0;
  bool nb_ready = false;
  uint32_t b_lo = 0, b_hi = 0, nb_lo = 0, nb_hi = 0;
  uint32_t b_off[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    b_off[j] = static_cast<uint32_t>(lane_row(j) * K) +
               static_cast<uint32_t>(lane_chunk(TL_B_OPS * wave + j));
  auto set_b = [&](const TT& t) {
    nb_rot = t.rot;
    constexpr int W = G::B_WROWS, HALF = S::WAVES / 2;
    const bool second = UP && wave >= HALF;
    int wr0 = t.n0 + W * (second ? wave - HALF : wave);
    wr0 = wr0 + W <= N_out ? wr0 : N_out - W;
    const uint16_t* wm_base = t.expert == E ? (second ? sw1 : sw0)
                                            : (second ? w1 : w0) + t.expert * w_expert_stride;
    const uint64_t b_addr = reinterpret_cast<uint64_t>(wm_base + static_cast<size_t>(wr0) * K);
    nb_lo = static_cast<uint32_t>(b_addr);
    nb_hi = static_cast<uint32_t>(b_addr >> 32);
  };
  // the loaders' next setups, each by its own tile (a lookahead of a tile or more)
  const bool short_k = nk < TL_B_SLOTS;
  auto tile_at = [&](int i) {
    const int j = j0 + i * per_xcd;
    return j < sh_mine ? decode(true, xcd + GM_XCDS * j) : decode(false, r_begin + j - sh_mine);
  };
  auto ready_a = [&]() {
    n_ready = a_tile + 1 < n_my;
    if (!n_ready) return;
    set_a(tile_at(a_tile + 1));
    gather_a();
  };
  auto ready_b = [&]() {
    nb_ready = b_tile + 1 < n_my;
    if (nb_ready) set_b(tile_at(b_tile + 1));
  };
  // The K offset of a loader's next slice; then it advances (past the workgroup's last
  // tile it stays on its last slice, so the issue never branches and every source
  // address stays in bounds).
  auto a_next = [&]() {
    if (a_k == nk) {
      if (n_ready) {
        n_ready = false;
        ++a_tile;
        a_k = 0;
        a_rot = n_rot;
        a_ops = n_ops;
#pragma unroll
        for (int j = 0; j < TL_A_OPS; ++j) {
          int src = n_row[j];
          if (UP) src = src < 0 ? 0 : (src >= x_rows ? x_rows - 1 : src);
          a_off[j] = static_cast<Off>(src) * static_cast<Off>(K) +
                     static_cast<Off>(lane_chunk(TL_A_OPS * wave + j));
        }
      } else {
        a_k = nk - 1;
      }
    }
    int kr = a_k + a_rot;
    kr = kr >= nk ? kr - nk : kr;
    ++a_k;
    return kr * TL_BK;
  };
  auto b_next = [&]() {
    if (b_k == nk) {
      if (nb_ready) {
        nb_ready = false;
        ++b_tile;
        b_k = 0;
        b_rot = nb_rot;
        b_lo = nb_lo;
        b_hi = nb_hi;
      } else {
        b_k = nk - 1;
      }
    }
    int kr = b_k + b_rot;
    kr = kr >= nk ? kr - nk : kr;
    ++b_k;
    return kr * TL_BK;
  };
  const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(x), static_cast<short>(0),
      BIG ? 0 : static_cast<int>(static_cast<uint32_t>(x_rows) * static_cast<uint32_t>(K) * 2u),
      0x00020000);
  auto dma_a = [&](int j, uint16_t* As_, int k0_) {
    if constexpr (BIG) {
      lds_dma(x + a_off[j] + k0_, As_ + (TL_A_OPS * wave + j) * 512);
      return;
    }
    const uint32_t voff = j < a_ops ? (a_off[j] + static_cast<uint32_t>(k0_)) * 2u : 0x80000000u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        x_rsrc, (__attribute__((address_space(3))) void*)(As_ + (TL_A_OPS * wave + j) * 512), 16,
        voff, 0, 0, kDmaPolicy);
  };
  auto dma_b = [&](int j, uint16_t* Bs_, int k0_) {
    // the resource is rebuilt from wave-uniform halves at each use, so that it always
    // lives in scalar registers (held across the loop it could end up in vector
    // registers, and each copy would then become a loop over the distinct values)
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b_lo)));
    const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b_hi)));
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(lo | (hi << 32)), static_cast<short>(0), 2 * G::B_WROWS * K, 0x00020000);
    const uint32_t voff = (b_off[j % 2] + static_cast<uint32_t>(k0_ + 16 * (j / 2) * K)) * 2u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        b_rsrc, (__attribute__((address_space(3))) void*)(Bs_ + (TL_B_OPS * wave + j) * 512), 16,
        voff, 0, 0, kDmaPolicy);
  };
  // ---- multiply: pair blocks WM i + wm of the tile, weight blocks b_row[j]
  const int b_row[TL_NJ] = {UP ? 32 * wn : 64 * wn, UP ? G::BROWS / 2 + 32 * wn : 64 * wn + 32};
  const int frow = lane & 31, fsel = lane >> 5, fx = (frow / TL_RG) % TL_CH;
  f32x16_t acc[TL_MI][TL_NJ];
  // prologue: the copies the steps before the first would have issued, except that the first
  // weight slices go out ahead of the input rows, whose gather entries are still on their way
  ready_a();
  for (int q = 0; q < TL_B_SLOTS - 1; ++q) {
    if (b_k == nk) ready_b();
    const int kb = b_next();
#pragma unroll
    for (int j = 0; j < TL_B_OPS; ++j) dma_b(j, b_ring + q * TL_B_ELEMS, kb);
  }
  for (int q = 0; q < TL_A_SLOTS - 1; ++q) {
    if (q > 0 && a_k == nk) ready_a();
    const int ka = a_next();
#pragma unroll
    for (int j = 0; j < TL_A_OPS; ++j) dma_a(j, a_ring + q * TL_A_ELEMS, ka);
  }
  waitcnt_vm<0>();       // (not in the order the steps count on)
  int s = 0;     // K steps so far (the rings' slot counter)
  // The K loop of one tile with NB active pair blocks (0: this wave only copies).  The
  // MFMAs of each slice's last 16-wide sub-step run after the next step's barrier, from
  // fragments read before it, so they overlap the LDS reads of the next slice's first
  // sub-step instead of every SIMD waiting for those reads after each barrier (16-layer
  // stack and skewed layer: 3-4 % less GEMM time, identical output; traced in one
  // process).  The fragments stay in the second register buffer across the barrier.
  TT t = tile_at(0), next_t = t;
  auto k_loop = [&](auto nb_c) {
    constexpr int NB = decltype(nb_c)::value;
    constexpr int kReads = NB + TL_NJ, kMfmas = NB * TL_NJ;
    bf16x8_t af[2][TL_MI], bfr[2][TL_NJ];
    // weights as the MFMA's A operand: the accumulator is the transposed tile, so each
    // lane ends up holding 4 consecutive output columns of one row
    auto mfmas = [&](int buf) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < TL_NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[buf][j], af[buf][i], acc[i][j],
                                                              0, 0, 0);
    };
    // a copy after every kPer MFMAs: the copies drain at the rate the texture path takes
    // them while the matrix cores keep busy
    auto interleave_copies = [&](auto ops_c) {
      constexpr int kOps = decltype(ops_c)::value, kPer = kMfmas / kOps > 0 ? kMfmas / kOps : 1;
#pragma unroll
      for (int q = 0; q < kOps; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, kPer, 0);
        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
    };
    // One K step.  FIRST: the tile's first, with no deferred MFMAs of a previous slice.
    auto step = [&](auto first_c) {
      constexpr bool FIRST = decltype(first_c)::value;
      const int ka = a_next();
      const int kb = b_next();
      // Input-row slice s and weight slice s have landed (the copies issued after them may
      // be in flight; copies land in order among themselves, so other outstanding ops, the
      // previous tile's stores or the gather loads, only lengthen the wait) and are visible
      // to all waves; the slots of the slices the previous step read are free.
      waitcnt_vm<G::IN_FLIGHT>();
      lds_barrier();
      if constexpr (FIRST)
        if (!short_k) gather_a();
      // Raised issue priority from the barrier through the deferred MFMAs and the first
      // copies: the SIMD's two waves leave the barrier together, and the one served first
      // gets its MFMAs going while the other's LDS reads are in flight (16-layer stack:
      // 1.1 / 1.5 % less up / down GEMM time, skewed layer 0.2 / 0.5 %; traced in one
      // process.  Raised around every MFMA group instead: 1.3 % slower).
      __builtin_amdgcn_s_setprio(1);
      uint16_t* An = a_ring + ((s + TL_A_SLOTS - 1) % TL_A_SLOTS) * TL_A_ELEMS;
      uint16_t* Bn = b_ring + ((s + TL_B_SLOTS - 1) % TL_B_SLOTS) * TL_B_ELEMS;
      if constexpr (NB == 0) {
#pragma unroll
        for (int j = 0; j < TL_A_OPS; ++j) dma_a(j, An, ka);
#pragma unroll
        for (int j = 0; j < TL_B_OPS; ++j) dma_b(j, Bn, kb);
        __builtin_amdgcn_s_setprio(0);
      } else {
        const uint16_t* As = a_ring + (s % TL_A_SLOTS) * TL_A_ELEMS;
        const uint16_t* Bs = b_ring + (s % TL_B_SLOTS) * TL_B_ELEMS;
        auto load = [&](int kk, int buf) {
          const int slot = ((2 * kk + fsel) ^ fx) * 8;
#pragma unroll
          for (int i = 0; i < NB; ++i)
            af[buf][i] =
                *reinterpret_cast<const bf16x8_t*>(As + (32 * (S::WM * i + wm) + frow) * TL_BK + slot);
#pragma unroll
          for (int j = 0; j < TL_NJ; ++j)
            bfr[buf][j] = *reinterpret_cast<const bf16x8_t*>(Bs + (b_row[j] + frow) * TL_BK + slot);
        };
        // (the instruction scheduler is told the order: reads of kk+1, then MFMAs of kk)
        load(0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
        if constexpr (!FIRST) {
          mfmas(1);     // the previous slice's last sub-step
#pragma unroll
          for (int j = 0; j < TL_A_OPS; ++j) dma_a(j, An, ka);
          interleave_copies(std::integral_constant<int, TL_A_OPS>{});
        }
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int kk = 0; kk < TL_BK / 16 - 1; ++kk) {
          load(kk + 1, (kk + 1) & 1);
          __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
          mfmas(kk & 1);
          if (FIRST ? kk == 0 : false) {
#pragma unroll
            for (int j = 0; j < TL_A_OPS; ++j) dma_a(j, An, ka);
          }
          if (FIRST ? kk == 1 : kk == 0) {
#pragma unroll
            for (int j = 0; j < TL_B_OPS; ++j) dma_b(j, Bn, kb);
          }
          if (FIRST && kk == 0)
            interleave_copies(std::integral_constant<int, TL_A_OPS>{});
          else if (FIRST ? kk == 1 : kk == 0)
            interleave_copies(std::integral_constant<int, TL_B_OPS>{});
          else
            __builtin_amdgcn_sched_group_barrier(0x008, kMfmas, 0);
        }
      }
    };
    step(std::true_type{});
    ++s;
    for (int kt = 1; kt < nk; ++kt, ++s) step(std::false_type{});
    if constexpr (NB > 0) mfmas(1);     // the last slice's last sub-step
  };
  for (int tile_i = 0; tile_i < n_my; ++tile_i) {
    // the loaders' next setups; unless short_k both loaders are in this tile and leave it in
    // a step after the first
    if (short_k) {
      ready_a();
      ready_b();
    } else {
      n_ready = nb_ready = tile_i + 1 < n_my;
      if (n_ready) {
        next_t = tile_at(tile_i + 1);
        set_a(next_t);
        set_b(next_t);
      }
    }
    // pair blocks of this wave that hold pairs (wave-uniform): blocks wm, wm + WM, .. of the tile
    const int blocks = (t.row_end - t.row0 + 31) >> 5;
    const int nb = __builtin_amdgcn_readfirstlane(
        wm < S::WM ? min(max(blocks - wm + S::WM - 1, 0) / S::WM, TL_MI) : 0);
#pragma unroll
    for (int i = 0; i < TL_MI; ++i)
#pragma unroll
      for (int j = 0; j < TL_NJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // one instance of the K loop per count of active blocks
    if constexpr (TL_MI == 4) {
      switch (nb) {
        case 4: k_loop(std::integral_constant<int, 4>{}); break;
        case 3: k_loop(std::integral_constant<int, 3>{}); break;
        case 2: k_loop(std::integral_constant<int, 2>{}); break;
        case 1: k_loop(std::integral_constant<int, 1>{}); break;
        default: k_loop(std::integral_constant<int, 0>{}); break;
      }
    } else if constexpr (TL_MI == 2) {
      switch (nb) {
        case 2: k_loop(std::integral_constant<int, 2>{}); break;
        case 1: k_loop(std::integral_constant<int, 1>{}); break;
        default: k_loop(std::integral_constant<int, 0>{}); break;
      }
    } else {
      static_assert(TL_MI == 1, "instances");
      if (nb == 1)
        k_loop(std::integral_constant<int, 1>{});
      else
        k_loop(std::integral_constant<int, 0>{});
    }
    // every wave has read the tile's last slices: the input-row slot takes the staging, or the
    // weight slot where that one is too small
    // (the next tile's first step refills it only after its own barrier)
    lds_barrier();
    uint16_t* stage = (G::STAGE_IN_A ? a_ring + ((s + TL_A_SLOTS - 1) % TL_A_SLOTS) * TL_A_ELEMS
                                     : b_ring + ((s + TL_B_SLOTS - 1) % TL_B_SLOTS) * TL_B_ELEMS) +
                      wave * ST_ELEMS;
#pragma unroll
    for (int i = 0; i < TL_MI; ++i) {
      if (i < nb) {
        const int rb = t.row0 + 32 * (S::WM * i + wm);
        if (UP) {
          store_block<true>(acc[i][0], acc[i][1], rb, t.n0 + 32 * wn, t.row_end, N_out, out, stage);
        } else {
#pragma unroll
          for (int j = 0; j < TL_NJ; ++j)
            store_block<false>(acc[i][j], acc[i][j], rb, t.n0 + 64 * wn + 32 * j, t.row_end, N_out,
                               out, stage);
        }
      }
    }
    t = short_k && tile_i + 1 < n_my ? tile_at(tile_i + 1) : next_t;
  }
  waitcnt_vm<0>();     // the last (unused) copies land before the workgroup's LDS is released
}
// The tile shapes (pair rows x weight rows); the rule between them is at launch_gemm.
using Tall = Shape<4, 2, 4, 8, 2, 3>;       // 256 x 256, 160 KB of LDS, one workgroup per CU
using Half = Shape<2, 2, 4, 8, 3, 3>;       // 128 x 256, 144 KB, one per CU
using Medium = Shape<1, 2, 2, 4, 3, 3>;     // 64 x 128, 72 KB, two per CU
using Narrow = Shape<1, 1, 1, 4, 3, 3>;     // 32 x 64, 36 KB, four per CU

// Persistent workgroups: as many as the LDS admits per CU, rounded up to a multiple of the
// XCD count.
template <class S>
int persistent_grid() {
  const int cus = device_cus() * static_cast<int>(160 * 1024 / Geometry<S>::LDS);
  return (cus + GM_XCDS - 1) / GM_XCDS * GM_XCDS;
}

template <bool UP, class S, bool BIG>
int launch_gemm_as(const uint16_t* x, const int32_t* gather, const int32_t* eo, int E,
                   const uint16_t* w0, const uint16_t* w1, size_t stride, const AlwaysOn& sh, int K,
                   int N, int x_rows, int out_rows, uint16_t* out, hipStream_t s) {
  auto* kernel = &swiglu_gemm_kernel<UP, S, BIG>;
  constexpr size_t lds = Geometry<S>::LDS;
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(lds)) != hipSuccess)
      return REFLEX_ERR_LAUNCH;
    attr_set = true;
  }
  hipLaunchKernelGGL(kernel, dim3(persistent_grid<S>()), dim3(Geometry<S>::THREADS), lds, s, x,
                     gather, eo, E, w0, w1, stride, sh.w0, sh.w1, sh.row0, sh.rows, K, N, x_rows,
                     out_rows, out);
  return launch_status();
}

// Tiles of one launch at capacity: cap rows spread evenly over the experts they can reach.
template <bool UP, class S>
long capacity_tiles(int cap, int E, int sh_rows, int N) {
  using G = Geometry<S>;
  constexpr int BN = UP ? G::UP_BN : G::DOWN_BN;
  const long experts = std::min(E, cap), rows = experts > 0 ? (cap + experts - 1) / experts : 0;
  const long m = experts * ((rows + G::BM - 1) / G::BM) + (sh_rows + G::BM - 1) / G::BM;
  return m * ((N + BN - 1) / BN);
}

// The tile shape of a launch.  An expert has at most as many rows as there are tokens (T), so
// up to 32 (64) tokens a 32-row (64-row) tile reads its weights once, as the 256-row tile
// does, and its finer tiles spread over the CUs more evenly: forward of the LLaDA-MoE shape
// at T = 1 / 5 / 32 60 / 139 / 162 us with 256-row tiles, 47 / 112 / 158 us with 32-row ones,
// LLaDA2.0-mini shape at T = 8 / 32 148 / 279 against 119 / 252 us; at T = 64 64-row tiles 97
// against 98 us (skewed).
//
// With more tokens the pair capacity decides, the most rows the experts may hold on average
// (LLaDA-MoE and LLaDA2.0-mini use 0.4 to 0.6 of it).  Up to 192, weights bound the launch: 128-row
// tiles leave LDS for a third input-row slice, and so a whole K step more for the copies to
// land; forward with 256- / 128-row tiles: LLaDA-MoE T = 256 / 1024 (48 / 192) 171 / 187
// against 168 / 184 us, T = 2048 (384, whose experts need two 128-row tiles) 224 against 243;
// LLaDA2.0-mini T = 777 / 4096 (36 / 192) 342 / 415 against 336 / 417, T = 5000 (234) 444 against
// 458; skewed T = 1500 / 4096 (70 / 192) 176 / 281 against 155 / 265.  Up to 32, 64-row tiles:
// few experts hold more, and half as many weight rows per tile spread a skewed load better
// (T = 128 / 512, 128- against 64-row tiles: skewed 134 / 131 against 118 / 122 us;
// LLaDA-MoE T = 170 165.5 against 164.4, LLaDA2.0-mini T = 300 331 against 329; past the line
// skewed T = 1024 145 against 156).  Where the smaller tiles just pass a whole number of rounds
// of the grid they lose, which the host cannot know: skewed, 12 pairs per token, T = 90 / 100 /
// 110 / 120 95 / 112 / 112 / 117 us with 64-row tiles, 97 / 103 / 108 / 131 with 128-row ones
// (100 / 106 / 111 / 139 with the former 128-row kernel).  Other launches of smaller tiles read an expert's weights
// more than once (LLaDA-MoE, T = 1024: 191 / 228 / 288 us with 256 / 64 / 32 rows) and pay only
// where 256-row tiles would leave half of the CUs without work (8 experts of width 512, d =
// 256: forward at T = 128 / 512 / 2048 34.8 / 40.3 / 49.7 us with 256-row tiles, 28.6 / 29.9 /
// 40.5 with 64-row ones; T = 4096, 256 tiles: up GEMM 16.9 against 20.1 us).  Weights of more than
// 8 MB do not stay in an XCD's L2 for the next tile to read: there only while the 64-row tiles
// run in one round at capacity, else 128-row ones (8 experts of width 1792, d = 3840, top-8, T =
// 193: forward 179 us with 64-row tiles, 119 with 128-row ones; experts that fill less of the
// capacity lose by it, d = 2048, width 1024, K_max 4, T = 1000: 57 and 66).  The same line
// one shape down: 64-row tiles for a quarter of the CUs or fewer (T = 128: 28.6 against 27.9
// us with 32-row tiles; down GEMM at T = 512: 10.3 against 9.2 us; up GEMM there, 256 tiles:
// 9.4 against 11.1 us).
//
// Input operands of fewer than 2^30 elements are read through a buffer resource, whose byte
// offsets are 32 bits wide with the upper half kept for skipped copies; larger ones
// through 64-bit pointers.
template <bool UP>
int launch_gemm(const uint16_t* x, const int32_t* gather, const int32_t* eo, int T, int E, int cap,
                const uint16_t* w0, const uint16_t* w1, size_t stride, const AlwaysOn& sh, int K,
                int N, int x_rows, uint16_t* out, hipStream_t s) {
  const int cus = device_cus();
  auto* launch = &launch_gemm_as<UP, Tall, false>;
  if (static_cast<size_t>(x_rows) * static_cast<size_t>(K) >= (size_t(1) << 30)) {
    launch = &launch_gemm_as<UP, Tall, true>;
  } else {
    // the always-on expert in launches of its own runs beside the routing: 256-row tiles (cut
    // to 128 rows by the kernel) leave the routing launches more CUs than smaller ones
    const bool alone = E == 0 && T > Geometry<Medium>::BM;
    const bool few = 2 * capacity_tiles<UP, Tall>(cap, E, sh.rows, N) <= cus;
    if (!alone) {
      const auto holds = [&](int rows) { return cap <= static_cast<long>(rows) * E; };
      const long medium = capacity_tiles<UP, Medium>(cap, E, sh.rows, N);
      const bool stay = static_cast<size_t>(E) * N * K <= (size_t(1) << 22);
      if (T <= Geometry<Narrow>::BM || (few && 4 * medium <= cus))
        launch = &launch_gemm_as<UP, Narrow, false>;
      else if (T <= Geometry<Medium>::BM || (few && (stay || medium <= 2 * cus)) || holds(32))
        launch = &launch_gemm_as<UP, Medium, false>;
      else if (few || holds(192))
        launch = &launch_gemm_as<UP, Half, false>;
    }
  }
  return launch(x, gather, eo, E, w0, w1, stride, sh, K, N, x_rows, cap, out, s);
}

}  // namespace

size_t swiglu_ws_bytes(int rows, int f) {
  return align_up(std::max<size_t>(static_cast<size_t>(rows) * f * sizeof(uint16_t), 1));
}

int launch_swiglu_up(const uint16_t* h, const int32_t* sorted_token, const int32_t* expert_offsets,
                     const uint16_t* wg, const uint16_t* wu, int T, int E, int d, int f, int cap,
                     const AlwaysOn& sh, uint16_t* act, hipStream_t s) {
  if (cap <= 0 && sh.rows <= 0) return REFLEX_OK;
  return launch_gemm<true>(h, sorted_token, expert_offsets, T, E, cap, wg, wu,
                           static_cast<size_t>(f) * d, sh, d, f, T, act, s);
}

int launch_swiglu_down(const int32_t* expert_offsets, const uint16_t* wd, int T, int E, int d,
                       int f, int cap, const AlwaysOn& sh, const uint16_t* act, uint16_t* y_sorted,
                       hipStream_t s) {
  if (cap <= 0 && sh.rows <= 0) return REFLEX_OK;
  return launch_gemm<false>(act, nullptr, expert_offsets, T, E, cap, wd, nullptr,
                            static_cast<size_t>(d) * f, sh, f, d, cap + sh.rows, y_sorted, s);
}

int launch_swiglu_dense(const uint16_t* x, const uint16_t* wg, const uint16_t* wu,
                        const uint16_t* wd, int M, int d, int f, uint16_t* y, uint16_t* act,
                        hipStream_t s) {
  if (M <= 0) return REFLEX_OK;
  int rc = launch_swiglu_up(x, nullptr, nullptr, nullptr, nullptr, M, 0, d, f, 0,
                            AlwaysOn{wg, wu, 0, M}, act, s);
  if (rc == REFLEX_OK)
    rc = launch_swiglu_down(nullptr, nullptr, M, 0, d, f, 0, AlwaysOn{wd, nullptr, 0, M}, act, y, s);
  return rc;
}

}  // namespace rfx
