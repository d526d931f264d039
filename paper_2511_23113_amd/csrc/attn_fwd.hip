// Persistent block-sparse flash-attention forward for gfx950 (MI355X), bf16 MFMA, f32 accumulate.
//
// One workgroup per partition walks its own list of work items (head, query block, range of
// the row's active KV blocks).  For every active KV block J of an item it computes, per head,
//   S = scale * Q_I K_J^T,  running row max m and row sum l,  P = exp(S - m),  O += P V_J,
// and ends with O / l and LSE = m + ln l: the block-sparse evaluation of
// O = softmax(Q K^T / sqrt(d)) V (arXiv 2511.23113, Background: "Visual Generative Models",
// "Block-wise Sparse Attention"), where only the dense blocks of the mask are visited, so an
// item costs its number of dense blocks.
//
// Work split inside a workgroup (wave = 64 lanes, lane = 32*g + r):
//   * waves form a (query group) x (key group) grid.  Wave (a, c) owns 64 queries (two tiles of 32)
//     and, of every KV block, the 32-key slices of key group c; it keeps its own running softmax
//     statistics over its keys (so its probabilities are rounded to bf16 against its own running max:
//     O is 2.3e-3 from 64 bits in the 2-norm, most of it the rounding of O itself, and no further
//     with two or four key groups than with one), and the key groups are combined once per item.  Two query tiles per
//     wave mean that every K and V^T operand read from the LDS feeds two MFMAs.
//       64-token blocks              1 query group,  2 key groups of 1 slice:  2 waves
//       128-token blocks, d = 64     2 query groups, 4 key groups of 1 slice:  8 waves
//       128-token blocks, d = 128    2 query groups, 2 key groups of 2 slices: 4 waves
//     d = 64 runs two waves per SIMD in 256 registers, d = 128 one wave per SIMD in 512, with Q
//     (and K or V operands) in accumulation registers, from which an MFMA reads directly.
//   * Products are formed transposed, S^T = K Q^T and O^T = V^T P^T, with
//     v_mfma_f32_32x32x16_bf16: lane r holds query r, so m and l are per-lane scalars.
//   * S^T's accumulator registers 8h..8h+7 of a 32-key tile hold, in lane group g, the keys
//     16h + {4g..4g+3, 8+4g..8+4g+3}; packed to bf16 they are the B operand of the PV product
//     for that 16-key step.  The matching V^T operand comes from two transposing LDS reads
//     (ds_read_b64_tr_b16) of row-major V: in a group of 16 lanes, lane 4j+a supplies the
//     address of 4 consecutive d-values of key j, and lane i receives d-value i of 4 keys.
// Pair mode (64-token mask blocks, the block size of the paper's PAROAttention masks, at d = 128):
//   the workgroup of 128-token blocks serves two neighbouring query blocks at once, and its KV tile is
//   a pair of 64-token blocks from the union of the two rows' lists; each wave's (query block, KV
//   block) combination carries a flag, and where it is clear the wave's probabilities are exact zeros.
// Software pipeline:
//   the unit of work is 32 keys x 32 queries; a wave's units alternate between its two query tiles.
//   A step issues, as independent work,
//     the MFMAs of  K Q^T of one unit  and of  V^T P^T of the unit two steps back,  and
//     the VALU work of the softmax of the unit in between,
//   as a sequence of sub-slots fenced from each other: ONE MFMA each, then the softmax of one (d = 128)
//   or two scores per lane and at most three LDS reads.  One MFMA per sub-slot matters: an MFMA keeps
//   the matrix pipe busy for 32 clocks and blocks the wave's next MFMA, but not its vector work, for
//   that long.  Measured on the sequence of a step of 16 MFMAs and 56 vector instructions, one wave:
//   530 clocks with single MFMAs, 672 with pairs of them, 840 with no interleaving.
//   LDS operands are read a whole step ahead of their MFMAs.  At d = 128 a wave has its SIMD to itself, and
//   what it issues per 32 clocks beside the MFMA bounds the sequence: six instructions are free, a copy counts as
//   three to four, a wait for anything is the matrix pipe's wait.  So
//     * the other work of a slice's two steps is dealt to their sub-slots by table (Cfg): operand reads, copies, their
//       addresses one sub-slot ahead of them, the barrier;
//     * the first half of a slice's operands has a second set of registers (24 more at d = 128), so that its
//       reads need not wait for the last use of the operands before them;
//     * K Q^T comes before V^T P^T in every pair of sub-slots: a step's softmax then begins two MFMAs behind the
//       last of the scores' products (with V^T P^T first the compiler has to put 32 clocks of nothing in between);
//     * the vote on the running max ends a sub-slot before its branch, which otherwise costs 24 clocks a step.
//   A block of 128 x 128 at d = 128, item ends included: 3065 clocks with the operand reads, the copies and the
//   barrier in one step of the two, 2700 so (2048 of them MFMA; in isolation the loop takes 2430, its MFMAs and softmax
//   alone 2072).  40 heads of 256 x 256 blocks: 5838 -> 5538 us; 24 of 928 x 928: 35.1 -> 32.8 ms.
//   The softmax is speculative: probabilities are formed against the running max as it stands; only
//   when a unit's per-lane sum of probabilities exceeds SPEC_SUM_LIMIT (some score is far above the
//   running max) is the unit redone with a raised max and the accumulator rescaled.  That path is kept
//   out of line: a taken branch over it in every step costs a wave that has its SIMD to itself 2 %.
// At full occupancy of the chip the kernel runs power-limited (the shader clock drops to 1.7 - 1.8 GHz
// with all 256 compute units busy), so instructions and bytes saved count as much as cycles saved.
// Data movement:
//   * K and V slices go L2 -> LDS directly (global_load_lds_dwordx4, 16 bytes per lane, no VGPR
//     staging).  64-token blocks: a wave copies its own slices into its own ring of two and waits for
//     its own copies only; no barrier couples the two waves until the end of an item.  128-token
//     blocks: the two waves of a key group share its ring of four slices and copy half of each; a
//     barrier in the first step of a slice publishes the next one and retires the last, whose
//     positions are refilled behind it and have the two slices after this one to land (a barrier every second
//     slice with a wait for all copies gave them two to three steps instead of four); where K and V come from behind the
//     L2s, K has until the next barrier and V until the one after it, see dbsp_launch_fwd.  An item's first slice has its
//     barrier in its second step, and three slices of copies in front of it, where no softmax runs yet.  The loop goes
//     once round the ring, so that no address depends on the position.
//   * A copy instruction occupies its wave for about 18 clocks, so copies are spread over sub-slots.
//   * LDS tiles are unpadded; 16-byte chunks are XOR-swizzled inside each row instead (the
//     permutation is applied to the per-lane global source address, the LDS side of the copy
//     is linear): K by the row index so that the 16-byte operand reads of 16 lanes (16
//     consecutive keys) hit distinct banks; V by (row & 3) so that the 4 keys of a
//     transposing read hit distinct bank quarters.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cfloat>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "attn_common.hpp"
#include "fwd_params.hpp"

namespace {

// D: head dim.  NQ: groups of 64 queries per workgroup.  NC: groups of keys, U: 32-key slices per group
// and block.  NB: slices of K, and of V, a group's LDS ring holds.
template <int D, int NQ_, int NC_, int U_>
struct Cfg {
  static constexpr int NQ = NQ_, NC = NC_, U = U_, NB = NQ == 1 ? 2 : 4;
  static constexpr int QROWS = 64 * NQ;     // queries of an item
  static constexpr int KROWS = 32 * NC * U; // keys of a KV block
  static constexpr int NW = NQ * NC;        // waves: (query group, key group)
  static constexpr int NT = 64 * NW;
  static constexpr int DT = D / 32;         // 32-wide tiles of the head dim
  static constexpr int KS = D / 16;         // k-steps of K Q^T = MFMAs of one K Q^T unit = of one V^T P^T unit
  static constexpr int NCH = D / 8;         // 16-byte chunks per row
  static constexpr int RPL = 128 / D;       // rows per 256 bytes (one sweep over the 64 LDS banks)
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int SL = 32 * ROW_BYTES; // bytes of a slice
  static constexpr int LOADS = SL / 1024 / NQ;   // 1-KiB direct-to-LDS copies per slice and wave: the waves that use a slice share its copy
  static constexpr int RPC = 64 / NCH;      // rows per copy
  static constexpr int KVAR = (NCH * RPL) / RPC;   // copies per period (16 rows) of K's swizzle
  static constexpr int RING = 2 * NB * SL;  // a key group's ring: NB slices of K, then NB of V
  // End-of-item exchange: of the 2 DT accumulator tiles (32 d x 32 queries) a wave finalises TPW and hands
  // the others to the waves of the other key groups.  Its outbox lies at the end of its group's ring, clear
  // of the first two K slices, which already belong to the next item by then.
  static constexpr int TPW = 2 * DT / NC, XCH = (NC - 1) * TPW * 4096;
  static_assert(TPW <= kMaxTilesPerWave, "what plans go by that are read where they are staged");
  // Where the query groups share slices an item's Q comes by way of the LDS, tiles of 32 queries laid out like slices of K:
  // each wave copies QCP KiB of it.  It lies in the third and fourth K slice of the ring of key group wa, which neither the
  // next item's first slices nor the outboxes use, or behind the rings.
  static constexpr int QCP = 2 * SL / 1024 / NC;
  static constexpr bool Q_IN_RING = NQ * XCH + 4 * SL <= RING && NQ <= NC && NB == 4;
  static constexpr int LDS_BYTES = NC * RING + (NQ > 1 && !Q_IN_RING ? NQ * 2 * SL : 0);
  static_assert(NQ * XCH <= RING - 2 * SL, "the outboxes must leave the first two K slices alone");
  static_assert(U == 1 || (U == 2 && NQ > 1), "what the step sequence assumes");
  static_assert(NC == 2 || (NC == 4 && TPW == 1), "tile ownership at the end of an item");
  // The sub-slots of a step (SUB, one MFMA each) and of a slice (two steps) at which its other work is done.
  // d = 128: eight dealings of reads and copies took 2420 to 2580 clocks a block in isolation.  This one, 2430, ten
  // off the best, is the one that was timed in the kernel with K Q^T first in every pair.  The barrier stands where the
  // operand reads of the step before have all returned.  d = 64: the first dealing tried.  64-token blocks' copies in
  // the second half of a step: four other places took up to 2 % longer.
  static constexpr int SUB = 2 * KS;
  static_assert(NQ == 1 || (4 * LOADS == SUB && LOADS <= 4), "the first step of an item copies four slices");
  static constexpr int H = NQ > 1 && D == 128 ? KS / 2 : 0;        // operands with two sets of registers
  static_assert(H == 0 || U == 2, "an item's last slice is an odd one where its operands' set of registers goes by parity");
  static constexpr int BARRIER_AT = 3 * KS / 4;
  static constexpr int UNDER_WAY = 4 * LOADS;       // copies that may be under way at a barrier: those of the last two slices
  static constexpr int SOFTMAX_END = D == 128 ? 14 : SUB - 1;
  // exponential of score j
  static __device__ constexpr int exp_at(int j) { return D == 64 ? j / 2 : j == 0 ? 0 : j < 5 ? (j + 1) / 2 : j - 2; }
  // operand read k of the first H operands (K, V^T, V^T of each)
  static __device__ constexpr int read_at(int k) {
    constexpr int at[12] = {7, 8, 9, 11, 12, 14, 15, 16, 19, 20, 22, 23};
    return at[k];
  }
  static __device__ constexpr int copy_at(int k) {
    constexpr int at[8] = {10, 13, 17, 18, 21, 24, 26, 28}, at64[4] = {4, 6, 9, 11};
    if (NQ == 1) return SUB / 2 + k / (4 * LOADS / SUB);
    return D == 128 ? at[k % 8] : at64[k % 4];
  }
  // tile k of key group cc: d-tile and query tile
  static __device__ constexpr int tile_dt(int cc, int k) { return NC == 2 ? cc * (DT / 2) + k % (DT / 2) : cc % DT; }
  static __device__ constexpr int tile_qt(int cc, int k) { return NC == 2 ? k / (DT / 2) : cc / DT; }
  // does key group cc store the LSE of the query tiles it finalises, and with which of its tiles?
  static __device__ constexpr bool has_lse(int cc) { return NC == 2 ? cc == 0 : cc % DT == 0; }
  static __device__ constexpr bool lse_tile(int k) { return k % (TPW > 1 ? TPW / 2 : 1) == 0; }
};

// f(0), ..., f(N - 1), as constants
template <class F, int... I>
__device__ __forceinline__ void for_each_of(F& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void for_each(F&& f) { for_each_of(f, std::make_integer_sequence<int, N>{}); }

// a < b ? x : y, all of them the wave's own (the compiler makes a branch of it)
__device__ __forceinline__ const unsigned char* if_less(int a, int b, const unsigned char* x, const unsigned char* y) {
  const unsigned char* z;
  asm("s_cmp_lt_i32 %1, %2\n\ts_cselect_b64 %0, %3, %4" : "=s"(z) : "s"(a), "s"(b), "s"(x), "s"(y) : "scc");
  return z;
}

template <int N>
__device__ __forceinline__ void wait_copies() {      // all but the N youngest copies of this wave have landed
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The same, and all LDS reads have returned.  At d = 128 by the builtin, whose meaning the compiler knows: behind an asm
// block it waits for these reads again, operand by operand, nine instructions of a slice's two hundred.  us by asm / by the
// builtin: pair rows, 40 heads, 512 x 512 blocks 5338 / 5285, 24 heads, 301 x 301 blocks of 64 992 / 987, 40 heads,
// 256 x 256 of 128 5579 / 5556, 12 heads, 21 x 23 49.8 / 49.3.  At d = 64 another wave takes the slots, and the asm is the
// better one: 48 heads, 275 x 275 blocks of 64 1025 / 1027, 30 heads, 137 x 137 of 128 1477 / 1481.
template <int D, int N>
__device__ __forceinline__ void wait_reads() {
  if constexpr (D == 64) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
  } else {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | 7 << 4 | 0 << 8 | (N >> 4) << 14);      // vmcnt, expcnt (not waited for), lgkmcnt
    asm volatile("" ::: "memory");
  }
}

// Partial results of split rows cross from one compute die's L2 to another's inside a launch: they are
// written and read with the chip as their scope (past the L2s), two floats per lane at a time and the
// lanes of a wave side by side: single rows' 8-byte pieces, which the L2 cannot gather on that way, took
// ten times as long.
__device__ __forceinline__ void store_shared(float* to, float a, float b) {
  const uint64_t v = ((uint64_t)__builtin_bit_cast(uint32_t, b) << 32) | __builtin_bit_cast(uint32_t, a);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(to), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Four floats a lane, what a launch behind this one reads: half the instructions.  us a pass, 8 / 16 bytes a lane, in
// turn: d = 64, 6 heads, 84 x 84 blocks of 128 118.6 / 117.4; 64-token blocks at d = 128, 8 heads, 40 x 40 49.1 / 48.4;
// d = 128, 2 heads, 97 x 97 blocks of 128 104.7 / 104.1; 12 heads, 21 x 23 no difference.  Past the L2s here too: left in
// them, the launch boundary has to write them back, and where the last case took 56.9 us by these it took 58.3 by plain
// stores, 60.4 by streaming ones.
// gfx950 needs two wait states between a store of more than 8 bytes and the next vector write to its data's registers, and
// the compiler, which keeps them for its own stores, does not look into an asm block.
__device__ __forceinline__ void store_shared(float* to, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(to), "v"(v) : "memory");
}
__device__ __forceinline__ f32x2 load_shared(const float* from) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(from), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return f32x2{__builtin_bit_cast(float, (uint32_t)v), __builtin_bit_cast(float, (uint32_t)(v >> 32))};
}

// Stores one accumulator tile: lane (r, g) holds, of query r, d-values 8 e4 + 4 g .. + 3 in res[e4].  The
// lane pair swaps halves so that each lane stores 16 bytes side by side.
template <int D>
__device__ __forceinline__ void store_tile(uint16_t* o, const f32x4 (&res)[4], int64_t tok, int dt, int g) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t a0 = pack_bf16x2(res[2 * i].x, res[2 * i].y), a1 = pack_bf16x2(res[2 * i].z, res[2 * i].w);
    uint32_t b0 = pack_bf16x2(res[2 * i + 1].x, res[2 * i + 1].y), b1 = pack_bf16x2(res[2 * i + 1].z, res[2 * i + 1].w);
    swap_upper_lower(a0, b0);
    swap_upper_lower(a1, b1);
    *reinterpret_cast<u32x4*>(o + tok * D + 32 * dt + 16 * i + 8 * g) = u32x4{a0, a1, b0, b1};
  }
}

// Where lane l of wave w keeps two floats (and two more 128 on) of tile k of a chunk; where a launch of its own merges
// them, there lie four floats a lane side by side instead.
template <class C>
__device__ __forceinline__ float* partial_of(float* part_o, int64_t slot_no, int w, int k, int e4, int l) {
  return part_o + (slot_no * C::NW + w) * (C::TPW * 1024) + (k * 4 + e4) * 256 + l * 2;
}

template <class C>
__device__ __forceinline__ float* partial4_of(float* part_o, int64_t slot_no, int w, int k, int e4, int l) {
  return part_o + (slot_no * C::NW + w) * (C::TPW * 1024) + (k * 4 + e4) * 256 + l * 4;
}

// Is a sum of weights +0?  By its bits: this file is compiled without regard to NaNs, where a comparison of floats
// may come out either way for one.
__device__ __forceinline__ bool is_zero(float x) { return __builtin_bit_cast(uint32_t, x) == 0u; }

// Merges tile k of wave w's share of a split row's chunks, G of them fetched at once, and stores it: token
// tok, d-tile dt.  qloc: this lane's query inside the row.
template <class C, int D, int G, bool PAIR, bool LATER>
__device__ __forceinline__ void merge_tile(const dbsp_fwd_params& p, int64_t first, int n_chunks, int w, int k, int l, int qloc,
                                           int64_t tok, int dt, bool with_lse, bool q_there) {
  float m = -INFINITY, tot = 0.f;
  f32x4 acc[4];
#pragma unroll
  for (int e4 = 0; e4 < 4; ++e4) acc[e4] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int x0 = 0; x0 < n_chunks; x0 += G) {
    float ls[G];
    f32x2 lo[G][4], hi[G][4];
#pragma unroll
    for (int y = 0; y < G; ++y) {
      const int64_t sl = first + min(x0 + y, n_chunks - 1);
      ls[y] = __hip_atomic_load(p.part_lse + sl * C::QROWS + qloc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        if constexpr (LATER) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(partial4_of<C>(p.part_o, sl, w, k, e4, l));
          lo[y][e4] = f32x2{v.x, v.y};
          hi[y][e4] = f32x2{v.z, v.w};
        } else {
          lo[y][e4] = load_shared(partial_of<C>(p.part_o, sl, w, k, e4, l));
          hi[y][e4] = load_shared(partial_of<C>(p.part_o, sl, w, k, e4, l) + 128);
        }
      }
    }
    float mn = m;
#pragma unroll
    for (int y = 0; y < G; ++y) mn = fmaxf(mn, ls[y]);
    const float mref = (mn == -INFINITY) ? 0.f : mn;       // nothing for this query yet: weights of 0, not inf - inf
    const float old = __expf(m - mref);
    m = mn;
    tot *= old;
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) acc[e4] *= old;
#pragma unroll
    for (int y = 0; y < G; ++y) {
      const float wgt = (x0 + y < n_chunks) ? __expf(ls[y] - mref) : 0.f;
      tot += wgt;
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        acc[e4].x += wgt * lo[y][e4].x;  acc[e4].y += wgt * lo[y][e4].y;
        acc[e4].z += wgt * hi[y][e4].x;  acc[e4].w += wgt * hi[y][e4].y;
      }
    }
  }
  // no chunk has anything for this query: LSE = -inf, and O = 0 for a query block of pair rows that has no active
  // block; scores that are all -inf give 0 / 0 as in a row that is not split.  (A sum of NaN is not
  // nothing: some score is undefined, and O and LSE say so.)
  const bool none = is_zero(tot);
  const float inv = (PAIR && none) ? 0.f : 1.0f / tot;
#pragma unroll
  for (int e4 = 0; e4 < 4; ++e4) acc[e4] *= inv;
  if (!q_there) return;
  store_tile<D>(p.o, acc, tok, dt, l >> 5);
  if (with_lse && l < 32 && p.lse != nullptr) p.lse[tok] = none ? -INFINITY : m + __logf(tot);
}

// Merges all split rows behind the kernel that made their chunks: one wave for every tile (x: split row and
// batch entry, y: tile of the wave's share).  Bound by reading the partial results once: 9925 chunks of 64 KiB
// are 650 MB.  Four chunks in flight a wave, 20 thousand waves.
template <int D, int NQ, int NC, int U, bool PAIR>
__global__ __launch_bounds__(64 * NQ * NC) void dbsp_merge_kernel(const dbsp_fwd_params p) {
  using C = Cfg<D, NQ, NC, U>;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = threadIdx.x & 63, r = l & 31;
  const int wa = w / C::NC, wc = w % C::NC, k = blockIdx.y;
  const int bb = blockIdx.x / p.n_split;
  const int32_t* row = p.split_rows + 4 * (blockIdx.x % p.n_split);       // row, first slot, chunks
  const int64_t bh = (int64_t)bb * p.H + row[0] / p.nQ;
  const int first_q = (row[0] % p.nQ) * C::QROWS + 64 * wa, qt = C::tile_qt(wc, k);
  merge_tile<C, D, 4, PAIR, true>(p, (int64_t)bb * p.n_slots + row[1], row[2], w, k, l, 64 * wa + 32 * qt + r, bh * p.Nq + first_q + 32 * qt + r,
                      C::tile_dt(wc, k), C::has_lse(wc) && C::lse_tile(k), !PAIR || first_q < p.Nq);
}

// SCATTERED: from an item's third slice on, a barrier leaves only the last slice's V under way, see dbsp_launch_fwd.
template <int D, int NQ, int NC, int U, bool PAIR, bool SCATTERED>
__global__ __launch_bounds__(64 * NQ * NC) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1, D == 64 ? 2 : 1)))
void dbsp_fwd_kernel(const dbsp_fwd_params p, const int32_t* __restrict__ g_kv_idx, const int4* __restrict__ g_sched,
                       const int32_t* __restrict__ g_part_ptr) {
  using C = Cfg<D, NQ, NC, U>;
  constexpr int NB = C::NB, H = C::H;
  constexpr bool SHARED = NQ > 1;      // the waves of the query groups share the slices' copies
  static_assert(!SCATTERED || (SHARED && D == 128), "a barrier's wait, at d = 128");
  static_assert(!PAIR || (D == 128 && NQ == 2 && NC == 2 && U == 2), "pair rows: two query blocks, two KV blocks of 64 tokens, d = 128");
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  __shared__ float xstat[C::NW][4 * 64];
  __shared__ uint32_t tail_pos;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(LDS_PTR(unsigned char))lds;

  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l = t & 63, r = l & 31, g = l >> 5;
  const int wa = w / C::NC, wc = w % C::NC;     // query group, key group
  const int part = blockIdx.x;
  const float c = p.scale_log2;

  // per-lane source offsets of the copies: the LDS image is linear, the chunk swizzle inside a row is
  // applied to the global side
  uint32_t k_src[C::KVAR], v_src;
  {
    const int row_in = l / C::NCH, pch = l % C::NCH;
#pragma unroll
    for (int v = 0; v < C::KVAR; ++v) {
      const int row = v * C::RPC + row_in;
      k_src[v] = row_in * C::ROW_BYTES + ((pch ^ ((row / C::RPL) % C::NCH)) * 16);
    }
    v_src = row_in * C::ROW_BYTES + ((pch ^ (((row_in / C::RPL) % (C::NCH / 4)) << 2)) * 16);
  }
  const uint32_t ring = lds_base + wc * C::RING;          // this wave's slices in the LDS
  const uint32_t share = wa * C::LOADS * 1024;            // the part of a slice this wave copies
  // K operand reads: key row r, logical chunk 2*ks + g, physical chunk (2*ks + g) ^ sw
  uint32_t k_rd[C::KS];
  {
    const int sw = (r / C::RPL) % C::NCH;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) k_rd[ks] = ring + r * C::ROW_BYTES + (((2 * ks + g) ^ sw) << 4);
  }
  // V^T operand reads (transposing): lane 4j+a of a 16-lane group addresses key j, d-quad a
  uint32_t v_rd[C::DT];
  {
    const int hh = (l >> 4) & 1, j = (l & 15) >> 2, a4 = l & 3;
    const int key = 4 * g + j;
    const int sw = ((key / C::RPL) % (C::NCH / 4)) << 2;
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
      v_rd[dt] = ring + NB * C::SL + key * C::ROW_BYTES + ((((4 * dt) ^ sw) + 2 * hh + (a4 >> 1)) << 4) + (a4 & 1) * 8;
  }
  // where this wave's copies come from inside a KV block (pair rows: inside its key group's own block)
  const uint32_t src_off = (PAIR ? 0 : wc * U * C::SL) + share;
  constexpr uint32_t BLOCK_BYTES = PAIR ? U * C::SL : NC * U * C::SL;

  // Rows with no active block: O = 0, LSE = -inf, dealt to the workgroups in turn.
  for (int64_t x = part; x < (int64_t)p.B * p.n_empty; x += gridDim.x) {
    const int row = p.empty_rows[x % p.n_empty];
    const int64_t head = (x / p.n_empty) * p.H + row / p.nQ;
    const int first = (row % p.nQ) * C::QROWS, rows = PAIR ? min(C::QROWS, p.Nq - first) : C::QROWS;
    u32x4* to = reinterpret_cast<u32x4*>(p.o + (head * p.Nq + first) * D);
    for (int y = t; y < rows * (D / 8); y += C::NT) to[y] = u32x4{0u, 0u, 0u, 0u};
    if (p.lse != nullptr)
      for (int y = t; y < rows; y += C::NT) p.lse[head * p.Nq + first + y] = -INFINITY;
  }

  uint64_t busy = 0;
  // Work of this workgroup: its own list (once per batch entry), then items from the queue all
  // workgroups share, taken one by one with an atomic counter -- the greedy rule "each unit to the
  // least-loaded partition" (Methodology, "Head-level Partitioning") applied at run time, where
  // "least loaded" is "first to run out of work".  Where nothing is placed (fewer items than
  // partitions) every workgroup starts at the queue: the first takes are then known beforehand,
  // one each in workgroup order, and need no counter.  A take costs about 11 ns of everybody's time
  // (one address for the whole chip): with 1024 workgroups, a first take and a failing one each,
  // that used to be half of a short launch.
  const int it_begin = g_part_ptr[part], n_own = g_part_ptr[part + 1] - it_begin;
  const uint32_t total_tail = (uint32_t)p.B * (uint32_t)p.n_tail;
  const uint32_t n_first = p.n_placed == 0 ? gridDim.x : 0u;       // takes without the counter

  // An item overlaps with the end of the one before it in the workgroup's own list: its description, the
  // ids of its first KV blocks, its Q and its first two K slices are fetched while that one drains its
  // pipeline and stores its result.  What an item costs besides its blocks, at d = 128 and 128-token blocks: 9 thousand
  // clocks, of which 800 at its start, 1800 for the first slice's steps, 850 to drain, 200 to meet, 1300 for the exchange's
  // writes and their barrier, 3400 to combine and store, 600 to read the next Q.
  const unsigned char* from = nullptr;      // of the copies, see copy_begin
  int4 da = {}, db = {};         // what the item is, see upload() in api.hip
  int pos = 0, bb = 0;           // its place in the schedule, its batch entry
  int ids = 0;                   // ids of its first 64 KV blocks, one per lane
  uint64_t act = ~0ull;
  bf16x8 q[2][C::KS];
  auto load_q = [&](int64_t bh, int I) {
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      // pair rows: the last pair of a head may lack its second query block; its waves load some valid
      // row instead, work on nothing (all their flags are clear) and store nothing
      const int tq = I * C::QROWS + 64 * wa + 32 * qt + r;
      const uint16_t* qrow = p.q + (bh * p.Nq + (PAIR ? min(tq, p.Nq - 1) : tq)) * D;
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks) q[qt][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(qrow + 16 * ks + 8 * g));
    }
  };
  // The same by way of the LDS: whole rows a KiB at a time, each of them once, where the loads above take 32 bytes of
  // 32 rows at a time and both (d = 64: all four) waves of a query group take them all: 64 such loads kept the compute unit's
  // one path to the cache busy for 2 - 3 thousand clocks, at the end of every item.  us with those loads / this way, in turn:
  // 12 heads, 21 x 23 blocks 53.1 / 50.5, 16 heads, 513 x 513, 22 a row 1349 / 1330, 10 heads, 128 x 256 458 / 454, pair rows, 40
  // heads, 512 x 512 5402 / 5372, d = 64, 30 heads, 137 x 137, B = 2 1513 / 1498, 40 heads, 256 x 256 5700 / 5686, dense 97 x 97 the same.
  // 64-token blocks, whose one query group loads each row twice, have no room for it: two (d = 64: four) workgroups' rings
  // and statistics leave 14 (6) KiB of a compute unit's LDS to each, Q is 16 (8).
  const uint32_t q_at = SHARED ? lds_base + (C::Q_IN_RING ? wa * C::RING + 2 * C::SL : NC * C::RING + wa * 2 * C::SL) : 0u;
  auto q_rows = [&](int64_t bh, int I, int group) {      // pair rows: some valid ones in the place of a block that is not there
    int first = I * C::QROWS + 64 * group;
    if (PAIR && first >= p.Nq) first = I * C::QROWS;
    return reinterpret_cast<const unsigned char*>(p.q + (bh * p.Nq + first) * D);
  };
  // this wave's share of Q as if it were K: key group wc takes query group wc's rows
  auto q_of = [&](int64_t bh, int I) { return q_rows(bh, I, wc) + share; };
  auto copy_q = [&](int64_t bh, int I) {
    const unsigned char* rows = q_rows(bh, I, wa) + wc * C::QCP * 1024;
#pragma unroll
    for (int x = 0; x < C::QCP; ++x) {
      if (x % 4 == 0) {
        from = rows + x * 1024;
        set_copy_dst(q_at + wc * C::QCP * 1024 + x * 1024);
      }
      copy16_nth(x % 4, from, k_src[x % C::KVAR]);
    }
  };
  const bool q_by_lds = SHARED && (reinterpret_cast<uintptr_t>(p.q) & 15) == 0;     // (plain loads take any address)
  auto read_q = [&]() {
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks)
        q[qt][ks] = as_bf16x8(*(LDS_PTR(u32x4))(uintptr_t)(k_rd[ks] - ring + q_at + qt * C::SL));
  };
  auto pin_q = [&]() {
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks) {
        // d = 128 (one wave per SIMD, 512 registers): Q lives in accumulation registers, from which MFMAs read operands directly
        if constexpr (D == 64) asm volatile("" : "+v"(q[qt][ks]));
        else asm volatile("" : "+a"(q[qt][ks]));
      }
  };
  // Block ids, 64 at a time, one per lane (a scalar load per block would make every LDS wait a full
  // wait, since the two share a counter).  Past the end the last id repeats.  Pair rows: id of this
  // wave's KV block of the super block, and a mask of the super blocks in which the wave's
  // (query block, KV block) combination is active.
  struct id_words { int w0, w1; };
  auto load_ids = [&](const int4& d, int from) -> id_words {
    const int x = min(from + l, d.w - 1);
    const int32_t* kv = g_kv_idx + d.z;
    if constexpr (PAIR) return {kv[2 * x], kv[2 * x + 1]};
    else return {kv[x], 0};
  };
  auto set_ids = [&](const id_words& v, int& id, uint64_t& am) {
    if constexpr (PAIR) {
      id = wc ? (v.w1 & 0xffffff) : v.w0;
      am = __builtin_amdgcn_ballot_w64(((v.w1 >> (24 + wa + 2 * wc)) & 1) != 0);
    } else {
      id = v.w0;
    }
  };
  auto head_of = [&](const int4& d, int batch) { return (int64_t)batch * p.H + d.x; };
  // Copies of this wave's share of a slice: K or V of slice u of block J into position b of its ring,
  // KiB by KiB: begin() once (destination and base), then one() for x = 0 .. LOADS - 1.  Past the end of
  // the list the last block is copied again (U == 2: the first one, or the next item's K and Q, see past),
  // into positions nobody reads: that costs less than a branch in the step sequence.
  auto copy_begin = [&](const unsigned char* base, int J, int u, uint32_t b, int x) {
    from = base + (int64_t)(SHARED && U == 1 ? __builtin_amdgcn_readfirstlane(J) : J) * BLOCK_BYTES + u * C::SL + x * 1024;
    set_copy_dst(ring + b * C::SL + share + x * 1024);
  };
  auto copy_one = [&](bool is_k, int x) { copy16_nth(x % 4, from, is_k ? k_src[x % C::KVAR] : v_src); };
  auto copy_k = [&](const unsigned char* base, int J, int u, uint32_t b) {
#pragma unroll
    for (int x = 0; x < C::LOADS; ++x) {
      if (x % 4 == 0) copy_begin(base, J, u, b, x);
      copy_one(true, x);
    }
  };
  auto copy_v = [&](const unsigned char* base, int J, int u, uint32_t b) {
#pragma unroll
    for (int x = 0; x < C::LOADS; ++x) {
      if (x % 4 == 0) copy_begin(base, J, u, NB + b, x);
      copy_one(false, x);
    }
  };
  auto k_of = [&](int64_t bh) { return reinterpret_cast<const unsigned char*>(p.k + bh * p.Nk * D) + src_off; };
  auto v_of = [&](int64_t bh) { return reinterpret_cast<const unsigned char*>(p.v + bh * p.Nk * D) + src_off; };

  auto tile_dt = [](int cc, int k) { return C::tile_dt(cc, k); };
  auto tile_qt = [](int cc, int k) { return C::tile_qt(cc, k); };
  auto has_lse = [](int cc) { return C::has_lse(cc); };
  auto by_key_group = [&](auto&& f) {
    if constexpr (C::NC == 4) {
      if (wc == 2) return f(std::integral_constant<int, 2>{});
      if (wc == 3) return f(std::integral_constant<int, 3>{});
    }
    if (wc == 0) f(std::integral_constant<int, 0>{});
    else f(std::integral_constant<int, 1>{});
  };
  auto store_tile = [&](const f32x4 (&res)[4], int64_t tok, int dt) { ::store_tile<D>(p.o, res, tok, dt, g); };

  // Split rows.  A chunk's partial result (f32, the accumulator tiles as the lanes hold them) goes to memory,
  // and is merged (log-sum-exp identity, the same one that combines per-chunk partial attention in Ring
  // Attention):
  //   LSE = log sum_k exp(LSE_k),  O = sum_k exp(LSE_k - LSE) O_k.
  // by dbsp_merge_kernel, or in place (p.merge_later is 0, see launch_fwd) by the wave that stores the last
  // chunk's share of a row.  Waves count for themselves (they finalise the same tiles in every chunk), so no
  // barrier is needed.
  // Pair rows: a query block may have no active block in some or all chunks (LSE_k = -inf).
  auto partial = [&](int64_t slot_no, int k, int e4) { return partial_of<C>(p.part_o, slot_no, w, k, e4, l); };
  auto merge_if_last = [&]() {                 // the current item's share is stored
    wait_copies<0>();                          // and has reached memory
    uint32_t* count = p.split_cnt + ((int64_t)bb * p.n_split + db.y) * C::NW + w;
    const int n_chunks = db.z;
    uint32_t before = 0;
    if (l == 0) before = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != (uint32_t)n_chunks - 1) return;
    if (l == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // ready for the next launch
    const int64_t first = (int64_t)bb * p.n_slots + db.w;
    const int64_t tok0 = head_of(da, bb) * p.Nq + (int64_t)da.y * C::QROWS + 64 * wa + r;
    const bool q_there = !PAIR || da.y * C::QROWS + 64 * wa < p.Nq;
    by_key_group([&](auto c_tag) {
      constexpr int WC = decltype(c_tag)::value;
#pragma unroll
      for (int k = 0; k < C::TPW; ++k) {
        const int qt = tile_qt(WC, k);
        merge_tile<C, D, 2, PAIR, false>(p, first, n_chunks, w, k, l, 64 * wa + 32 * qt + r, tok0 + 32 * qt, tile_dt(WC, k), has_lse(WC) && C::lse_tile(k), q_there);
      }
    });
  };
  int own_i = 0, own_b = n_own > 0 ? 0 : p.B;      // own list: position and batch entry of the current item (p.B: done)
  bool first_take = true;
  bool ready = false;            // the item's ids are there, its Q and first K slices on their way
  bool landed = false;           // and these have arrived, Q in its registers
  int stores = 0;                // what the item before stored: 1 = TPW tiles of O, 2 = a chunk's partial result, 0 = maybe nothing
  for (;;) {
    if (!ready) {
      if (own_b < p.B) {                          // the first item
        bb = 0;
        pos = it_begin;
      } else {
        uint32_t tp = blockIdx.x;
        if (n_first == 0 || !first_take) {
          if (total_tail <= n_first) break;
          if (t == 0) {
            const uint32_t raw = atomicAdd(&p.queue[0], 1u);
            // every workgroup fails once: the last to do so rewinds the queue for the next launch
            if (raw == total_tail - n_first + gridDim.x - 1) p.queue[0] = 0;
            tail_pos = n_first + raw;
          }
          __syncthreads();
          tp = __builtin_amdgcn_readfirstlane(tail_pos);
          __syncthreads();                        // everybody has read it before the next take overwrites it
        }
        first_take = false;
        if (tp >= total_tail) break;
        bb = (int)(tp / (uint32_t)p.n_tail);
        const int tq = (int)(tp % (uint32_t)p.n_tail);
        pos = p.n_placed + tq;
        if (t == 0) atomicAdd(&p.queue[1 + tq], 1u);     // take count, read back by dbsp_plan_tail_takes
      }
      da = g_sched[2 * pos];
      db = g_sched[2 * pos + 1];
      set_ids(load_ids(da, 0), ids, act);
      asm volatile("" : "+v"(ids));      // waited for here, so that nobody waits where the two ways meet
    }
    const uint64_t t0 = wall_clock64();
    const int I = da.y, n = __builtin_amdgcn_readfirstlane(da.w), slot = db.x;
    const int64_t bh = head_of(da, bb);
    const unsigned char *kbase = k_of(bh), *vbase = v_of(bh);
    const int nS = n * U;                     // slices
    auto id_of = [&](int T) { return __builtin_amdgcn_readlane(ids, T & 63); };
    auto act_of = [&](int T) { return ((act >> (T & 63)) & 1) != 0; };
    if (!ready) {
      if (q_by_lds) copy_q(bh, I);
      copy_k(kbase, id_of(0), 0, 0);
      copy_k(kbase, id_of(1 / U), 1 % U, 1);
      if constexpr (!SHARED) {
        load_q(bh, I);
        pin_q();      // (waited for where nothing else is under way, see the ids)
      } else {
        wait_copies<2 * C::LOADS>();
        __syncthreads();
        stores = 0;      // the first K slices are younger than any
      }
    }
    if (SHARED && !landed) {
      if (q_by_lds) {
        read_q();
      } else {
        load_q(bh, I);
        pin_q();
      }
    }
    id_words ids_next = {0, 0};
    if (n > 64) ids_next = load_ids(da, 64);
    // the next item of this workgroup's own list
    if (own_b < p.B && ++own_i == n_own) { own_i = 0; ++own_b; }
    const bool more = own_b < p.B;
    // (or this one again: loads in a branch would be waited for behind it, whatever else is under way)
    const int npos = more ? it_begin + own_i : pos, nbb = more ? own_b : bb;
    const int4 na = g_sched[2 * npos], nb = g_sched[2 * npos + 1];
    int ids_n = 0;
    uint64_t act_n = ~0ull;
    copy_v(vbase, id_of(0), 0, 0);
    // 128-token tiles at d = 128: the next item's first block of K, and its Q as if it were the second, take the places of the
    // copies past the end of this one's list, so that they land while it still runs and Q is read in front of the item's
    // last barrier: 1 us of the 6 us an item took besides its steps.  us without / with it: 16 heads, 513 x 513 blocks, 22
    // a row 1329 / 1312, 12 heads, 21 x 23 51.5 / 50.4, 40 heads, 256 x 256 5569 / 5566, dense 97 x 97 no difference.  Not for
    // items of one or two blocks, whose first copies are past their end already.
    const bool in_flow = U == 2 && more && n >= 3 && q_by_lds;

    pin_q();      // the wait for the Q loads belongs here, not at their first use behind later copies
    // the first K slices have landed; the first V slice and the stores of the item before may be under way
    if (!landed) {
      if (stores == 1) wait_copies<C::LOADS + 2 * C::TPW>();
      else if (stores == 2) wait_copies<C::LOADS + 4 * C::TPW>();      // (or twice as many)
      else wait_copies<C::LOADS>();
      if constexpr (SHARED) __syncthreads();
    }

    f32x16 o[C::DT][2];
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][qt][e] = 0.f;
    // the running max starts at the lowest finite value: scores of -inf (masked keys) then have probability 0
    // from the first unit on, where -inf minus -inf would be a NaN
    float m_run[2] = {-FLT_MAX, -FLT_MAX}, mc_run[2] = {-FLT_MAX, -FLT_MAX}, l_run[2] = {0.f, 0.f};

    f32x16 S[2];                  // scores of the last unit of each query tile
    bf16x8 P[2][2];               // [query tile][16-key step]: probabilities, packed as B operands
    // K operands of the current slice, V^T operands of the slice before ([16-key step * DT + d-tile]).  The first H
    // of them have two sets of registers, by the parity of their slice.
    bf16x8 kop[C::KS - H], kop2[2][H > 0 ? H : 1];
    s16x4 vop[C::KS - H][2], vop2[2][H > 0 ? H : 1][2];
    auto kop_of = [&](int par, int x) -> bf16x8& { return x < H ? kop2[par][x] : kop[x - H]; };
    auto vop_of = [&](int par, int x, int hf) -> s16x4& { return x < H ? vop2[par][x][hf] : vop[x - H][hf]; };
    auto read_k = [&](int at, int ks) {       // at: place of the slice in its ring
      kop_of(at & 1, ks) = as_bf16x8(*(LDS_PTR(u32x4))(uintptr_t)(k_rd[ks] + at * C::SL));
    };
    auto read_v = [&](int at, int x, int hf) {      // x = 16-key step * DT + d-tile; hf: keys 0 .. 7 or 8 .. 15 of the step
      const uint32_t a = v_rd[x % C::DT] + at * C::SL + ((x / C::DT) * 16 + hf * 8) * C::ROW_BYTES;
      vop_of(at & 1, x, hf) = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(uintptr_t)(a));
    };

    // blocks whose copies come next (SHARED: K of slice s + 4, V of slice s + 3; else of slices s + 2, s + 1)
    int jk = id_of(SHARED ? 3 / U : 1), jv = jk;
    // (U == 2) the block whose two slices of K are copied next, and what comes in the places of the first two past the
    // end of the list
    [[maybe_unused]] const unsigned char *k_next = nullptr, *k_past = nullptr, *past[2] = {kbase + (int64_t)id_of(0) * BLOCK_BYTES, kbase + (int64_t)id_of(0) * BLOCK_BYTES};
    [[maybe_unused]] bool a_prev = false, a_cur = act_of(0), a_next = act_of(1), a_next2 = false;

    // One step: K Q^T of (slice s, tile QT), softmax of the step before, V^T P^T of the step before
    // that = (slice s-1, tile QT).  AT = place of slice s in its ring, WAIT: copies that its barrier leaves under way.  What else the two steps of a slice do is
    // placed by sub-slot z = 0 .. 2 SUB - 1 of the two.
    auto step = [&](int s, auto qt_tag, auto at_tag, auto wait_tag, auto qk_tag, auto sm_tag, auto pv_tag) __attribute__((always_inline)) {
      constexpr int QT = decltype(qt_tag)::value, AT = decltype(at_tag)::value, ODD = AT & 1, WAIT = decltype(wait_tag)::value;
      constexpr bool QK = decltype(qk_tag)::value, SM = decltype(sm_tag)::value, PV = decltype(pv_tag)::value;
      constexpr bool FIRST = SHARED && !PV;       // shared slices: the item's first slice
      constexpr int QS = 1 - QT;                  // the softmax stage's tile
      constexpr int UU = U == 2 ? ODD : 0;        // slice s inside its block
      constexpr int SUB = C::SUB;
      // Softmax of the 16 scores in three stages one sub-slot apart (scaled difference, exponential,
      // sum and packing), so that no instruction waits for the one right before it.
      float xs[16], pr[16];
      float ls0 = 0.f, ls1 = 0.f, l_spec = 0.f;
      bool pend = false;
      float mc_eff = mc_run[QS];                  // the running max the probabilities are formed against
      if constexpr (PAIR) mc_eff = ((QT == 0 && UU == 0) ? a_prev : a_cur) ? mc_run[QS] : INFINITY;   // not this wave's block: exp2(-inf) = 0
      auto stage_x = [&](int j) { xs[j] = __builtin_fmaf(S[QS][j], c, -mc_eff); };
      auto stage_e = [&](int j) { pr[j] = __builtin_amdgcn_exp2f(xs[j]); };
      auto stage_s = [&](int j) {
        if (j == 0) ls0 = pr[0];
        else if (j == 1) ls1 = pr[1];
        else if (j & 1) ls1 += pr[j];
        else ls0 += pr[j];
        if (j & 1) {
          u32x4 pb = __builtin_bit_cast(u32x4, P[QS][j / 8]);
          pb[(j % 8) / 2] = pack_bf16x2(pr[j - 1], pr[j]);
          P[QS][j / 8] = as_bf16x8(pb);
        }
      };
      auto softmax_sub = [&](int y) __attribute__((always_inline)) {             // y = 0 .. SUB - 1
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int e = C::exp_at(j);
          if (y == (e > 0 ? e - 1 : 0)) stage_x(j);
          if (y == e) stage_e(j);
          if (y == e + 1) stage_s(j);
        }
        if (y == C::SOFTMAX_END) {
          if (C::exp_at(15) == y) { stage_s(14); stage_s(15); }
          const float ls = ls0 + ls1;
          pend = __builtin_amdgcn_ballot_w64(ls > SPEC_SUM_LIMIT) != 0;
          l_spec = l_run[QS] + ls;
        }
      };
      // LDS operands: K of slice s + 1 and V of slice s, each into registers whose last use is behind it.
      auto reads = [&](int y) __attribute__((always_inline)) {
        const int z = QT * SUB + y;
        if constexpr (SHARED) {
#pragma unroll
          for (int k = 0; k < 3 * H; ++k)
            if (z == (FIRST ? SUB + k : C::read_at(k))) {
              if (k % 3 == 0) read_k((AT + 1) % NB, k / 3);
              else read_v(AT, k / 3, k % 3 - 1);
            }
        }
        if (QT == 1 && y / 2 >= H) {
          if (y % 2 == 0) read_k((AT + 1) % NB, y / 2);
          else { read_v(AT, y / 2, 0); read_v(AT, y / 2, 1); }
        }
      };
      // Copies, spread over the steps' sub-slots.
      //   Own slices: in steps with QT = 0, K of slice s+2 and V of slice s+1 into the positions of K of
      //   slice s and V of slice s-1, whose operands are in registers by the second half of the step.
      //   Shared slices: behind the barrier of slice s, K of slice s+4 and V of slice s+3 into the positions of K of
      //   slice s and V of slice s-1, which that barrier has retired; they have the two slices after this one to land.
      //   Address and destination of a group are made a sub-slot ahead.
      auto copies = [&](int y) __attribute__((always_inline)) {                  // sub-slot y
        const int z = QT * SUB + y;
        if (FIRST && QT == 0) {                   // K of slices 2 and 3, V of 1 and 2, one copy a sub-slot
          const int grp = y / C::LOADS, x = y % C::LOADS, sl = grp == 0 ? 2 : grp == 1 ? 1 : grp == 2 ? 3 : 2;
          const bool is_k = grp % 2 == 0;
          if (x == 0) copy_begin(is_k ? kbase : vbase, id_of(sl / U), sl % U, is_k ? sl : NB + sl, 0);
          copy_one(is_k, x);
          return;
        }
        if constexpr (U == 2) {                   // the block of K of slice s + 4, a little at a time; V's is one behind
          const int T = (s + 4) / 2;
          if (z == (FIRST ? SUB : 1)) {
            jv = jk;
            if constexpr (ODD == 0) jk = id_of(T);
          }
          if constexpr (ODD == 0) {
            if (z == (FIRST ? SUB : 2)) k_next = kbase + (int64_t)jk * BLOCK_BYTES;
            if (!FIRST && z == 3) k_past = if_less(T, n + 1, past[0], past[1]);
            if (!FIRST && z == 4) k_next = if_less(T, n, k_next, k_past);
          }
        }
#pragma unroll
        for (int k = 0; k < 2 * C::LOADS; ++k) {
          const int x = k % C::LOADS, at = FIRST ? SUB + 2 + k : C::copy_at(k);
          const bool is_k = k < C::LOADS;
          if (z == at) copy_one(is_k, x);
          if (x % 4 == 0 && z == at - 1) {
            if (k == 0) {
              if constexpr (!SHARED) wait_reads<D, 63>();    // the operand reads of the step before are done
              if constexpr (U == 1) {
                jv = jk;
                jk = id_of(s + (SHARED ? 4 : 2));
              }
              if constexpr (PAIR && ODD == 0) a_next2 = act_of((s + 4) / U);
            }
            if (is_k && U == 2) copy_begin(k_next, 0, UU, AT, x);
            else if (is_k) copy_begin(kbase, jk, UU, SHARED ? AT : ODD, x);
            else copy_begin(vbase, jv, U == 2 ? 1 - UU : 0, NB + (SHARED ? (AT + 3) % NB : 1 - ODD), x);
          }
        }
      };
      if constexpr (!SHARED && QK && QT == 1) wait_copies<2 * C::LOADS>();      // K of slice s+1 and V of slice s have landed; the copies of the step before may be under way
      // K of slice s+1 and V of slice s have landed for everybody (what is younger: the copies of the last two slices, of
      // which the wait may leave fewer), and everybody has read all before them
      auto publish = [&](int y) __attribute__((always_inline)) {
        if (!SHARED || QT != FIRST || y != (FIRST ? 0 : C::BARRIER_AT)) return;
        wait_reads<D, WAIT>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      };
      // (by constants, not an unrolled loop: with the tables the loop would be past what the compiler unrolls)
      for_each<SUB>([&](auto y_tag) __attribute__((always_inline)) {
        constexpr int y = decltype(y_tag)::value, x = y / 2;
        if constexpr (y % 2 == 0) {
          if constexpr (QK) {
            if constexpr (x == 0) {
#pragma unroll
              for (int e = 0; e < 16; ++e) S[QT][e] = 0.f;
            }
            S[QT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop_of(ODD, x), q[QT][x], S[QT], 0, 0, 0);
          }
        } else if constexpr (PV) {
          const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vop_of(1 - ODD, x, 0), vop_of(1 - ODD, x, 1), 0, 1, 2, 3, 4, 5, 6, 7));
          o[x % C::DT][QT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, P[QT][x / C::DT], o[x % C::DT][QT], 0, 0, 0);
        }
        if constexpr (QK) { publish(y); reads(y); }
        if constexpr (SM) softmax_sub(y);
        if constexpr (QK) copies(y);
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (PAIR && QK && QT == 1 && UU == U - 1) { a_prev = a_cur; a_cur = a_next; a_next = a_next2; }   // on to the next block
      if constexpr (SM) {
        asm volatile("" ::"v"(P[QS][0]), "v"(P[QS][1]), "v"(l_spec));
        if (__builtin_expect(pend, 0)) {      // raise the running max, redo the unit, rescale
          const f32x16& sv = S[QS];
          float mx0 = fmaxf(fmaxf(sv[0], sv[1]), sv[2]), mx1 = fmaxf(fmaxf(sv[3], sv[4]), sv[5]);
#pragma unroll
          for (int e = 6; e < 14; e += 4) {
            mx0 = fmaxf(fmaxf(mx0, sv[e]), sv[e + 1]);
            mx1 = fmaxf(fmaxf(mx1, sv[e + 2]), sv[e + 3]);
          }
          mx0 = fmaxf(fmaxf(mx0, sv[14]), sv[15]);
          const float m_new = fmaxf(m_run[QS], max_xor32(fmaxf(mx0, mx1)));
          const float alpha = __builtin_amdgcn_exp2f((m_run[QS] - m_new) * c);
          m_run[QS] = m_new;
          mc_run[QS] = fmaxf(m_new * c, -FLT_MAX);
          float a0 = 0.f, a1 = 0.f;
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            uint32_t w4[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
              const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[8 * hf + 2 * e2], c, -mc_run[QS]));
              const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[8 * hf + 2 * e2 + 1], c, -mc_run[QS]));
              a0 += p0;
              a1 += p1;
              w4[e2] = pack_bf16x2(p0, p1);
            }
            const u32x4 pb = {w4[0], w4[1], w4[2], w4[3]};
            P[QS][hf] = as_bf16x8(pb);
          }
          l_spec = l_run[QS] * alpha + (a0 + a1);
#pragma unroll
          for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][QS][e] *= alpha;
        }
        l_run[QS] = l_spec;
      }
    };

    using T0 = std::integral_constant<int, 0>;
    using T1 = std::integral_constant<int, 1>;
    using Yes = std::true_type;
    using No = std::false_type;
    using Early = std::integral_constant<int, C::UNDER_WAY>;
    using Steady = std::integral_constant<int, SCATTERED ? C::LOADS : C::UNDER_WAY>;
#pragma unroll
    for (int x = 0; x < C::KS; ++x) read_k(0, x);
    auto next_ids = [&](int T) {       // before block id T is asked for: it may start a new group of 64
      if ((T & 63) == 0) {
        set_ids(ids_next, ids, act);
        if (T + 64 < n) ids_next = load_ids(da, T + 64);
      }
    };
    auto slice_of = [&](int s, auto at_tag, auto wait_tag) __attribute__((always_inline)) {       // both steps of a slice
      step(s, T0{}, at_tag, wait_tag, Yes{}, Yes{}, Yes{});
      step(s, T1{}, at_tag, wait_tag, Yes{}, Yes{}, Yes{});
    };
    auto slice = [&](int s, auto at_tag) __attribute__((always_inline)) { slice_of(s, at_tag, Steady{}); };
    step(0, T0{}, T0{}, Early{}, Yes{}, No{}, No{});
    const id_words words_n = load_ids(na, 0);
    const id_words first_n = {g_kv_idx[na.z], PAIR ? g_kv_idx[na.z + 1] : 0};
    step(0, T1{}, T0{}, Early{}, Yes{}, Yes{}, No{});
    // The loops go once round a ring, so that places in it are constants.
    int s = 1;
    if constexpr (SHARED) {
      using T2 = std::integral_constant<int, 2>;
      using T3 = std::integral_constant<int, 3>;
      if constexpr (U == 2) {
        slice_of(s++, T1{}, Early{});
        if (in_flow) {       // an even number of blocks: the third and fourth slice's places come second
          past[n & 1] = k_of(head_of(na, nbb)) + (int64_t)(PAIR && wc ? first_n.w1 & 0xffffff : first_n.w0) * BLOCK_BYTES;
          past[1 - (n & 1)] = q_of(head_of(na, nbb), na.y);
        }
      }
      while (s < nS) {
        if constexpr (U == 1) {
          slice(s, T1{});
          if (++s >= nS) break;
        }
        slice(s, T2{});
        if (++s >= nS && U == 1) break;
        slice(s, T3{});
        if (++s >= nS) break;
        next_ids((s + 4) / U);                   // (groups of 64 start at a multiple of four slices)
        slice(s, T0{});
        ++s;
        if constexpr (U == 2) slice(s++, T1{});
      }
    } else {
      for (; s + 1 < nS; s += 2) {
        next_ids(s + 2);
        slice(s, T1{});
        next_ids(s + 3);
        slice(s + 1, T0{});
      }
      if (s < nS) slice(s, T1{});
    }
    set_ids(words_n, ids_n, act_n);
    const int jn0 = __builtin_amdgcn_readlane(ids_n, 0), jn1 = __builtin_amdgcn_readlane(ids_n, 1 / U);
    auto drain = [&]() {       // where the operands have two sets of registers, the last slice's are in the odd one (see Cfg)
      step(nS, T0{}, T0{}, Steady{}, No{}, Yes{}, Yes{});
      if constexpr (!SHARED) {
        if (more) load_q(head_of(na, nbb), na.y);
      }
      step(nS, T1{}, T0{}, Steady{}, No{}, No{}, Yes{});
    };
    drain();

    // ---- end of item: combine the slices' shares of the keys and store.  Wave c finalises TPW of the
    //      accumulator tiles and hands the others to the waves of their slices.
    if (!SHARED && more) wait_copies<2 * C::KS>();       // all copies; the loads of the next item's Q may be under way
    else wait_copies<0>();
    if constexpr (SHARED) __syncthreads();    // everybody is done with the slices: the rings become the exchange area
    if (more && !in_flow) {
      if (q_by_lds) copy_q(head_of(na, nbb), na.y);
      const unsigned char* kb = k_of(head_of(na, nbb));
      copy_k(kb, jn0, 0, 0);
      copy_k(kb, jn1, 1 % U, 1);
    }
    const int64_t tok0 = bh * p.Nq + (int64_t)I * C::QROWS + 64 * wa + r;
    // pair rows: false for the waves of a query block past the end of the head (they still fill their
    // rows of a split row's partial result: zeros and -inf)
    const bool q_there = !PAIR || I * C::QROWS + 64 * wa < p.Nq;
    const int64_t ps = (int64_t)bb * p.n_slots + slot;
    auto finish = [&](auto c_tag) {
      constexpr int WC = decltype(c_tag)::value;
      // this wave's outbox: TPW tiles for each of the other slices, in ascending order of their slice
      auto box = [&](int from_c, int to_c, int k) {
        const int idx = (to_c < from_c ? to_c : to_c - 1) * C::TPW + k;
        return reinterpret_cast<float*>(lds + from_c * C::RING + (C::RING - NQ * C::XCH) + wa * C::XCH) + idx * 1024;
      };
      float lf[2];
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        lf[qt] = sum_xor32(l_run[qt]);
        xstat[w][(2 * qt + 0) * 64 + l] = m_run[qt];
        xstat[w][(2 * qt + 1) * 64 + l] = lf[qt];
      }
#pragma unroll
      for (int cc = 0; cc < C::NC; ++cc) {
        if (cc == WC) continue;
#pragma unroll
        for (int k = 0; k < C::TPW; ++k) {
          const f32x16& ov = o[tile_dt(cc, k)][tile_qt(cc, k)];
          float* to = box(WC, cc, k);
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            const f32x4 f = {ov[4 * e4], ov[4 * e4 + 1], ov[4 * e4 + 2], ov[4 * e4 + 3]};
            *reinterpret_cast<f32x4*>(to + (e4 * 64 + l) * 4) = f;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        if (C::NC == 4 && qt != tile_qt(WC, 0)) continue;      // no tile of these queries here
        float ms[C::NC], f[C::NC];
        float mt = m_run[qt];
#pragma unroll
        for (int cc = 0; cc < C::NC; ++cc) {
          ms[cc] = (cc == WC) ? m_run[qt] : xstat[wa * C::NC + cc][(2 * qt + 0) * 64 + l];
          mt = fmaxf(mt, ms[cc]);
        }
        float lt = 0.f;
#pragma unroll
        for (int cc = 0; cc < C::NC; ++cc) {
          f[cc] = __builtin_amdgcn_exp2f((ms[cc] - mt) * c);
          lt += f[cc] * ((cc == WC) ? lf[qt] : xstat[wa * C::NC + cc][(2 * qt + 1) * 64 + l]);
        }
        // a query block of pair rows may have nothing in this item, and a query's scores in a chunk may all be
        // -inf (all maxima at their start, sums 0): O = 0, LSE = -inf, which the merge leaves out
        const float inv = ((PAIR || slot >= 0) && is_zero(lt)) ? 0.f : 1.0f / lt;
#pragma unroll
        for (int cc = 0; cc < C::NC; ++cc) f[cc] *= inv;
        const int64_t tok = tok0 + 32 * qt;
        const int qloc = 64 * wa + 32 * qt + r;
#pragma unroll
        for (int k = 0; k < C::TPW; ++k) {
          if (tile_qt(WC, k) != qt) continue;
          const f32x16& ov = o[tile_dt(WC, k)][qt];
          f32x4 res[4];
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            res[e4] = f32x4{ov[4 * e4] * f[WC], ov[4 * e4 + 1] * f[WC], ov[4 * e4 + 2] * f[WC], ov[4 * e4 + 3] * f[WC]};
#pragma unroll
            for (int cc = 0; cc < C::NC; ++cc) {
              if (cc == WC) continue;
              const f32x4 y = *reinterpret_cast<const f32x4*>(box(cc, WC, k) + (e4 * 64 + l) * 4);
              res[e4].x += y.x * f[cc];  res[e4].y += y.y * f[cc];  res[e4].z += y.z * f[cc];  res[e4].w += y.w * f[cc];
            }
          }
          if (slot >= 0 && p.merge_later) {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) store_shared(partial4_of<C>(p.part_o, ps, w, k, e4, l), res[e4]);
          } else if (slot >= 0) {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
              store_shared(partial(ps, k, e4), res[e4].x, res[e4].y);
              store_shared(partial(ps, k, e4) + 128, res[e4].z, res[e4].w);
            }
          } else if (q_there) {
            store_tile(res, tok, tile_dt(WC, k));
          }
        }
        if (g == 0) {
          // every wave that finalises a tile of these queries stores the LSE of a chunk (the same bits), so
          // that its own count vouches for it
          const float lse = mt * p.scale + __logf(lt);
          if (slot >= 0) __hip_atomic_store(p.part_lse + ps * C::QROWS + qloc, lse, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          else if (has_lse(WC) && p.lse != nullptr && q_there) p.lse[tok] = lse;
        }
      }
    };
    by_key_group(finish);
    if (in_flow) {
      read_q();
      pin_q();
    } else if constexpr (SHARED) {     // the next item's Q has landed; its first K slices and the stores may be under way
      if (slot >= 0) wait_copies<2 * C::LOADS + 4 * C::TPW>();
      else if (q_there) wait_copies<2 * C::LOADS + 2 * C::TPW>();
      else wait_copies<2 * C::LOADS>();
    }
    __syncthreads();      // the exchange has been read before the next item's copies overwrite it
    if (slot >= 0 && !p.merge_later) merge_if_last();
    stores = slot >= 0 ? 2 : q_there ? 1 : 0;
    ready = more;
    landed = in_flow;
    if (more) {
      pos = npos;
      da = na;
      db = nb;
      bb = nbb;
      ids = ids_n;
      act = act_n;
    }
    busy += wall_clock64() - t0;
  }
  if (t == 0) {
    p.busy[part] = busy;
    const uint32_t hw = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 4);    // HW_ID
    const uint32_t xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20);   // XCC_ID[3:0]
    const uint32_t cu = (hw >> 8) & 0xf, sh = (hw >> 12) & 0x1, se = (hw >> 13) & 0x7;
    p.hw_id[part] = (xcc << 16) | (se << 8) | (sh << 4) | cu;
  }
}

template <int D, int NQ, int NC, int U, bool PAIR = false, bool SCATTERED = false>
hipError_t launch_fwd(dbsp_fwd_params p, int grid, hipStream_t stream) {
  using C = Cfg<D, NQ, NC, U>;
  // Who merges split rows.  In place, the wave that ends a row merges its share, TPW tiles of every chunk one
  // after the other, where there are no more items than partitions, all batch entries counted (a workgroup mostly
  // has one then, but a placed item runs there once for every batch entry); a launch of its own has a wave
  // for every tile and costs 2 us behind the kernel.  us in place / by a second launch, one item at most for
  // a workgroup: 64-token blocks at d = 64, 3 chunks 24.7 / 27.0, 7 chunks 30.5 / 31.3, 14 chunks 38.0 / 29.8;
  // 128 at d = 128, 3 chunks 226 / 227, 4 chunks 162 / 158.  Where items queue up, who merges falls behind,
  // ends its next rows last and merges these as well: 12 heads, 21 x 23 blocks of 128, up to 4 chunks
  // 72 / 65; 10 heads, 128 x 256, up to 8 chunks 1068 / 771.
  p.merge_later = p.max_chunks > 0 && (p.max_chunks * C::TPW > kTilesInPlace || !p.in_place_ok);
  // the dynamic-LDS limit is a per-device function attribute: set it once per device
  static std::atomic<uint32_t> attr_set_mask{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint32_t bit = 1u << (dev & 31);
  if (!(attr_set_mask.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dbsp_fwd_kernel<D, NQ, NC, U, PAIR, SCATTERED>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set_mask.fetch_or(bit, std::memory_order_release);
  }
  const int4* sched = reinterpret_cast<const int4*>(p.sched);
  hipLaunchKernelGGL((dbsp_fwd_kernel<D, NQ, NC, U, PAIR, SCATTERED>), dim3(grid), dim3(C::NT), C::LDS_BYTES, stream, p, p.kv_idx, sched, p.part_ptr);
  e = hipGetLastError();
  if (e != hipSuccess || !p.merge_later) return e;
  const dim3 merge_grid((uint32_t)p.B * (uint32_t)p.n_split, C::TPW);
  hipLaunchKernelGGL((dbsp_merge_kernel<D, NQ, NC, U, PAIR>), merge_grid, dim3(C::NT), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t dbsp_launch_fwd(const dbsp_fwd_params& p, int block, int d, bool pair, int grid, hipStream_t stream) {
  if ((block != 64 && block != 128) || (d != 64 && d != 128) || (pair && (block != 64 || d != 128))) return hipErrorInvalidValue;
  // How many copies a slice's barrier leaves under way, at d = 128 and 128-token tiles.  Under a placement without
  // locality K and V come from behind the L2s, and long launches are bound by that: with two slices' copies under
  // way every second die then gets more of the fabric than its neighbour (busy times 6.2 and 7.0 ms, with the shorter wait
  // all at 6.6), nothing evens out the end, and the slower dies make the launch longer.  us, two slices' copies / one V
  // slice's, with the greedy's items in the order of their heads and its partitions dealt to the dies one by one: 40 heads,
  // 256 x 256 blocks 7755 / 7175; pair rows, 40 heads, 512 x 512 7460 / 6860 (5, 6 or 8 copies in place of 4, or the short wait
  // at every second slice, keep part of the loss, 2 copies cost 1 - 10 % of other cases).  That is how the naive
  // and the reward-biased placement run, and so does a greedy one of an item at most a workgroup and at least seven eighths of the
  // chip's workgroups, which has no order and rows of all lengths: 16 heads, 16 x 256 blocks 238 - 271 / 229 - 254 and 8 heads, 32 x 900
  // 819 - 883 / 772 - 832 (ranges over five kinds of masks), 512 workgroups, 16 heads, 32 rows of 100 to 400 of 500 blocks
  // 1125 / 1028, pair rows, 16 heads, 16 x 400 527 / 507, 4 heads, 64 x 400 317 / 318, 32 heads, 8 x 400 382 / 378; 224 workgroups, 8, 16
  // and 32 heads 324 / 322, 344 / 338, 345 / 353.  With fewer nothing is short, and the longer wait is worth its copies: 192 workgroups,
  // 4, 8, 16 and 32 heads 277 / 278, 299 / 299, 310 / 308, 309 / 326, 128 260 / 263, 269 / 275, 276 / 303, 281 / 325, 32 heads, 2 rows
  // each 275 / 343.  The rounds' and, longest items first and partitions in a row on a die
  // (see run_order in api.hip), the greedy's run does better with two slices' copies: rounds, 40 heads, 256 x 256 5646 / 5666,
  // dense 97 x 97 up to 4 %; greedy, 40 heads, 256 x 256 5969 / 6187, 24 heads, 928 x 928 36.9 / 38.0 ms, pair rows, 40 heads, 512 x 512
  // 5816 / 5933, 16 heads, 513 x 513 1402 / 1410; 12 heads, 21 x 23, 5 blocks an item, 56.2 / 55.8.  So do the greedy's short items,
  // which run as listed: 48 heads, 256 x 256 blocks, 3 an item 503 / 516, 40 heads, 160 x 160, 3.2 an item 273 / 280, pair rows, 40 heads,
  // 256 x 256, 2.9 an item 129 / 131; with a twentieth of the rows long, 24 heads, 928 x 928 1071 / 1086.  An item's first two
  // slices have their copies in front of them in either case.  d = 64 takes half the bytes a clock and loses nothing by
  // two slices' copies.
  const bool scattered = !p.local;
  if (pair) return scattered ? launch_fwd<128, 2, 2, 2, true, true>(p, grid, stream) : launch_fwd<128, 2, 2, 2, true>(p, grid, stream);
  if (block == 64) return d == 128 ? launch_fwd<128, 1, 2, 1>(p, grid, stream) : launch_fwd<64, 1, 2, 1>(p, grid, stream);
  if (d == 64) return launch_fwd<64, 2, 4, 1>(p, grid, stream);
  return scattered ? launch_fwd<128, 2, 2, 2, false, true>(p, grid, stream) : launch_fwd<128, 2, 2, 2>(p, grid, stream);
}
