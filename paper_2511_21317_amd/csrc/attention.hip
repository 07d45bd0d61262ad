// Stage 3: attention over the reduced per-head sequences (paper Sec. 3.2 Eq. 3-4):
//   O = softmax(Q K^T * scale) V, per head, no mask, ragged (M_q[h], M_k[h]).
//
// Flash-style single pass with bf16 MFMA (v_mfma_f32_16x16x32_bf16) and fp32 softmax state.
// The kernel is bound by the matrix cores (4*M_q*M_k*64 flop per head against a few MB of
// K/V that stay in L2 / Infinity Cache); with d_head = 64 the softmax needs about as many
// vector-ALU cycles as the two matrix products need MFMA cycles, so the design is about
// (a) taking vector instructions out of the inner loop and (b) giving every wave independent
// MFMA and vector work in the same stretch of code so that both pipes run at once.
//
// Why 16x16x32.  Under these kernels the chip is at its power limit and the clock follows the energy of an
// instruction: a register-only loop of 16x16x32 products sustains 1.95 PFLOP/s (2.0 GHz), one of
// 32x32x16 products - same nominal rate, half the instructions - 1.76 (1.77 GHz).  With the instruction
// mix of a step (products, exp2, packs) in registers a step takes 307 against 330 ns, although the finer
// products leave less room between them for vector instructions (595 against 527 cycles).  This kernel:
// 16 heads x 16384 x 16384 860 -> 807 us, x 28700 x 28700 2.51 -> 2.45 ms.
//
// Work decomposition
//   * workgroup = NW waves = one tile of 16*NQ*NW query rows of one head; a wave owns 16*NQ rows;
//   * K/V are streamed in tiles of 64 rows through LDS, double buffered, one barrier per tile;
//   * blockIdx -> tile mapping is XCD-aware: workgroups are dispatched round-robin over the 8
//     XCDs, so tile = (bid % 8) * (grid/8) + bid / 8 gives every XCD a contiguous range of
//     tiles, i.e. about two heads, whose K/V then stay in that XCD's L2.
//
// Transposed formulation.  Each wave computes S^T = K Q^T (A = K tile from LDS, B = Q^T from
// registers) so that in the 16x16 accumulator layout a lane owns ONE query column and 4 of the
// 16 key rows: the softmax reductions are sums inside a lane plus two exchanges between the four lane
// groups at the very end, and every per-row quantity is a per-lane scalar for the O^T = V^T P^T
// accumulators as well.  P^T goes from the accumulator registers straight into the B operand of
// the second MFMA (fp32 -> bf16 in registers, no LDS round trip).  That fixes which 8 keys a lane
// group g supplies per step of 32: {4g + 0..3, 16 + 4g + 0..3}.  The matching A operand
// (V^T: a lane's channel, those 8 keys) comes out of the row-major V tile through two transposing
// LDS reads (ds_read_b64_tr_b16), so V is never transposed in memory or in registers.
//
// Both tiles go from global memory straight into LDS (global_load_lds_dwordx4: no registers, no
// LDS store instructions); every lane fetches the 16-byte chunk that belongs at its position
// under the tile's swizzle, which keeps the operand reads free of bank conflicts.
//
// Software pipeline.  Work is cut into steps of 32 keys.  In step t a wave issues, in one
// basic block, the QK^T MFMAs of step t+1, the PV MFMAs of step t-1 and the softmax of step t:
// the 32 MFMAs do not depend on the ~50 vector instructions next to them, so the matrix core
// and the vector ALU overlap inside a single wave (two waves per SIMD then fill what is left).
// V lags K by one tile in LDS because of the t-1.  In the steady state the order of issue is
// written out (steady_step(): one MFMA, then an exp2 and at times a pack, behind a scheduling fence; two
// MFMAs and then their vector instructions together take 40 % more cycles), the
// loop runs two tiles per trip so that the LDS buffer indices are constants, and the global->LDS
// requests of an iteration are issued behind the last LDS read of its first step.
//
// Softmax without a running maximum.  softmax is invariant to the per-row shift m, and fp32 /
// bf16 keep their relative precision over the whole exponent range, so m only has to keep
// exp2(s - m) inside that range - it does not have to be the maximum.  When stage 2 has left the
// merged keys multiplied by scale * log2(e) ("log2 keys": the factor goes into the fp32 mean before its
// one rounding to bf16, so nothing is rounded twice), the raw MFMA scores are the base-2 logits and the
// kernel (SHIFT = false) uses the weights exp2(s) as they are.  With any other keys (SHIFT = true) it
// takes one fma per score, scale and shift, with m the row's exact maximum over the first 32 keys until a step's
// weights outgrow it (guard_step()).  The row sums come from the matrix cores (row_sum_operand()).  A tile without
// shifts is checked once, at its end: if a row's sum is outside [2^-64, 2^64] (or inf / NaN), the workgroup takes
// the tile again with per-row shifts (16 x 9000 x 9000, one key 60 nats above the rest: 514 us against 266; with
// running maxima 747, with a second launch for marked tiles 645).  A key group's or piece's own sum may be smaller
// (half of the keys masked: 16 x 2048 x 8192 179 -> 57 us) if the row's is not: the groups are checked together, a
// piece looks at a few key tiles of the others (rest_holds).  The same check behind the shifts finds what they cannot
// hold (logits beyond 2^30, NaN next to a number): running maxima, not pipelined (running_max_step(): the classic
// online softmax).
// Measured against a guard that sums on the vector ALU (a dot2 against ones and a compare per score pair) and, for
// log2 keys, a second launch that redid marked tiles: 16 ragged heads of 5500 x 9000 plain keys 219 -> 205 us, two
// 16 x 16 frames 27.3 -> 24.3 us a layer.
//
// End of a launch.  A CU runs its 256-row tiles two at a time, but one alone at 0.8 of the rate of two,
// so the launch time follows the largest number of whole tiles a CU gets.  When the caller has given
// scratch memory, the tiles in excess of a multiple of the CU count are not run whole: their work
// is cut into equal shares over the keys, one per CU, that are dispatched behind the whole
// tiles, and attention_split_reduce_kernel adds the pieces of every tile up (attention_split.hpp).
//
// Few rows.  With less than a 256-row tile per CU a launch is as long as one workgroup's walk over the
// keys.  Workgroups with KS key groups walk a KS-th of them and the groups meet in LDS at the end - no scratch
// memory, no second kernel.  Tiles of 32 rows (4 waves, 4 groups), 64 (8 waves, 4), 128 (8 waves, 2) have waves of 32
// rows: a short walk is a chain of waits (LDS reads at the head of a tile, the tile's arrival, the barrier), which two
// waves per SIMD or fewer rows per wave shorten more than their reading twice the LDS per product costs.  Long
// walks are bound by the LDS reads and the products: waves of 64 rows, tiles of 128 (8 waves, 4 groups) and 256 rows
// (8 waves, 2).  16 heads x 500 x 500 9.2 (128-row tiles of one group) -> 6.7 us, 1000 x 1000 12.1 -> 10.3, 1384 x 1384
// 16.9 -> 15.3, 1000 x 6000 40.5 (64-row tiles, 4 waves of 64 rows) -> 34.8; a layer of 2 frames of 16 x 16 17.4 ->
// 14.8.  All times and the choice: choose_key_groups().
#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "attention_split.hpp"
#include "dev_common.hpp"
#include "kernels.hpp"

namespace httm {

namespace {

constexpr int kKvTile = 64;
constexpr int kStep = 32;                               // keys per pipeline step

struct AttnArgs {
  const bf16_t* q;
  const bf16_t* k;
  const bf16_t* v;
  bf16_t* o;
  float scale_log2;  // scale * log2(e); 1 when the keys carry that factor already
  int32_t H;
  int32_t n_full;                             // tiles with all BQ query rows
  int32_t n_ragged;                           // heads whose last tile is partial
  int32_t full_per_xcd;                       // ceil(n_full / 8)
  int32_t ragged_per_xcd;                     // ceil(n_ragged / 8)
  int32_t tile_start[kAttnMaxHeads + 1];      // first full tile of every head
  int32_t ragged_head[kAttnMaxHeads];         // head of every partial tile
  int64_t q_off[kAttnMaxHeads];               // first query row of every head, and how many
  int32_t q_rows[kAttnMaxHeads];
  int64_t k_off[kAttnMaxHeads + 1];
  // When set, a second set of query tiles is described by device memory: rows of head h are
  // [dev_q_off[h], dev_q_off[h+1]) and workgroup t takes tile (head, first row) =
  // (dev_tiles[1+2t], dev_tiles[2+2t]) for t < dev_tiles[0].
  // The workgroups behind the whole tiles and the segments take these tiles; their queries and outputs
  // are q2 / o2.
  const int32_t* dev_q_off;
  const int32_t* dev_tiles;
  const bf16_t* q2;
  bf16_t* o2;
  // Every XCD (workgroup b goes to XCD b % 8) walks a sequence of full_per_xcd + ragged_per_xcd whole
  // tiles and then split_per_xcd shares of the tiles that run in segments over the keys
  // (attention_split.hpp).  A segment writes
  // un-normalised fp32 results into its slot of the scratch memory and attention_split_reduce_kernel
  // adds them up.  The workgroups behind main_blocks = 8 * (sequence length) take the device-side tile
  // list.  n_ragged / ragged_head and n_full count only the tiles that stay whole.
  int32_t split_per_xcd;
  int32_t main_blocks;
  int32_t share_block0;   // 512-row tiles: the shares come last, from this workgroup on
  int32_t dev_halves;     // 256-row tiles: 1 if the device-side list's are 512-row tiles, which two workgroups take then
  float* split_o;   // [slots * 256][64] sums of weight * v
  float* split_l;   // [slots * 256]     sums of weights
  float* split_m;   // [slots * 256]     the rows' shifts
  SplitPlan sp;
  UnmergeTarget um;
};
static_assert(sizeof(AttnArgs) <= 4096, "kernel arguments are limited to 4 KB");

// V tile in LDS: 64 rows of 128 bytes, written by global->LDS loads like the K tile; the 16-byte
// chunk c of row r sits at chunk position c ^ (2 * ((r >> 1) & 3)), so that the eight rows which half a
// transposing read touches (32 bytes each, same channels) fall into eight different 32-byte bank groups.
__device__ __forceinline__ int v_swizzle(int row) { return ((row >> 1) & 3) << 1; }

// One tile of K or V in LDS
typedef bf16_t KvTile[kKvTile * kDHead];

typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
// One half of a pair of query tiles' P^T: the B operand of a 16x16x32 MFMA
__device__ __forceinline__ bf16x8 p_half(const u32x8& p, int j) {
  return __builtin_bit_cast(bf16x8, j ? __builtin_shufflevector(p, p, 4, 5, 6, 7) : __builtin_shufflevector(p, p, 0, 1, 2, 3));
}

// Per-wave softmax state and accumulators; a wave owns NQ query tiles of 16 rows.
template <int NQ>
struct WaveState {
  bf16x8 qf[NQ][2];      // Q^T fragments, 32 channels each
  f32x4 o_acc[4][NQ];    // O^T accumulators, [16 channels][query tile]
  f32x4 s_cur[2][NQ];    // raw scores of the current step, [16 keys][query tile]
  u32x8 p_old[NQ / 2];   // bf16 P^T of the previous step, two query tiles each: two 16x16x32 B operands, one 16x16x64 one
  float nm[NQ];          // minus the shift m, in log2 units
  float c;               // factor from raw scores to log2 units (kernel with per-row shifts only)
  f32x4 l_acc[NQ / 2];   // row sums, from the matrix cores: see row_sum_operand()
  bf16x8 ones_a;         // A operand and index operand of the row sums
  int ones_idx;
};

// A constant in a register of its own, here and now: the compiler moves constants that an instruction cannot hold
// in front of the loop over a share's segments, where they take registers through the whole tile.
__device__ __forceinline__ uint32_t local(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Row sums on the matrix cores.  A sum does not need the zeros of a structured-sparse A
// operand: v_smfmac_f32_16x16x64_bf16 takes 64 dense k per instruction in the time the dense
// 16x16x32 takes 32 (18 against 16 cycles in a register-only loop), and the two k of every four that a row
// of A drops are taken by another row.  Its B operand are the eight P^T registers of two query tiles
// (query l%16 of both): the first tile's values are the k below 32 and the second one's the others,
// which are multiplied by lanes 0..31 and lanes 32..63 of A.  So rows 0 and 4 of A hold ones in lanes below
// 32 and rows 8 and 12 in the others; rows 0 and 8 keep the k 0, 1 of every four (index 0x4), rows 4 and 12
// the k 2, 3 (0xE).  D[0][n] + D[4][n] is the sum of query n of the first tile, D[8][n] + D[12][n] that of
// the second: register 0 of the four lane groups (row_sums()), so that one comparison per pair looks at
// every row.  A step's 32 products take 512 matrix-core cycles; its
// row sums take 36 instead of the 64 of four dense 16x16x32.  Stage 3 is bound by those cycles and the
// power they draw: 16 heads x 16384 x 16384 878 -> 860 us.
__device__ __forceinline__ bf16x8 row_sum_operand(int lane) {
  const int m = lane & 15;
  const uint32_t w = (m & 3) == 0 && (m >> 3) == (lane >> 5) ? local(0x3F803F80u) : 0u;
  return __builtin_bit_cast(bf16x8, u32x4{w, w, w, w});
}
__device__ __forceinline__ int row_sum_index(int lane) { return (int)((lane & 4) ? local(0xEEEEEEEEu) : local(0x44444444u)); }
// Exchange between neighbouring lane groups of 16 (halves of the wave): both lanes of a pair receive {x of the lower
// one, x of the upper one}.
struct LanePair {
  float a, b;
};
__device__ __forceinline__ LanePair swap16(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t lo = r[0], hi = r[1];
  return {__uint_as_float(lo), __uint_as_float(hi)};
}
__device__ __forceinline__ LanePair swap32(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t lo = r[0], hi = r[1];
  return {__uint_as_float(lo), __uint_as_float(hi)};
}
// The sums of query column l16 of a pair's two query tiles from its register 0, in all lanes.
__device__ __forceinline__ LanePair row_sums(float l0) {
  const LanePair h = swap16(l0);
  return swap32(h.a + h.b);
}

// exp2(s*c - m) (SHIFT) or exp2(s) of a step's 8 scores of one query column, packed to bf16: one half of
// a pair's P^T operand.
template <bool SHIFT>
__device__ __forceinline__ void exp_pack(const f32x4& s0, const f32x4& s1, float c, float nm, u32x8& p, int half) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const f32x4& s = e < 2 ? s0 : s1;
    const float x0 = s[2 * (e & 1)], x1 = s[2 * (e & 1) + 1];
    const float p0 = __builtin_amdgcn_exp2f(SHIFT ? fmaf(x0, c, nm) : x0);
    const float p1 = __builtin_amdgcn_exp2f(SHIFT ? fmaf(x1, c, nm) : x1);
    p[4 * half + e] = pack_bf16x2(p0, p1);
  }
}

// The largest score of a query column among the 32 keys of a step (all four lane groups).
__device__ __forceinline__ float step_max(const f32x4& s0, const f32x4& s1) {
  float t = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])), fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
  LanePair o = swap16(t);
  o = swap32(fmaxf(o.a, o.b));
  return fmaxf(o.a, o.b);
}

// Sums of weights a step may leave behind (of the keys one lane group adds up); beyond it the shift is raised, in
// rows with a score 55 above it or with a sum before the step beyond kGuardGrown (one of which holds then).
constexpr float kGuardSum = 1.152921504606846976e18f;    // 2^60
constexpr float kGuardGrown = 2.88230376151711744e17f;   // 2^58
constexpr float kLowestScore = -3.402823466e38f;         // no finite score is below: the shift of sums without a key

template <int NQ>
__device__ __forceinline__ void add_row_sums(WaveState<NQ>& w, const u32x8& p, int i) {
  w.l_acc[i] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(w.ones_a, __builtin_bit_cast(bf16x16, p), w.l_acc[i], w.ones_idx, 0, 0);
}

// MFMA A operands of one step: 4 K fragments (16 key rows x 32 channels, [key tile * 2 + channel half]) and
// 4 V^T fragments (16 channels x 32 key positions), 16 bytes per lane each.
struct StepOperands {
  bf16x8 ak[4];
  bf16x8 av[4];
};

// K tile in LDS: 64 rows of 128 bytes, unpadded (it is written by global->LDS loads, 1 KB per
// wave instruction); the 16-byte chunk c of row r sits at chunk position c ^ ((r >> 1) & 7), which
// makes the operand reads of 16 consecutive rows hit 16 distinct bank groups.
__device__ __forceinline__ int k_swizzle(int row) { return (row >> 1) & 7; }

// `sk` points at the first of the 32 rows of this step (row 0 or 32 of the tile).
__device__ __forceinline__ void load_k_operands(StepOperands& op, const bf16_t* sk, int l16, int grp) {
  const int sw = k_swizzle(l16);
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      op.ak[kt * 2 + ks] = *(const bf16x8*)(sk + (kt * 16 + l16) * kDHead + ((ks * 4 + grp) ^ sw) * 8);
}
// A operands of O^T += V^T P^T from the row-major V tile: ds_read_b64_tr_b16 hands lane 4a+e of a
// 16-lane group element e of the 8 bytes that lane 4r+a of the group addressed, as its r-th value.
// Lane 4r+a addresses key k0+r, channels c0+4a..c0+4a+3, so lane i receives keys k0..k0+3 of channel
// c0+i - four consecutive keys of one V^T row.  Two reads (k0 = 4*grp and 16 keys further) give the 8 keys
// a lane's P^T registers hold.
// `sv` points at the first of the 32 key rows of this step.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void load_v_operands(StepOperands& op, const bf16_t* sv, int l16, int grp) {
  const int krow = 4 * grp + (l16 >> 2);
  const int sw = v_swizzle(krow);
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    const bf16_t* base = sv + krow * kDHead + ((2 * ct + ((l16 & 3) >> 1)) ^ sw) * 8 + 4 * (l16 & 1);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)base);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base + 16 * kDHead));
    op.av[ct] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Waves of 128 rows (NQ = 8) hold their accumulators in accumulation registers.  The compiler decides between the two
// register files once for all products of a kernel, and the scores are read by vector instructions, so these products are
// written out.  The compiler keeps no wait states around an asm statement: two between a vector instruction that writes an
// operand and the product, and what the product takes before its result is touched.  accumulators_settled() in front of the
// first product and behind the last one holds the latter where the accumulators are set and read; inside the loop only
// products touch them (one that adds to the register of an earlier one needs no wait), and the operands are written long
// before, by LDS reads, which are waited for, and by the step before.  That it came out so, without spills and copies in
// between, is checked in the assembly by every build, which fails otherwise (isa_check.py).
template <int NQ>
__device__ __forceinline__ void mfma_o(f32x4& o, const bf16x8& a, const bf16x8& b) {
  if constexpr (NQ == 8)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
  else
    o = mfma16(a, b, o);
}
template <int NQ>
__device__ __forceinline__ void accumulators_settled(WaveState<NQ>& w) {
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt)
    asm volatile("s_nop 15\n\ts_nop 3" : "+a"(w.o_acc[0][qt]), "+a"(w.o_acc[1][qt]), "+a"(w.o_acc[2][qt]), "+a"(w.o_acc[3][qt]));
}

// Per-row shifts: the weights of a step are added to the row sums before they are multiplied with V, and a step that
// brings a sum beyond kGuardSum (or to inf or NaN) is taken back here; `before` are the sums without it.  A row
// with a score far above its shift takes that score for the shift, one whose sum has grown over many keys moves
// it by 58; sums and accumulators follow, and the weights are taken again, from scores computed again with
// the 32 rows of K at `kv_first` in memory: held to the end of the step they need 32 registers too many (100 to
// 400 spilled).  One comparison per pair of query tiles and step.  Sums and guard on the vector ALU / no guard, where a
// row that leaves the range costs its tile 1.8 more passes / this: 16 ragged heads of 5500 x 9000 keys 217 / 198 / 206 us;
// 9000 x 9000 with the last key 60 nats above the rest 308 / 771 / 288.
template <int NQ>
__device__ __forceinline__ void guard_step(WaveState<NQ>& w, u32x8 (&p)[NQ / 2], const float (&before)[NQ / 2], const char* kg,
                                           int kv_first, int Mk, int lane) {
  bool out = false;
#pragma unroll
  for (int i = 0; i < NQ / 2; ++i) out = out || !(w.l_acc[i][0] <= kGuardSum);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(out) == 0, 1)) return;
  asm volatile("" : "+v"(lane));      // (nothing of the addresses below is to live in registers outside)
  const float masked = __uint_as_float(local(0xFF800000u));   // -inf
  const int l16 = lane & 15, grp = lane >> 4;
  bf16x8 ak[4];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int row = kv_first + kt * 16 + l16;
      ak[kt * 2 + ks] = *(const bf16x8*)(kg + (uint32_t)((row < Mk ? row : Mk - 1) * kRowBytes + (ks * 4 + grp) * 16));
    }
#pragma unroll
  for (int i = 0; i < NQ / 2; ++i) {
    float sc[2];
    const LanePair sum = row_sums(before[i]);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int qt = 2 * i + j;
      f32x4 s[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        s[kt] = mfma16(ak[kt * 2], w.qf[qt][0], f32x4{0.f, 0.f, 0.f, 0.f});
        s[kt] = mfma16(ak[kt * 2 + 1], w.qf[qt][1], s[kt]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kv_first + 16 * kt + 4 * grp + r >= Mk) s[kt][r] = masked;
      }
      const float top = step_max(s[0], s[1]);
      const float grown = (j ? sum.b : sum.a) > kGuardGrown ? 58.f : 0.f;
      const float nm = fmaf(top, w.c, w.nm[qt]) > 55.f ? -(top * w.c) : w.nm[qt] - grown;
      sc[j] = __builtin_amdgcn_exp2f(nm - w.nm[qt]);
      w.nm[qt] = nm;
      // (as a vector: from single elements the compiler builds the accumulators anew, in other registers)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) w.o_acc[ct][qt] = w.o_acc[ct][qt] * f32x4{sc[j], sc[j], sc[j], sc[j]};
      exp_pack<true>(s[0], s[1], w.c, w.nm[qt], p[i], j);
      __builtin_amdgcn_sched_barrier(0);
    }
    w.l_acc[i] = f32x4{before[i] * (grp >= 2 ? sc[1] : sc[0]), 0.f, 0.f, 0.f};
    add_row_sums(w, p[i], i);
  }
}

// One pipeline step of a wave outside the steady state (first tile, last tile, drain); the order of
// issue is the compiler's.
//   DO_QK : scores of the NEXT step from the 32 K rows at `sk`           -> becomes s_cur
//   DO_PV : O^T += V^T P^T of the PREVIOUS step, V rows at `svt`
//   DO_SM : softmax of the CURRENT step (s_cur -> p_old); its first key is `kv_first` (row of `kg`, K in memory)
//   MASK  : keys >= Mk get weight 0;  FIRST : this is step 0 and fixes m
template <int NQ, bool SHIFT, bool DO_QK, bool DO_PV, bool DO_SM, bool MASK, bool FIRST>
__device__ __forceinline__ void pipeline_step(WaveState<NQ>& w, const bf16_t* sk, const bf16_t* svt, const char* kg,
                                              int kv_first, int Mk, int lane) {
  const int l16 = lane & 15, grp = lane >> 4;
  StepOperands op;
  f32x4 s_next[2][NQ];
  if (DO_QK) {
    load_k_operands(op, sk, l16, grp);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt)
          s_next[kt][qt] = mfma16(op.ak[kt * 2 + ks], w.qf[qt][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s_next[kt][qt]);
  }
  // (waves of 128 rows have no registers for two of a step's three parts side by side)
  if (NQ == 8) __builtin_amdgcn_sched_barrier(0);
  if (DO_PV) {
    load_v_operands(op, svt, l16, grp);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt)
        mfma_o<NQ>(w.o_acc[ct][qt], op.av[ct], p_half(w.p_old[qt >> 1], qt & 1));
    if (!SHIFT) {
#pragma unroll
      for (int i = 0; i < NQ / 2; ++i) add_row_sums(w, w.p_old[i], i);
    }
  }
  // (per-row shifts: products and softmax side by side need 4 to 6 registers too many)
  if ((SHIFT || NQ == 8) && DO_QK && DO_PV) __builtin_amdgcn_sched_barrier(0);
  if (DO_SM) {
    // s_cur[kt][qt][r]: key kv_first + 16*kt + 4*grp + r, query column l16 of tile qt
    if (MASK) {
      const float masked = __uint_as_float(local(0xFF800000u));   // -inf
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int kv = kv_first + 16 * kt + 4 * grp + r;
          if (kv >= Mk) {
#pragma unroll
            for (int qt = 0; qt < NQ; ++qt) w.s_cur[kt][qt][r] = masked;
          }
        }
    }
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      if (SHIFT && FIRST) w.nm[qt] = -fmaxf(step_max(w.s_cur[0][qt], w.s_cur[1][qt]) * w.c, kLowestScore);
      exp_pack<SHIFT>(w.s_cur[0][qt], w.s_cur[1][qt], w.c, w.nm[qt], w.p_old[qt >> 1], qt & 1);
    }
    if (SHIFT) {
      float before[NQ / 2];
#pragma unroll
      for (int i = 0; i < NQ / 2; ++i) {
        before[i] = w.l_acc[i][0];
        add_row_sums(w, w.p_old[i], i);
      }
      guard_step(w, w.p_old, before, kg, kv_first, Mk, lane);
    }
  }
  if (DO_QK) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) w.s_cur[kt][qt] = s_next[kt][qt];
  }
}

// The steady-state step with the order of issue written out: one MFMA, then its
// share of the softmax of the current step (an exp2, and behind every second one the bf16 pack of the pair
// before), fenced so that the compiler keeps the interleave.  PV of step t-1 first (the V operands
// retire, their successors are requested), then QK^T of step t+1 and the K operands; a row-sum MFMA after
// every sixteenth product.  Neighbouring products share one operand (the query tiles run forth
// and back): the sources that toggle cost power, and the clock follows it.  `between` runs after the
// step's last LDS read: the global->LDS requests of the iteration go there, because the compiler makes
// every LDS read wait for all requests issued before it in program order.
template <int NQ, bool SHIFT, bool PREFETCH, typename Between>
__device__ __forceinline__ void steady_step(WaveState<NQ>& w, StepOperands& op, const bf16_t* sk_next,
                                            const bf16_t* sv_next, const char* kg, int kv_first, int Mk, int lane,
                                            Between between) {
  const int l16 = lane & 15, grp = lane >> 4;
  // 8 * NQ groups: 4 * NQ products of each kind, every group with one of the 8 * NQ scores of the lane
  constexpr int NG = 8 * NQ;
  f32x4 s_next[2][NQ];
  float ex[8 * NQ];
  u32x8 p_new[NQ / 2];
  auto soft = [&](int g) {   // value g of the scores of this lane: query tile g / 8, key register g % 8
    // (the empty asm after a result only pins where the instruction is issued)
    const int qt = g >> 3;
    const float x = w.s_cur[(g >> 2) & 1][qt][g & 3];
    ex[g] = __builtin_amdgcn_exp2f(SHIFT ? fmaf(x, w.c, w.nm[qt]) : x);
    asm volatile("" : "+v"(ex[g]));
  };
  auto pack = [&](int p) {   // values 2p, 2p + 1
    uint32_t r = pack_bf16x2(ex[2 * p], ex[2 * p + 1]);
    asm volatile("" : "+v"(r));
    p_new[p >> 3][p & 7] = r;
  };
  float before[NQ / 2];
  auto sums = [&](int i) {   // per-row shifts: the new weights of a pair, complete now
    before[i] = w.l_acc[i][0];
    asm volatile("" : "+v"(before[i]));      // (this register, not a copy of all four)
    add_row_sums(w, p_new[i], i);
  };
  auto group_end = [&](int g) {
    soft(g);
    if (g >= 2 && (g & 1) == 0) pack((g >> 1) - 1);
    if (!SHIFT && (g & 15) == 7) add_row_sums(w, w.p_old[g >> 4], g >> 4);
    if (SHIFT && g >= 16 && (g & 15) == 0) sums(g / 16 - 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // PV of step t-1 first: the V operands retire and their successors are requested ...
#pragma unroll
  for (int g = 0; g < NG / 2; ++g) {
    const int ct = g / NQ, qt = ct & 1 ? NQ - 1 - g % NQ : g % NQ;
    w.o_acc[ct][qt] = mfma16(op.av[ct], p_half(w.p_old[qt >> 1], qt & 1), w.o_acc[ct][qt]);
    group_end(g);
  }
  if (PREFETCH) {
    load_v_operands(op, sv_next, l16, grp);
    __builtin_amdgcn_sched_barrier(0);
  }
  // ... then QK^T of step t+1
#pragma unroll
  for (int g = NG / 2; g < NG; ++g) {
    const int i = g - NG / 2, ks = i / (2 * NQ), kt = (i / NQ) & 1, qt = kt ? NQ - 1 - i % NQ : i % NQ;
    s_next[kt][qt] = mfma16(op.ak[kt * 2 + ks], w.qf[qt][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s_next[kt][qt]);
    group_end(g);
  }
  pack(NG / 2 - 1);
  if (SHIFT) {
    sums(NQ / 2 - 1);
    guard_step(w, p_new, before, kg, kv_first, Mk, lane);
  }
  if (PREFETCH) load_k_operands(op, sk_next, l16, grp);
  __builtin_amdgcn_sched_barrier(0);
  between();        // requests that must follow the step's last LDS read in program order
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    w.s_cur[0][qt] = s_next[0][qt];
    w.s_cur[1][qt] = s_next[1][qt];
  }
#pragma unroll
  for (int i = 0; i < NQ / 2; ++i) w.p_old[i] = p_new[i];
}

// The steady-state step of a wave of 128 rows (log2 keys): steady_step()'s order of issue, with the LDS reads between the
// products as well - its K operands among the products with V, the next step's V operands among its products with K.
// One wave per SIMD has nothing to issue while a burst of reads waits for its turn at the LDS.  `middle` runs between the two
// kinds of products, `fill(g)` in the groups of the first kind.
template <typename Middle, typename Fill>
__device__ __forceinline__ void wide_step(WaveState<8>& w, StepOperands& op, const bf16_t* sk, const bf16_t* sv_next, int lane, Middle middle, Fill fill) {
  constexpr int NQ = 8, NG = 8 * NQ;
  const int l16 = lane & 15, grp = lane >> 4;
  f32x4 s_next[2][NQ];
  float ex[NG];
  u32x8 p_new[NQ / 2];
  s16x4 v_part[2];
  auto pack = [&](int p) {   // values 2p, 2p + 1
    uint32_t r = pack_bf16x2(ex[2 * p], ex[2 * p + 1]);
    asm volatile("" : "+v"(r));
    p_new[p >> 3][p & 7] = r;
  };
  auto group_end = [&](int g) {
    ex[g] = __builtin_amdgcn_exp2f(w.s_cur[(g >> 2) & 1][g >> 3][g & 3]);
    asm volatile("" : "+v"(ex[g]));
    if (g >= 2 && (g & 1) == 0) pack((g >> 1) - 1);
    if ((g & 15) == 7) add_row_sums(w, w.p_old[g >> 4], g >> 4);
    __builtin_amdgcn_sched_barrier(0);
  };
  const int ksw = k_swizzle(l16), krow = 4 * grp + (l16 >> 2), vsw = v_swizzle(krow);
#pragma unroll
  for (int g = 0; g < NG / 2; ++g) {
    const int ct = g / NQ, qt = ct & 1 ? NQ - 1 - g % NQ : g % NQ;
    mfma_o<NQ>(w.o_acc[ct][qt], op.av[ct], p_half(w.p_old[qt >> 1], qt & 1));
    if (g % 4 == 1 && g / 4 < 4) {
      const int i = g / 4;
      op.ak[i] = *(const bf16x8*)(sk + ((i >> 1) * 16 + l16) * kDHead + (((i & 1) * 4 + grp) ^ ksw) * 8);
    }
    fill(g);
    group_end(g);
  }
  middle();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int g = NG / 2; g < NG; ++g) {
    const int i = g - NG / 2, ks = i / (2 * NQ), kt = (i / NQ) & 1, qt = kt ? NQ - 1 - i % NQ : i % NQ;
    s_next[kt][qt] = mfma16(op.ak[kt * 2 + ks], w.qf[qt][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s_next[kt][qt]);
    if (i % 3 == 1 && i < 24) {
      const int ct = i / 6, half = i / 3 & 1;
      const bf16_t* p = sv_next + (krow + 16 * half) * kDHead + ((2 * ct + ((l16 & 3) >> 1)) ^ vsw) * 8 + 4 * (l16 & 1);
      v_part[half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
      if (half) op.av[ct] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v_part[0], v_part[1], 0, 1, 2, 3, 4, 5, 6, 7));
    }
    group_end(g);
  }
  pack(NG / 2 - 1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    w.s_cur[0][qt] = s_next[0][qt];
    w.s_cur[1][qt] = s_next[1][qt];
  }
#pragma unroll
  for (int i = 0; i < NQ / 2; ++i) w.p_old[i] = p_new[i];
}

// Row sums the pipelined pass accepts (inf and NaN fail the test as well): inside, the weights of a
// row's best keys are far from both ends of the fp32 range, and no weight exceeds 2^64, so that the
// unnormalised products with V stay finite for |v| below 1e19.
constexpr float kFastSumMin = 5.421010862427522e-20f;    // 2^-64
constexpr float kFastSumMax = 1.8446744073709552e19f;    // 2^64

// One step of 32 keys with a running maximum per row (the classic online softmax), for tiles with
// rows that no pipelined pass holds: any finite scores.  Not pipelined: rare.  The maxima are kept in
// units of the raw scores: near the ends of the fp32 range the rounding of max * c alone is more than
// the exponents can hold, s - max of neighbouring scores is exact.
template <int NQ>
__device__ __forceinline__ void running_max_step(WaveState<NQ>& w, float (&l)[NQ], float (&top)[NQ], const bf16_t* sk,
                                                 const bf16_t* sv, int kv_first, int Mk, int l16, int grp) {
  const bf16x2 ones2 = {(bf16_t)1.0f, (bf16_t)1.0f};
  StepOperands op;
  load_k_operands(op, sk, l16, grp);
  load_v_operands(op, sv, l16, grp);
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    f32x4 s[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      s[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) s[kt] = mfma16(op.ak[kt * 2 + ks], w.qf[qt][ks], s[kt]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (kv_first + 16 * kt + 4 * grp + r >= Mk) s[kt][r] = -INFINITY;
    }
    const float m = fmaxf(top[qt], step_max(s[0], s[1]));
    const float sc = __builtin_amdgcn_exp2f((top[qt] - m) * w.c);
    top[qt] = m;
    u32x8 p = {};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x4& x = s[e >> 1];
      const int i = 2 * (e & 1);
      p[e] = pack_bf16x2(__builtin_amdgcn_exp2f((x[i] - m) * w.c), __builtin_amdgcn_exp2f((x[i + 1] - m) * w.c));
    }
    l[qt] *= sc;
#pragma unroll
    for (int e = 0; e < 4; ++e) l[qt] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)p[e]), ones2, l[qt], false);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
#pragma unroll
      for (int r = 0; r < 4; ++r) w.o_acc[ct][qt][r] *= sc;
      w.o_acc[ct][qt] = mfma16(op.av[ct], p_half(p, 0), w.o_acc[ct][qt]);
    }
  }
}

// ---- stage 4 at the end of a query tile ------------------------------------------------------------
// (paper Sec. 3.2 Eq. 5-7 and the inverse reorder of Sec. 3.3, with the heads concatenated.)  The tile's
// normalised rows lie in LDS; its tokens are found by looking at the clusters of the tokens of its merging blocks,
// 64 per wave instruction, the ones that belong here moved to the front of the wave so that 8 lanes then copy
// a row each to out[pi(j)][h].  A kernel of its own for this is bound by writing `out`; here the writes go out
// under the products of the other workgroups, the rows are not read back and a launch is saved.  What is left
// of it at the end of a launch is one tile's chain of round trips (clusters, exchange, stores: 2 to 4 us).  In
// attention_split_reduce_kernel it is 1 to 2 us, 21 where a block keeps a thousand clusters (3840 tokens, which four
// workgroups a tile walk for 64 rows each: 15 -> 36 us, against a stage-4 kernel of 181).
// A layer with the stage-4 kernel behind it / with this: 2 frames of 16 x 16 22.8 / 17.4 us, 8 of 37 x 37 140.6 /
// 135.9, 200 of 37 x 37 2973 / 2918, with outliers 5753 / 5675; every random geometry of 12 was faster.

// 16-byte chunk c of row r of the tile, swizzled: the rows are 128 bytes apart.
__device__ __forceinline__ int out_chunk(int r, int c) { return r * kRowChunks + (c ^ (r & 7)); }

// The target out of the kernel's arguments, read here and now: the compiler would read it in front of the tile and
// hold it in scalar registers that the tile has none left of.
__device__ __forceinline__ UnmergeTarget unmerge_target() {
  typedef const __attribute__((address_space(4))) char* args_t;
  args_t p = (args_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(AttnArgs, um);
  asm volatile("" : "+s"(p));
  return *(const UnmergeTarget*)p;
}
// First row of a tile inside its head (where its clusters count from), likewise read late.
__device__ __forceinline__ int unmerge_row0(const UnmergeTarget& um, int h, int q0) {
  typedef const __attribute__((address_space(4))) char* args_t;
  args_t p = (args_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(AttnArgs, q_off) + h * sizeof(int64_t);
  asm volatile("" : "+s"(p));
  return row_in_head(*(const __attribute__((address_space(4))) int64_t*)p, h, um.M, q0);
}

// A tile's search: kUnmergeBatch tokens per lane are requested together.
constexpr int kUnmergeBatch = 4;
struct UnmergeBatch {
  int32_t row[kUnmergeBatch], token[kUnmergeBatch];   // row < 0: not of this tile
};
struct UnmergeSpan {
  int first, end;
};
__device__ __forceinline__ UnmergeSpan unmerge_span(const UnmergeTarget& um, int row0, int n) {
  return {um.spans[2 * (row0 / kUnmergeGroup)], um.spans[2 * ((row0 + n - 1) / kUnmergeGroup) + 1]};
}
template <int NT>
__device__ __forceinline__ void unmerge_load(UnmergeBatch& b, const UnmergeTarget& um, int h, int row0, int n, int first, int end, int tid) {
#pragma unroll
  for (int u = 0; u < kUnmergeBatch; ++u) {
    const int j = first + u * NT + tid, jc = j < end ? j : end - 1;
    const int r = um.assign[h * um.N + jc] - row0;
    b.token[u] = um.pi[jc];
    b.row[u] = j < end && r >= 0 && r < n ? r : -1;
  }
}
// Rows [row0, row0 + n) of head h, in LDS at `rows`, to their tokens; `b` holds the first batch.  NT threads.
template <int NT>
__device__ __forceinline__ void unmerge_store(UnmergeBatch& b, const UnmergeTarget& um, const u32x4* rows, int h, int row0, int n,
                                              UnmergeSpan sp, int tid) {
  const int lane = tid & 63, sub = lane >> 3, c = lane & 7;
  u32x4* __restrict__ out = (u32x4*)um.out;
  for (int first = sp.first; first < sp.end; first += NT * kUnmergeBatch) {
    UnmergeBatch cur = b;
    if (first + NT * kUnmergeBatch < sp.end) unmerge_load<NT>(b, um, h, row0, n, first + NT * kUnmergeBatch, sp.end, tid);
#pragma unroll
    for (int u = 0; u < kUnmergeBatch; ++u) {
      const unsigned long long hit = __builtin_amdgcn_ballot_w64(cur.row[u] >= 0);
      if (!hit) continue;
      const int cnt = __popcll(hit);
      const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(hit >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit, 0u));
      const int to = 4 * (cur.row[u] >= 0 ? before : cnt + lane - before);      // (every lane has a place of its own)
      const int r = __builtin_amdgcn_ds_permute(to, cur.row[u] >= 0 ? cur.row[u] : 0), t = __builtin_amdgcn_ds_permute(to, cur.token[u]);
      // (four rows a lane at a time: one after the other, each waits for two exchanges and an LDS read)
      for (int i = sub; i - sub < cnt; i += 32) {
        int ri[4], ti[4];
        u32x4 x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          ri[k] = __builtin_amdgcn_ds_bpermute(4 * (i + 8 * k), r);
          ti[k] = __builtin_amdgcn_ds_bpermute(4 * (i + 8 * k), t);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = rows[out_chunk(ri[k], c)];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i + 8 * k < cnt) __builtin_nontemporal_store(x[k], &out[((int64_t)ti[k] * um.H + h) * kRowChunks + c]);
      }
    }
  }
}

// What is left of a whole tile whose rows lie in LDS: they go to `o_rows`, and to their tokens.
template <int NT, int BQ>
__device__ __forceinline__ void unmerge_tile(const UnmergeTarget& um, UnmergeBatch& batch, const u32x4* rows,
                                             u32x4* __restrict__ o_rows, int h, int q0, int n, int64_t q_base, bool dev_tile, UnmergeSpan span, int tid) {
#pragma unroll
  for (int i = 0; i < BQ * kRowChunks / NT; ++i) {
    const int r = (tid >> 3) + i * (NT / 8), c = tid & 7;
    if (r >= n) continue;
    const u32x4 x = rows[out_chunk(r, c)];
    o_rows[(q_base + q0 + r) * kRowChunks + c] = x;
    if (dev_tile) {
      // an outlier query: the one token it belongs to
      const int64_t token = um.q2_token[q_base + q0 + r];
      __builtin_nontemporal_store(x, (u32x4*)um.out + (token * um.H + h) * kRowChunks + c);
    }
  }
  if (!dev_tile) unmerge_store<NT>(batch, um, rows, h, unmerge_row0(um, h, q0), n, span, tid);
}

// 8 KB tiles of LDS of a workgroup: per key group two of K and two of V, and with several key groups room
// for everybody's accumulators in their place.
template <int NQ, int NW, int KS>
constexpr int lds_tiles() {
  const int acc = KS > 1 ? NQ * NW * 4 * 64 * 16 / (kKvTile * kDHead * 2) : 0;
  return KS * 4 > acc ? KS * 4 : acc;
}

// One query tile (or one segment of it) of a workgroup: see attention_kernel.
//   h, q0          : head and first query row of the tile
//   dev_tile       : the tile comes from the device-side list (rows q_base_dev .. + mq_dev of q2 / o2)
//   seg.slot >= 0  : only the key tiles [seg.t0, seg.t1) of the head, results into scratch slot seg.slot
//   KS > 1         : the waves form KS groups that take a KS-th of the keys each, for the same rows; every
//                    group has tile buffers of its own, and the groups' results meet in LDS at the end
template <int NQ, int NW, int KS, bool SHIFT>
__device__ __forceinline__ void attention_tile(const AttnArgs& a, bf16_t (*lds)[kKvTile * kDHead], const int h,
                                               const int q0, const bool dev_tile, const int64_t q_base_dev,
                                               const int mq_dev, const SplitSegment seg) {
  constexpr int NT = 64 * NW;
  constexpr int RG = NW / KS;                              // waves of a key group
  constexpr int BQ = 16 * NQ * RG;
  constexpr int LDK = 8 / RG;                              // 1 KB global->LDS loads per wave per tile
  const bool piece = seg.slot >= 0;
  const int64_t q_base = dev_tile ? q_base_dev : a.q_off[h];
  int64_t k_base = a.k_off[h];
  const int Mq = dev_tile ? mq_dev : a.q_rows[h];
  const bf16_t* __restrict__ q_rows = dev_tile ? a.q2 : a.q;
  bf16_t* __restrict__ o_rows = dev_tile ? a.o2 : a.o;
  int Mk = (int)(a.k_off[h + 1] - k_base);

  // (the empty asm keeps per-lane values that derive from the thread index from being computed once
  // in front of the loop over a share's segments and held in registers across the whole tile)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  // a segment sees its key tiles as the whole key sequence
  const int64_t piece_row0 = (int64_t)(piece ? seg.slot : 0) * BQ;
  if (piece) {
    k_base += (int64_t)seg.t0 * kKvTile;
    Mk = (seg.t1 * kKvTile < Mk ? seg.t1 * kKvTile : Mk) - seg.t0 * kKvTile;
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS destinations stay scalar
  const int key_group = KS == 1 ? 0 : wave / RG, rwave = KS == 1 ? wave : wave % RG;
  bf16_t (*s_k)[kKvTile * kDHead] = lds + key_group * 4;       // two tiles of K, two of V
  bf16_t (*s_v)[kKvTile * kDHead] = s_k + 2;
  const int l16 = lane & 15, grp = lane >> 4;
  const int wq0 = q0 + rwave * 16 * NQ;  // first query row of this wave
  // A wave of a partial tile that owns no valid row only helps to stage K/V and to keep the
  // barriers; it issues no MFMA and no softmax.
  const bool active = __builtin_amdgcn_readfirstlane((int)(wq0 < Mq)) != 0;   // wave-uniform, and known to be

  if (Mk == 0) {
    // softmax over an empty key set: defined as zero output
    const uint32_t zero = local(0);
    for (int e = tid; e < BQ * kRowChunks; e += NT) {
      const int row = q0 + (e >> 3);
      if (row < Mq) ((u32x4*)o_rows)[(q_base + row) * kRowChunks + (e & 7)] = u32x4{zero, zero, zero, zero};
    }
    return;
  }

  int max_tiles = 0;                              // of any key group (KS > 1)
  __shared__ int s_again, s_high;                 // a wave has rows out of range, above it
  __shared__ float s_sum[KS == 1 ? 1 : NW][NQ * 16], s_shift[KS == 1 ? 1 : NW][NQ * 16];
  const int all = (Mk + kKvTile - 1) / kKvTile;
  auto key_tiles = [&](int g) { return (g * all + KS - 1) / KS; };      // of the groups before group g
  if constexpr (KS > 1) {
    const int t0 = key_tiles(key_group), t1 = key_tiles(key_group + 1);   // (never none for the first)
    max_tiles = (all + KS - 1) / KS;
    k_base += (int64_t)t0 * kKvTile;
    Mk = (t1 * kKvTile < Mk ? t1 * kKvTile : Mk) - t0 * kKvTile;   // at most 0 for a group without a key tile
  }

  WaveState<NQ> w;
  // ---- Q^T fragments (B operand): lane -> query column, 8 consecutive channels ---------------
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    int row = wq0 + qt * 16 + l16;
    row = row < Mq ? row : Mq - 1;
    const bf16_t* p = q_rows + (q_base + row) * kDHead + grp * 8;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) w.qf[qt][ks] = *(const bf16x8*)(p + ks * 32);
    w.nm[qt] = 0.f;
    w.l_acc[qt >> 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) w.o_acc[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- K/V tile staging: global -> registers -> LDS ---------------------------------------------
  const char* kg = (const char*)(a.k + k_base * kDHead);   // wave-uniform bases; per-lane offsets
  const char* vg = (const char*)(a.v + k_base * kDHead);   // below fit 32 bits (rows < 2^24 here)
  // K: straight from global memory into LDS, no registers.  Lane l of a wave instruction fills
  // bytes [16 l, 16 l + 16) of a 1 KB block = rows 8*blk .. 8*blk+7; it fetches the chunk that
  // belongs at its position under the swizzle.
  auto load_rows = [&](const char* rows, int kv0, int n, bf16_t* buf, bool inside = false) {   // inside: the whole tile lies below n
#pragma unroll
    for (int i = 0; i < LDK; ++i) {
      const int blk = rwave * LDK + i;
      const int r = blk * 8 + (lane >> 3);
      const int c = (lane & 7) ^ k_swizzle(r);
      int row = kv0 + r;
      if (!inside) row = row < n ? row : n - 1;
      const char* src = rows + (uint32_t)(row * kRowBytes + c * 16);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)(buf + blk * 512), 16, 0, 0);
    }
  };
  auto load_k = [&](int kv0, int buf, bool inside = false) { load_rows(kg, kv0, Mk, s_k[buf], inside); };
  // V the same way, under its own swizzle
  auto load_v = [&](int kv0, int buf, bool inside = false) {
#pragma unroll
    for (int i = 0; i < LDK; ++i) {
      const int blk = rwave * LDK + i;
      const int r = blk * 8 + (lane >> 3);
      const int c = (lane & 7) ^ v_swizzle(r);
      int row = kv0 + r;
      if (!inside) row = row < Mk ? row : Mk - 1;
      const char* src = vg + (uint32_t)(row * kRowBytes + c * 16);
      bf16_t* dst = &s_v[buf][blk * 512];
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    }
  };

  w.c = a.scale_log2;
  w.ones_a = row_sum_operand(lane);
  w.ones_idx = row_sum_index(lane);
  const int n_tiles = (Mk + kKvTile - 1) / kKvTile;

  // Whether the keys outside this piece alone bring the sums of all rows into the range (no shifts): then this
  // piece's own sum may be as small as it is.  Looks at the head's first, middle and last key tile.
  auto rest_holds = [&]() -> bool {
    const int64_t k0 = a.k_off[h];
    const int keys = (int)(a.k_off[h + 1] - k0), last = (keys - 1) / kKvTile;
    float rest[NQ];
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) rest[qt] = 0.f;
#pragma unroll 1
    for (int i = 0; i < 3; ++i) {
      const int kv0 = (i * last / 2) * kKvTile;
      load_rows((const char*)(a.k + k0 * kDHead), kv0, keys, s_k[0]);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      if (active) {
#pragma unroll 1
        for (int st = 0; st < kKvTile; st += kStep) {
          StepOperands op;
          load_k_operands(op, &s_k[0][st * kDHead], l16, grp);
#pragma unroll
          for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
              const f32x4 sc = mfma16(op.ak[kt * 2 + 1], w.qf[qt][1], mfma16(op.ak[kt * 2], w.qf[qt][0], f32x4{0.f, 0.f, 0.f, 0.f}));
#pragma unroll
              for (int r = 0; r < 4; ++r)
                rest[qt] += kv0 + st + 16 * kt + 4 * grp + r < keys ? __builtin_amdgcn_exp2f(sc[r]) : 0.f;
            }
        }
      }
      __syncthreads();
    }
    bool low = false;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const LanePair r1 = swap16(rest[qt]), r2 = swap32(r1.a + r1.b);
      low = low || !(r2.a + r2.b >= kFastSumMin);
    }
    if (active && low) s_high = (int)local(1);       // (everybody has read it: two barriers a tile)
    __syncthreads();
    return !s_high;
  };

  // One pass over the keys; true if some row of the tile has left the range of its weights.
  // Steps are numbered t = 0 .. 2*n_tiles-1 (32 keys each).  Outer iteration j runs the pipeline
  // slots t = 2j-1 and t = 2j, which read K tile j (scores of steps 2j, 2j+1) and V tile j-1
  // (products of steps 2j-2, 2j-1), while K tile j+1 and V tile j are on their way into the
  // other LDS buffers.
  float l_tot[NQ];
  auto pass = [&](auto shifts) -> bool {
    constexpr bool S = decltype(shifts)::value;
    if (KS == 1 || n_tiles > 0) {
    // ---- j = 0 ---------------------------------------------------------------------------------------
    load_k(0, 0);
    load_v(0, 0);
    if (n_tiles > 1) load_k(kKvTile, 1);
    if (KS == 1 && tid == 0) s_again = s_high = 0;
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the global->LDS loads have landed
    __syncthreads();
    if (active) {
      pipeline_step<NQ, S, true, false, false, false, false>(w, &s_k[0][0], nullptr, kg, 0, Mk, lane);
    }
    if (active) {
      if (n_tiles > 1)
        pipeline_step<NQ, S, true, false, true, false, true>(w, &s_k[0][kStep * kDHead], nullptr, kg, 0, Mk, lane);
      else
        pipeline_step<NQ, S, true, false, true, true, true>(w, &s_k[0][kStep * kDHead], nullptr, kg, 0, Mk, lane);
    }
    __syncthreads();

    // ---- j = 1 .. n_tiles-2: steady state, no masking ------------------------------------------------
    int j = 1;
    StepOperands op;
    // Two tiles per trip with the buffer indices as constants (j is odd at the top): the LDS
    // addresses become instruction offsets instead of a dozen vector adds per tile.
    auto steady_tile = [&](auto parity, int jt) {
      constexpr int P = decltype(parity)::value;        // jt & 1
      const bf16_t* kb = &s_k[P][0];
      const bf16_t* vb = &s_v[P ^ 1][0];
      auto request = [&]() {
        if ((jt + 2) * kKvTile <= Mk)
          load_k((jt + 1) * kKvTile, P ^ 1, true);
        else
          load_k((jt + 1) * kKvTile, P ^ 1);
        load_v(jt * kKvTile, P, true);                     // jt < n_tiles - 1: a full tile
      };
      // (a wave without valid rows runs the loop below instead: no global->LDS request may precede
      // an LDS read on the path of an active wave, the compiler would wait for it before the read)
      load_k_operands(op, kb, l16, grp);
      load_v_operands(op, vb, l16, grp);
      steady_step<NQ, S, true>(w, op, kb + kStep * kDHead, vb + kStep * kDHead, kg, (2 * jt - 1) * kStep, Mk, lane, request);
      steady_step<NQ, S, false>(w, op, nullptr, nullptr, kg, 2 * jt * kStep, Mk, lane, [] {});
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): K tile jt+1 and V tile jt are in LDS
      __syncthreads();
    };
    if (!active) {
      // a wave of a partial tile without valid rows: it only stages its share of K / V
      for (; j < n_tiles - 1; ++j) {
        load_k((j + 1) * kKvTile, (j + 1) & 1);
        load_v(j * kKvTile, j & 1);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
      }
    } else {
      for (; j + 1 < n_tiles - 1; j += 2) {
        steady_tile(std::integral_constant<int, 1>{}, j);
        steady_tile(std::integral_constant<int, 0>{}, j + 1);
      }
      if (j < n_tiles - 1) {
        steady_tile(std::integral_constant<int, 1>{}, j);
        ++j;
      }
    }

    // ---- j = n_tiles-1 (if it is not j = 0): the last K tile, its first step may be ragged ---------
    if (j == n_tiles - 1) {
      load_v(j * kKvTile, j & 1);
      const bf16_t* kb = &s_k[j & 1][0];
      const bf16_t* vb = &s_v[(j - 1) & 1][0];
      if (active) {
        pipeline_step<NQ, S, true, true, true, false, false>(w, kb, vb, kg, (2 * j - 1) * kStep, Mk, lane);
        pipeline_step<NQ, S, true, true, true, true, false>(w, kb + kStep * kDHead, vb + kStep * kDHead, kg, 2 * j * kStep, Mk, lane);
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the last V tile is in LDS
      __syncthreads();
    }

    // ---- j = n_tiles: drain ---------------------------------------------------------------------------
    if (active) {
      const bf16_t* vb = &s_v[(n_tiles - 1) & 1][0];
      pipeline_step<NQ, S, false, true, true, true, false>(w, nullptr, vb, kg, (2 * n_tiles - 1) * kStep, Mk, lane);
      pipeline_step<NQ, S, false, true, false, false, false>(w, nullptr, vb + kStep * kDHead, kg, 0, Mk, lane);
    }
    }
    // a group of n tiles has met n + 1 barriers (none if it has no tile): the others of its workgroup wait
    if constexpr (KS > 1)
      for (int b = n_tiles ? n_tiles : -1; b < max_tiles; ++b) __syncthreads();

#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const LanePair sums = row_sums(w.l_acc[qt >> 1][0]);
      l_tot[qt] = qt & 1 ? sums.b : sums.a;
      if (KS > 1 && n_tiles == 0) w.nm[qt] = -kLowestScore;      // (no keys, no say in the common shift)
    }
    // Rare: a row of this tile left the range in which its weights are safe; the whole workgroup (it
    // stages its tiles together) takes the tile again.  The range is the row's, not that of
    // a part of its keys: without shifts only the sum of all parts may not be small.
    bool again = false;
    if constexpr (KS == 1) {
      // (one flag and one barrier: __syncthreads_or() takes three, 0.3 us of an 8 us launch)
      bool high = false, low = false;
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        high = high || !(l_tot[qt] <= kFastSumMax);
        low = low || l_tot[qt] < kFastSumMin;
      }
      if (active && (high || low)) s_again = (int)local(1);
      if (active && high) s_high = (int)local(1);
      __syncthreads();
      again = s_again;
      if (!S && again && piece && !s_high) again = !rest_holds();
    } else {
      // every wave looks at the sums of all rows, so that no second barrier is needed to agree
      static_assert(NQ * 16 == 64 || NQ * 16 == 32, "a lane (two) per row of a wave");
      if (grp == 0) {
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) s_sum[wave][qt * 16 + l16] = l_tot[qt];
      }
      __syncthreads();
      bool bad = false;
#pragma unroll
      for (int r = 0; r < RG; ++r) {
        if (q0 + r * 16 * NQ >= Mq) continue;
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          const float part = s_sum[k * RG + r][lane & (NQ * 16 - 1)];
          sum += part;
          // (groups with shifts of their own: each part; one without a key tile has none)
          if (S && key_tiles(k) < key_tiles(k + 1)) bad = bad || !(part >= kFastSumMin && part <= kFastSumMax);
        }
        if (!S) bad = bad || !(sum >= kFastSumMin && sum <= kFastSumMax);
      }
      again = __any(bad);
    }
    return again;
  };
  bool again = pass(std::integral_constant<bool, SHIFT>{});
  // Log2 keys, rare: once more with per-row shifts.  (The barrier: everybody has read the flags of the first pass.)
  if constexpr (!SHIFT) {
    if (again) {
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        w.l_acc[qt >> 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) w.o_acc[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      __syncthreads();
      again = pass(std::integral_constant<bool, true>{});
    }
  }
  if (again) {
    float top[NQ];
    if (active) {
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        top[qt] = kLowestScore;
        l_tot[qt] = 0.f;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) w.o_acc[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    const int end = KS == 1 ? Mk : max_tiles * kKvTile;      // (the groups meet at the same barriers)
#pragma unroll 1
    for (int kv0 = 0; kv0 < end; kv0 += kKvTile) {
      if (KS == 1 || kv0 < Mk) {
        load_k(kv0, 0);
        load_v(kv0, 0);
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      if (active) {
#pragma unroll 1
        for (int st = 0; st < kKvTile && kv0 + st < Mk; st += kStep)
          running_max_step<NQ>(w, l_tot, top, &s_k[0][st * kDHead], &s_v[0][st * kDHead], kv0 + st, Mk, l16, grp);
      }
      __syncthreads();
    }
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const LanePair l1 = swap16(l_tot[qt]), l2 = swap32(l1.a + l1.b);
      l_tot[qt] = l2.a + l2.b;
      if (active) w.nm[qt] = -fmaxf(top[qt] * w.c, kLowestScore);
    }
  }

  if constexpr (KS > 1) {
    // The groups' sums, brought to the largest of their shifts of a row (all zero unless a group had
    // to take shifts or the keys are plain), added in key order.  Every wave leaves its registers in
    // LDS as they are (the tile buffers: no group reads them any more) and adds up its share of the channels.
    f32x4* s_acc = (f32x4*)lds;                     // [wave][channel tile][query tile][lane]
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) s_acc[((wave * 4 + ct) * NQ + qt) * 64 + lane] = w.o_acc[ct][qt];
      if (grp == 0) {
        if (again) s_sum[wave][qt * 16 + l16] = l_tot[qt];
        s_shift[wave][qt * 16 + l16] = -w.nm[qt];
      }
    }
    __syncthreads();
    const UnmergeTarget um = unmerge_target();
    u32x2 o_part[NQ][4 / KS];
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      float wgt[KS], m = kLowestScore, l = 0.f;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        wgt[k] = s_shift[k * RG + rwave][qt * 16 + l16];
        m = fmaxf(m, wgt[k]);
      }
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const float sum = s_sum[k * RG + rwave][qt * 16 + l16];
        wgt[k] = sum == 0.f ? 0.f : __builtin_amdgcn_exp2f(wgt[k] - m);    // (a group without keys: no weight)
        l = fmaf(sum, wgt[k], l);
      }
      const float inv = 1.0f / l;
      const int row = wq0 + qt * 16 + l16;
#pragma unroll
      for (int c = 0; c < 4 / KS; ++c) {
        const int ct = key_group * (4 / KS) + c;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          const f32x4 x = s_acc[(((k * RG + rwave) * 4 + ct) * NQ + qt) * 64 + lane];
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = fmaf(x[r], wgt[k], o[r]);
        }
        o_part[qt][c] = u32x2{pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv)};
        if (row < Mq && !um.out) *(u32x2*)(o_rows + (q_base + row) * kDHead + 16 * ct + 4 * grp) = o_part[qt][c];
      }
    }
    if (um.out) {
      const int n = Mq - q0 < BQ ? Mq - q0 : BQ;
      UnmergeSpan span = {0, 0};
      UnmergeBatch batch;
      if (!dev_tile) {
        const int row0 = unmerge_row0(um, h, q0);
        span = unmerge_span(um, row0, n);
        unmerge_load<NT>(batch, um, h, row0, n, span.first, span.end, tid);
      }
      u32x4* s_rows = (u32x4*)lds;
      __syncthreads();                              // everybody has read the groups' sums
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        const int r = (rwave * NQ + qt) * 16 + l16;
#pragma unroll
        for (int c = 0; c < 4 / KS; ++c)
          *((u32x2*)&s_rows[out_chunk(r, 2 * (key_group * (4 / KS) + c) + (grp >> 1))] + (grp & 1)) = o_part[qt][c];
      }
      __syncthreads();
      unmerge_tile<NT, BQ>(um, batch, s_rows, (u32x4*)o_rows, h, q0, n, q_base, dev_tile, span, tid);
    }
    return;
  }

  if (piece) {
    // a segment: unnormalised sums and the shifts they are relative to, for attention_split_reduce_kernel
    if (active) {
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        const int row = wq0 + qt * 16 + l16;
        if (row < Mq) {
          // slot layout [16 channel groups of 4][BQ rows][4]: group 4 * ct + grp holds the channels
          // 16 * ct + 4 * grp .. + 3, so that the 16 lanes of a group write 256 contiguous bytes and the
          // kernel that adds the segments up reads whole lines
          float* po = a.split_o + piece_row0 * kDHead + (row - q0) * 4;
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) *(f32x4*)(po + (4 * ct + grp) * (BQ * 4)) = w.o_acc[ct][qt];
          if (grp == 0) {
            a.split_l[piece_row0 + (row - q0)] = l_tot[qt];
            a.split_m[piece_row0 + (row - q0)] = -w.nm[qt];
          }
        }
      }
    }
    return;
  }

  // ---- normalise and store ---------------------------------------------------------------------
  const UnmergeTarget um = unmerge_target();
  if (um.out) {
    // stage 4 as well.  (Every wave is through with the tile buffers: the barrier behind the last product.)
    const int n = Mq - q0 < BQ ? Mq - q0 : BQ;
    UnmergeSpan span = {0, 0};
    UnmergeBatch batch;
    if (!dev_tile) {
      const int row0 = unmerge_row0(um, h, q0);
      span = unmerge_span(um, row0, n);
      unmerge_load<NT>(batch, um, h, row0, n, span.first, span.end, tid);
    }
    u32x4* s_rows = (u32x4*)lds;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const float inv = 1.0f / l_tot[qt];
      const int r = (rwave * NQ + qt) * 16 + l16;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
        *((u32x2*)&s_rows[out_chunk(r, 2 * ct + (grp >> 1))] + (grp & 1)) =
            u32x2{pack_bf16x2(w.o_acc[ct][qt][0] * inv, w.o_acc[ct][qt][1] * inv),
                  pack_bf16x2(w.o_acc[ct][qt][2] * inv, w.o_acc[ct][qt][3] * inv)};
    }
    __syncthreads();
    unmerge_tile<NT, BQ>(um, batch, s_rows, (u32x4*)o_rows, h, q0, n, q_base, dev_tile, span, tid);
    return;
  }
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    const float inv = 1.0f / l_tot[qt];
    const int row = wq0 + qt * 16 + l16;
    if (row < Mq) {
      bf16_t* orow = o_rows + (q_base + row) * kDHead;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        u32x2 ow;
        ow[0] = pack_bf16x2(w.o_acc[ct][qt][0] * inv, w.o_acc[ct][qt][1] * inv);
        ow[1] = pack_bf16x2(w.o_acc[ct][qt][2] * inv, w.o_acc[ct][qt][3] * inv);
        *(u32x2*)(orow + 16 * ct + 4 * grp) = ow;
      }
    }
  }
}

// ---- tiles of 512 rows --------------------------------------------------------------------------------
// Long launches with log2 keys: four waves of 128 rows, one workgroup per CU.  What bounds a long launch is power, and an
// operand read from LDS that serves 8 products instead of 4 halves the LDS reads, the requests and the barriers of a
// product.  The accumulators and Q lie in accumulation registers (mfma_o()): 454 registers a lane, so
// there is one wave per SIMD and nothing hides its waits: every operand is read 10 to 30 products before its first use,
// between other products (wide_step()), the next tile's behind a barrier in the middle of the tile's second step, and a
// tile's requests have one and a half tiles until that barrier - three buffers each of K and V, LDS objects of their own, so
// that reads of one do not wait for the requests to another.  Products, their order and the sums of a row are
// those of the 256-row tiles, bit for bit.  16 heads of 24576 rows x 28700 keys: 1.855 GHz with the matrix cores busy 75 % of
// the cycles in 256-row tiles; 16 of 28650 x 28650 here 1.95 to 2.01 GHz and 71 %.  us, 256-row tiles / two buffers and the reads in
// bursts at the ends of a step's halves / two buffers / three: 16 x 16384 x 16384 780 / 775 / 754 / 749, 24576 x 28700 2040 / 2020 /
// 1965 / 1950, 24 x 37477 x 9201 1517 / - / 1515 / 1473 (later rounds are not in step any more: K and V come from further away).
// A half with a row out of the range of its weights is taken again as a 256-row tile with shifts: a workgroup alone on its CU,
// 0.6 of the time of a pair of them.  us, launches of 256-row tiles / every tile with such a row taken again whole / this,
// 16 x 28700 x 12001: one row in the first tile of each head 1121 / 1213 / 1116, one row in 4096 1436 / 1759 / 1373, one in 512 1965 /
// 2345 / 1686, all rows 2202 / 2342 / 2335, all scores low 2019 / 2244 / 2228, half of the keys masked 964 / 960 / 950; 16 x 16384 x 9000, one
// row a head 537 / 690 / 556, all rows 951 / 1011 / 1005.

// The halves of the tile (bit 0: rows 0 .. 255, bit 1: the others) with a row that has left the range of its weights; nothing is
// stored of these.
__device__ __forceinline__ int wide_tile(const AttnArgs& a, KvTile& k0, KvTile& k1, KvTile& k2, KvTile& v0, KvTile& v1, KvTile& v2, u32x4* s_rows, int (&s_again)[2], int (&s_low)[2],
                                          const int h, const int q0, const bool dev_tile, const int64_t q_base_dev, const int mq_dev,
                                          const SplitSegment seg) {
  constexpr int NQ = 8, NT = 256;
  const bool piece = seg.slot >= 0;
  const int64_t q_base = dev_tile ? q_base_dev : a.q_off[h];
  int64_t k_base = a.k_off[h];
  const int Mq = dev_tile ? mq_dev : a.q_rows[h];
  int Mk = (int)(a.k_off[h + 1] - k_base);
  if (piece) {
    k_base += (int64_t)seg.t0 * kKvTile;
    Mk = (seg.t1 * kKvTile < Mk ? seg.t1 * kKvTile : Mk) - seg.t0 * kKvTile;
  }
  const bf16_t* __restrict__ q_rows = dev_tile ? a.q2 : a.q;
  u32x4* __restrict__ o_rows = (u32x4*)(dev_tile ? a.o2 : a.o);
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));      // (as in attention_tile())
  const int lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq0 = q0 + wave * 16 * NQ, wave_half = wave >> 1;
  const bool active = __builtin_amdgcn_readfirstlane((int)(wq0 < Mq)) != 0;
  WaveState<NQ> w;
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    int row = wq0 + qt * 16 + l16;
    row = row < Mq ? row : Mq - 1;
    const bf16_t* p = q_rows + (q_base + row) * kDHead + grp * 8;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) w.qf[qt][ks] = *(const bf16x8*)(p + ks * 32);
    w.nm[qt] = 0.f;
    w.l_acc[qt >> 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) w.o_acc[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  w.c = 1.f;
  w.ones_a = row_sum_operand(lane);
  w.ones_idx = row_sum_index(lane);
  const char* kg = (const char*)(a.k + k_base * kDHead);
  const char* vg = (const char*)(a.v + k_base * kDHead);
  // (clamped without a branch: a loop of one block)
  auto load = [&](const char* rows, int kv0, KvTile& buf, auto is_v) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int blk = wave * 2 + i, r = blk * 8 + (lane >> 3);
      const int c = (lane & 7) ^ (decltype(is_v)::value ? v_swizzle(r) : k_swizzle(r));
      const int row = kv0 + r < Mk ? kv0 + r : Mk - 1;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(rows + (uint32_t)(row * kRowBytes + c * 16)),
                                       (__attribute__((address_space(3))) void*)(&buf[blk * 512]), 16, 0, 0);
    }
  };
  auto load_k = [&](int tile, KvTile& buf) { load(kg, tile * kKvTile, buf, std::false_type{}); };
  auto load_v = [&](int tile, KvTile& buf) { load(vg, tile * kKvTile, buf, std::true_type{}); };
  auto landed = [] {
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    __syncthreads();
  };
  const int n_tiles = (Mk + kKvTile - 1) / kKvTile;
  load_k(0, k0);
  load_v(0, v0);
  if (n_tiles > 1) load_k(1, k1);
  if (tid < 2) s_again[tid] = s_low[tid] = 0;
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) asm volatile("" : "+a"(w.qf[qt][0]), "+a"(w.qf[qt][1]));
  accumulators_settled(w);
  landed();
  // the steps, 0 .. 2 * n_tiles - 1, as in attention_tile()
  if (active) {
    pipeline_step<NQ, false, true, false, false, false, false>(w, k0, nullptr, kg, 0, Mk, lane);
    if (n_tiles > 1)
      pipeline_step<NQ, false, true, false, true, false, true>(w, k0 + kStep * kDHead, nullptr, kg, 0, Mk, lane);
    else
      pipeline_step<NQ, false, true, false, true, true, true>(w, k0 + kStep * kDHead, nullptr, kg, 0, Mk, lane);
  }
  __syncthreads();
  int j = 1;
  if (n_tiles > 1) {
    // Tile jt asks for K tile jt + 2 and V tile jt + 1 (past the end: the last rows again, so that it is always four requests),
    // and waits for those of the tile before.
    auto arrived = [] {
      __builtin_amdgcn_s_waitcnt(0x0074);   // vmcnt(4) lgkmcnt(0)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    load_k(2, k2);
    load_v(1, v1);
    if (!active) {
      // a wave of a partial tile without valid rows: it only stages its share of K / V
      for (; j < n_tiles - 1; ++j) {
        const int m = j % 3;
        load_k(j + 2, m == 0 ? k2 : m == 1 ? k0 : k1);
        load_v(j + 1, m == 0 ? v1 : m == 1 ? v2 : v0);
        arrived();
      }
    } else {
      StepOperands op;
      load_v_operands(op, v0, l16, grp);
      __builtin_amdgcn_sched_barrier(0);
      // K tile jt (kc) against V tile jt - 1 (vc), whose first operands are there, and the first operands of V tile jt (vn), behind the
      // barrier that says that it has arrived.  Requested are K tile jt + 2 into the buffer kr of K tile jt - 1 and V tile jt + 1 into
      // the buffer vr of V tile jt - 2: everybody has read those before the barrier of tile jt - 1.  (Behind a request the compiler
      // waits for all LDS reads, the youngest as well: the requests lie where the next wait is for all that there are.)
      auto tile = [&](int jt, KvTile& kc, KvTile& kr, KvTile& vc, KvTile& vn, KvTile& vr) {
        wide_step(w, op, kc, vc + kStep * kDHead, lane, [] {}, [&](int g) {
          if (g == 17) load_k(jt + 2, kr);
          if (g == 21) load_v(jt + 1, vr);
        });
        wide_step(w, op, kc + kStep * kDHead, vn, lane, arrived, [](int) {});
      };
      for (; j + 2 < n_tiles - 1; j += 3) {
        tile(j, k1, k0, v0, v1, v2);
        tile(j + 1, k2, k1, v1, v2, v0);
        tile(j + 2, k0, k2, v2, v0, v1);
      }
      if (j < n_tiles - 1) {
        tile(j, k1, k0, v0, v1, v2);
        ++j;
        if (j < n_tiles - 1) {
          tile(j, k2, k1, v1, v2, v0);
          ++j;
        }
      }
    }
    // the last K tile, its second step may be ragged
    const int m = j % 3;
    const bf16_t *kb = m == 0 ? k0 : m == 1 ? k1 : k2, *vb = m == 0 ? v2 : m == 1 ? v0 : v1;
    if (active) {
      pipeline_step<NQ, false, true, true, true, false, false>(w, kb, vb, kg, (2 * j - 1) * kStep, Mk, lane);
      pipeline_step<NQ, false, true, true, true, true, false>(w, kb + kStep * kDHead, vb + kStep * kDHead, kg, 2 * j * kStep, Mk, lane);
    }
    landed();
  }
  if (active) {
    const int m = n_tiles % 3;
    const bf16_t* vb = m == 0 ? v2 : m == 1 ? v0 : v1;
    pipeline_step<NQ, false, false, true, true, true, false>(w, nullptr, vb, kg, (2 * n_tiles - 1) * kStep, Mk, lane);
    pipeline_step<NQ, false, false, true, false, false, false>(w, nullptr, vb + kStep * kDHead, kg, 0, Mk, lane);
  }
  accumulators_settled(w);
  float l_tot[NQ];
  bool high = false, low = false;
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    const LanePair sums = row_sums(w.l_acc[qt >> 1][0]);
    l_tot[qt] = qt & 1 ? sums.b : sums.a;
    high = high || !(l_tot[qt] <= kFastSumMax);
    low = low || l_tot[qt] < kFastSumMin;
  }
  if (active && high) s_again[wave_half] = 1;
  if (active && low) s_low[wave_half] = 1;
  __syncthreads();
  if (piece) {
    if (s_low[0] | s_low[1]) {
      // its own sums may be small if those of the head's first, middle and last key tile alone are not (attention_tile())
      const int64_t head0 = a.k_off[h];
      const int keys = (int)(a.k_off[h + 1] - head0), last = (keys - 1) / kKvTile;
      kg = (const char*)(a.k + head0 * kDHead);
      Mk = keys;
      float rest[NQ];
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) rest[qt] = 0.f;
#pragma unroll 1
      for (int i = 0; i < 3; ++i) {
        load_k(i * last / 2, k0);
        landed();
        if (active) {
#pragma unroll 1
          for (int st = 0; st < kKvTile; st += kStep) {
            StepOperands op;
            load_k_operands(op, k0 + st * kDHead, l16, grp);
#pragma unroll
            for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
              for (int kt = 0; kt < 2; ++kt) {
                const f32x4 sc = mfma16(op.ak[kt * 2 + 1], w.qf[qt][1], mfma16(op.ak[kt * 2], w.qf[qt][0], f32x4{0.f, 0.f, 0.f, 0.f}));
#pragma unroll
                for (int r = 0; r < 4; ++r)
                  rest[qt] += i * last / 2 * kKvTile + st + 16 * kt + 4 * grp + r < keys ? __builtin_amdgcn_exp2f(sc[r]) : 0.f;
              }
          }
        }
        __syncthreads();
      }
      low = false;
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        const LanePair r1 = swap16(rest[qt]), r2 = swap32(r1.a + r1.b);
        low = low || !(r2.a + r2.b >= kFastSumMin);
      }
      if (active && low) s_again[wave_half] = 1;
      __syncthreads();
    }
    const int bad = __builtin_amdgcn_readfirstlane(s_again[0] | 2 * s_again[1]);
    if (active && !(bad >> wave_half & 1)) {
      // (slots as attention_tile() leaves them, two for a tile)
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        const int r = (wave * NQ + qt) * 16 + l16;
        if (q0 + r >= Mq) continue;
        const int64_t slot_row0 = (int64_t)(seg.slot + r / kAttnTileRows) * kAttnTileRows, sr = r % kAttnTileRows;
        float* po = a.split_o + slot_row0 * kDHead + sr * 4;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) *(f32x4*)(po + (4 * ct + grp) * (kAttnTileRows * 4)) = w.o_acc[ct][qt];
        if (grp == 0) {
          a.split_l[slot_row0 + sr] = l_tot[qt];
          a.split_m[slot_row0 + sr] = 0.f;
        }
      }
    }
    return bad;
  }
  const int bad = __builtin_amdgcn_readfirstlane((s_again[0] | s_low[0]) | 2 * (s_again[1] | s_low[1]));
  if (bad == 3) return bad;
  const UnmergeTarget um = unmerge_target();
  // the rows that are stored
  const int n_tile = Mq - q0 < kWideRows ? Mq - q0 : kWideRows;
  const int first = bad == 1 ? kAttnTileRows : 0, n = (bad == 2 ? kAttnTileRows : n_tile) - first;
  UnmergeSpan span = {0, 0};
  UnmergeBatch batch;
  if (um.out && !dev_tile) {
    const int row0 = unmerge_row0(um, h, q0 + first);
    span = unmerge_span(um, row0, n);
    unmerge_load<NT>(batch, um, h, row0, n, span.first, span.end, tid);
  }
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    const float inv = 1.0f / l_tot[qt];
    const int r = (wave * NQ + qt) * 16 + l16;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
      *((u32x2*)&s_rows[out_chunk(r, 2 * ct + (grp >> 1))] + (grp & 1)) =
          u32x2{pack_bf16x2(w.o_acc[ct][qt][0] * inv, w.o_acc[ct][qt][1] * inv),
                pack_bf16x2(w.o_acc[ct][qt][2] * inv, w.o_acc[ct][qt][3] * inv)};
  }
  __syncthreads();
  const u32x4* rows = s_rows + first * kRowChunks;
  if (um.out) {
    unmerge_tile<NT, kWideRows>(um, batch, rows, o_rows, h, q0 + first, n, q_base, dev_tile, span, tid);
    return bad;
  }
#pragma unroll
  for (int i = 0; i < kWideRows * kRowChunks / NT; ++i) {
    const int r = (tid >> 3) + i * (NT / 8), c = tid & 7;
    if (r < n) o_rows[(q_base + q0 + first + r) * kRowChunks + c] = rows[out_chunk(r, c)];
  }
  return bad;
}

// Whole tiles as in attention_kernel, then the device-side list's, then the shares.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void attention_wide_kernel(const AttnArgs a) {
  __shared__ __align__(16) KvTile k0, k1, k2, v0, v1, v2;
  __shared__ __align__(16) bf16_t rows[kWideRows / kKvTile][kKvTile * kDHead];   // the finished rows
  __shared__ int s_again[2], s_low[2];
  const int block = (int)blockIdx.x, xcd = block & 7, pos = block >> 3;
  int h = 0, q0 = 0, mq_dev = 0;
  int64_t q_base_dev = 0;
  int share = -1, first = 0, count = 1;
  const bool dev_tile = block >= a.main_blocks && block < a.share_block0;
  if (dev_tile) {
    if (!a.dev_tiles) return;
    const int t = block - a.main_blocks;
    if (t >= a.dev_tiles[0]) return;
    h = a.dev_tiles[1 + 2 * t];
    q0 = a.dev_tiles[2 + 2 * t];
    q_base_dev = a.dev_q_off[h];
    mq_dev = a.dev_q_off[h + 1] - a.dev_q_off[h];
  } else if (block >= a.share_block0) {
    const int item = (block - a.share_block0) >> 3;
    share = xcd * a.split_per_xcd + item;
    if (item >= a.split_per_xcd || share >= a.sp.shares) return;
    split_share_tiles(a.sp, share, &first, &count);
  } else if (pos < a.ragged_per_xcd) {
    const int i = pos * 8 + xcd;
    if (i >= a.n_ragged) return;
    h = a.ragged_head[i];
    q0 = (a.tile_start[h + 1] - a.tile_start[h]) * kWideRows;
  } else {
    const int tile = xcd * a.full_per_xcd + (pos - a.ragged_per_xcd);
    if (tile >= a.n_full) return;
    while (tile >= a.tile_start[h + 1]) ++h;
    q0 = (tile - a.tile_start[h]) * kWideRows;
  }
#pragma unroll 1
  for (int i = 0; i < count; ++i) {
    SplitSegment seg = {0, 0, 0, 0, -1};
    if (share >= 0) {
      seg = split_segment<true>(a.sp, share, first + i);
      h = seg.head;
      q0 = seg.q0;
      if (i) __syncthreads();                       // the tile buffers in LDS are free again
    }
    const int n = (dev_tile ? mq_dev : a.q_rows[h]) - q0;
    if (n <= kAttnTileRows) {
      // a partial tile with few rows: waves of 64 rows, which walk twice as fast
      attention_tile<4, 4, 1, false>(a, rows, h, q0, dev_tile, q_base_dev, mq_dev, seg);
      continue;
    }
    const int bad = wide_tile(a, k0, k1, k2, v0, v1, v2, (u32x4*)rows, s_again, s_low, h, q0, dev_tile, q_base_dev, mq_dev, seg);
    // Rare: with per-row shifts, in 256-row tiles.
#pragma unroll 1
    for (int half = 0; bad >> half != 0; ++half) {
      if (!(bad >> half & 1)) continue;
      SplitSegment part = seg;
      if (share >= 0) part.slot += half;
      __syncthreads();
      attention_tile<4, 4, 1, true>(a, rows, h, q0 + half * kAttnTileRows, dev_tile, q_base_dev, mq_dev, part);
    }
  }
}

// SHIFT = false: the keys carry the logit scale, weights exp2(s).  SHIFT = true: any keys and scale.
template <int NQ, int NW, int KS, bool SHIFT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NQ == 2 && KS == 1 ? 3 : 2, NQ == 2 && KS == 1 ? 3 : 2)))
void attention_kernel(const AttnArgs a) {
  constexpr int BQ = 16 * NQ * (NW / KS);
  // per key group two tiles of K and two of V: [kv][d], 128-byte rows, chunk-swizzled
  __shared__ __align__(16) bf16_t lds[lds_tiles<NQ, NW, KS>()][kKvTile * kDHead];

  // blockIdx -> work.  Workgroups go round-robin to the 8 XCDs, and in blockIdx order to free
  // slots.  Every XCD walks its whole tiles first - the partial last tiles of the heads (they are
  // short, so they should not be what the grid ends on), then a contiguous range of full tiles -
  // and then its shares of the tiles that run in segments; the device-side tile list comes last.
  const int block = (int)blockIdx.x;
  const int xcd = block & 7;
  int h = 0, q0 = 0, mq_dev = 0;
  int64_t q_base_dev = 0;
  int share = -1, first = 0, count = 1;           // share >= 0: `count` segments, in the tiles first, first + 1, ...
  const bool dev_tile = block >= a.main_blocks;
  const int pos = block >> 3, whole_per_xcd = a.full_per_xcd + a.ragged_per_xcd;
  if (dev_tile) {
    if (!a.dev_tiles) return;
    int t = block - a.main_blocks, half = 0;
    if constexpr (KS == 1 && BQ == kAttnTileRows) {
      half = t & a.dev_halves;
      t >>= a.dev_halves;
    }
    if (t >= a.dev_tiles[0]) return;
    h = a.dev_tiles[1 + 2 * t];
    q0 = a.dev_tiles[2 + 2 * t] + half * kAttnTileRows;
    q_base_dev = a.dev_q_off[h];
    mq_dev = a.dev_q_off[h + 1] - a.dev_q_off[h];
    if (half && q0 >= mq_dev) return;
  } else if (KS == 1 && pos >= whole_per_xcd) {
    const int item = pos - whole_per_xcd;
    share = xcd * a.split_per_xcd + item;
    if (item >= a.split_per_xcd || share >= a.sp.shares) return;
    split_share_tiles(a.sp, share, &first, &count);
  } else if (pos < a.ragged_per_xcd) {
    const int i = pos * 8 + xcd;
    if (i >= a.n_ragged) return;
    h = a.ragged_head[i];
    q0 = (a.tile_start[h + 1] - a.tile_start[h]) * BQ;
  } else {
    const int tile = xcd * a.full_per_xcd + (pos - a.ragged_per_xcd);
    if (tile >= a.n_full) return;
    while (tile >= a.tile_start[h + 1]) ++h;
    q0 = (tile - a.tile_start[h]) * BQ;
  }
  // a whole tile; or a share of the tiles that run in segments: its segments one after the other
  for (int i = 0; i < count; ++i) {
    SplitSegment seg = {0, 0, 0, 0, -1};
    if (share >= 0) {
      seg = split_segment<false>(a.sp, share, first + i);
      h = seg.head;
      q0 = seg.q0;
      if (i) __syncthreads();                       // the tile buffers in LDS are free again
    }
    attention_tile<NQ, NW, KS, SHIFT>(a, lds, h, q0, dev_tile, q_base_dev, mq_dev, seg);
  }
}

// The split tiles after attention_kernel ran them in segments: four (eight) workgroups per split tile (64 rows
// each) bring its segments to the largest of their shifts of a row (all zero unless a segment had
// to take shifts or the keys are plain), add them in ascending key order (run-to-run
// identical) and store the normalised rows.  Bound by the latency of one chain of loads - 16 to 30 MB
// over the chip - so every thread fetches the sums and the shifts of its own row next to its
// values instead of taking them from LDS behind a barrier, kReduceBatch segments at a time.
constexpr int kReduceRows = 64;
constexpr int kReduceBatch = 3;
template <bool WIDE>
__global__ __launch_bounds__(256) void attention_split_reduce_kernel(const AttnArgs a) {
  constexpr int BQ = kAttnTileRows;                // rows of a slot
  __shared__ u32x4 s_out[kReduceRows * kRowChunks];   // the normalised bf16 rows, for whole-line stores
  constexpr int TILE = WIDE ? kWideRows : BQ, PARTS = TILE / kReduceRows;
  const int e = blockIdx.x / PARTS, part = blockIdx.x % PARTS, tid = threadIdx.x;
  const SplitTile t = split_tile<WIDE>(a.sp, e);
  const int64_t q_base = a.q_off[t.head];
  const int left = a.q_rows[t.head] - t.q0;
  const int rows = left < TILE ? left : TILE;
  if (part * kReduceRows >= rows) return;
  const int np = t.last_share - t.first_share + 1;
  // consecutive shares of one tile have consecutive slots (pairs of slots, the second for the rows from 256 on)
  const int64_t step = slots_per_segment<WIDE>(a.sp, e) * BQ;
  const int64_t row0 = (int64_t)(split_slot<WIDE>(a.sp, t.first_share, e) + part * kReduceRows / BQ) * BQ;     // segment p: rows from row0 + p * step
  const int q_part = t.q0 + part * kReduceRows, n_part = rows - part * kReduceRows < kReduceRows ? rows - part * kReduceRows : kReduceRows;
  const int row0_part = row_in_head(q_base, t.head, a.um.M, q_part);
  UnmergeSpan span = {0, 0};
  UnmergeBatch batch;
  if (a.um.out) {
    span = unmerge_span(a.um, row0_part, n_part);
    unmerge_load<256>(batch, a.um, t.head, row0_part, n_part, span.first, span.end, tid);
  }
  // thread -> row r = tid % 64 of the part and the 16-byte output chunks c0, c0 + 4
  const int r = part * kReduceRows + (tid & 63), c0 = tid >> 6;
  const int rr = (r < rows ? r : rows - 1) % BQ;          // a row past the end reads a valid row and stores nothing
  float acc[2][8];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[i][q] = 0.f;
  float m_row = kLowestScore, l_row = 0.f;
  for (int p0 = 0; p0 < np; p0 += kReduceBatch) {
    f32x4 v[kReduceBatch][2][2];
    float m[kReduceBatch], l[kReduceBatch];
#pragma unroll
    for (int u = 0; u < kReduceBatch; ++u) {
      const int64_t row = row0 + (int64_t)(p0 + u < np ? p0 + u : np - 1) * step + rr;   // past the last one: that one again
      m[u] = a.split_m[row];
      l[u] = a.split_l[row];
      const float* ps = a.split_o + (row - rr) * kDHead + rr * 4;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) v[u][i][hf] = *(const f32x4*)(ps + ((c0 + 4 * i) * 2 + hf) * (BQ * 4));
    }
    float m_new = m_row;
#pragma unroll
    for (int u = 0; u < kReduceBatch; ++u) m_new = fmaxf(m_new, m[u]);
    const float old = __builtin_amdgcn_exp2f(m_row - m_new);
    m_row = m_new;
    l_row *= old;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[i][q] *= old;
#pragma unroll
    for (int u = 0; u < kReduceBatch; ++u) {
      const float wgt = p0 + u < np ? __builtin_amdgcn_exp2f(m[u] - m_row) : 0.f;
      l_row = fmaf(l[u], wgt, l_row);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[i][4 * hf + q] = fmaf(v[u][i][hf][q], wgt, acc[i][4 * hf + q]);
    }
  }
  const float inv = 1.0f / l_row;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = pack_bf16x2(acc[i][2 * q] * inv, acc[i][2 * q + 1] * inv);
    s_out[out_chunk(tid & 63, c0 + 4 * i)] = o;
  }
  __syncthreads();
  // whole 128-byte rows: 8 threads per row
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int lr = (tid >> 3) + 32 * i, ch = tid & 7;
    if (lr < n_part) ((u32x4*)a.o)[(q_base + q_part + lr) * kRowChunks + ch] = s_out[out_chunk(lr, ch)];
  }
  if (a.um.out) unmerge_store<256>(batch, a.um, s_out, t.head, row0_part, n_part, span, tid);
}

// compute units of the current device (asked once per device)
int64_t compute_units() {
  static int cached[64] = {0};
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev]) return cached[dev];
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
  cached[dev] = n;
  return n;
}

template <int NQ, int NW, int KS = 1>
void launch_kernel(const AttnArgs& a, bool log2_keys, unsigned grid, hipStream_t stream) {
  if (log2_keys)
    hipLaunchKernelGGL((attention_kernel<NQ, NW, KS, false>), dim3(grid), dim3(64 * NW), 0, stream, a);
  else
    hipLaunchKernelGGL((attention_kernel<NQ, NW, KS, true>), dim3(grid), dim3(64 * NW), 0, stream, a);
}

// The tiles of `tile_rows` rows of a launch, into its arguments; with a split (`route`) those that stay whole, and the
// segments, whose partial results go to `scratch`.
void set_tiles(AttnArgs& a, int tile_rows, const HeadRows& rows, const int64_t* k_off_host, int H, const AttnRoute* route, float* scratch) {
  int64_t full = 0;
  int ragged = 0;
  for (int h = 0; h < H; ++h) {
    const int64_t mq = rows.count[h];
    a.tile_start[h] = (int32_t)full;
    a.q_off[h] = rows.first[h];
    a.q_rows[h] = (int32_t)mq;
    a.k_off[h] = k_off_host[h];
    full += mq / tile_rows;
    if (mq % tile_rows) a.ragged_head[ragged++] = h;
  }
  for (int h = H; h <= kAttnMaxHeads; ++h) {
    a.tile_start[h] = (int32_t)full;
    if (h < kAttnMaxHeads) {
      a.q_off[h] = 0;
      a.q_rows[h] = 0;
    }
    a.k_off[h] = k_off_host[H];
  }
  for (int i = ragged; i < kAttnMaxHeads; ++i) a.ragged_head[i] = 0;
  a.n_full = (int32_t)full;
  a.n_ragged = ragged;
  a.split_per_xcd = 0;
  a.split_o = nullptr;
  a.split_l = nullptr;
  a.split_m = nullptr;
  a.sp.n_tiles = 0;
  a.sp.slots = 0;
  if (route && route->split.n_tiles > 0) {
    // the first partial tiles (in head order) and the last full tiles run in segments; the others
    // keep their order: partial tiles in front of the full tiles
    a.sp = route->split;
    const int64_t slots = split_slots(a.sp);
    a.n_full = (int32_t)route->kept_full;
    a.n_ragged = ragged - route->split_ragged;
    for (int i = 0; i < a.n_ragged; ++i) a.ragged_head[i] = a.ragged_head[route->split_ragged + i];
    a.split_per_xcd = (a.sp.shares + 7) / 8;
    a.split_o = scratch;
    a.split_l = scratch + slots * kAttnTileRows * kDHead;
    a.split_m = a.split_l + slots * kAttnTileRows;
  }
  a.full_per_xcd = (a.n_full + 7) / 8;
  a.ragged_per_xcd = (a.n_ragged + 7) / 8;
}

hipError_t launch_reduce(const AttnArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)(a.sp.tile_rows / kReduceRows * a.sp.n_tiles));
  if (a.sp.n_tiles > 0 && a.sp.tile_rows == kWideRows)
    hipLaunchKernelGGL((attention_split_reduce_kernel<true>), grid, dim3(256), 0, stream, a);
  else if (a.sp.n_tiles > 0)
    hipLaunchKernelGGL((attention_split_reduce_kernel<false>), grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

// `route`: the split of a launch of 256-row tiles, if it has one.
template <int NQ, int NW, int KS = 1>
hipError_t launch_cfg(AttnArgs& a, bool log2_keys, const HeadRows& rows, const int64_t* k_off_host, int H, hipStream_t stream, int extra_tiles = 0, const AttnRoute* route = nullptr, float* scratch = nullptr) {
  set_tiles(a, 16 * NQ * (NW / KS), rows, k_off_host, H, route, scratch);
  if (a.n_full + a.n_ragged + a.sp.n_tiles + extra_tiles == 0) return hipSuccess;
  a.main_blocks = 8 * (a.full_per_xcd + a.ragged_per_xcd + a.split_per_xcd);
  launch_kernel<NQ, NW, KS>(a, log2_keys, (unsigned)a.main_blocks + (unsigned)extra_tiles, stream);
  return launch_reduce(a, stream);
}

// 512-row tiles (log2 keys).  The shares come behind the device-side list's tiles: they are the shorter ones, and a launch
// ends the more evenly the shorter its last workgroups are.
hipError_t launch_wide(AttnArgs& a, const HeadRows& rows, const int64_t* k_off_host, int H, hipStream_t stream, int extra_tiles,
                       const AttnRoute* route = nullptr, float* scratch = nullptr) {
  set_tiles(a, kWideRows, rows, k_off_host, H, route, scratch);
  if (a.n_full + a.n_ragged + a.sp.n_tiles + extra_tiles == 0) return hipSuccess;
  a.main_blocks = 8 * (a.full_per_xcd + a.ragged_per_xcd);
  a.share_block0 = a.main_blocks + (extra_tiles + 7) / 8 * 8;
  hipLaunchKernelGGL(attention_wide_kernel, dim3((unsigned)(a.share_block0 + 8 * a.split_per_xcd)), dim3(256), 0, stream, a);
  return launch_reduce(a, stream);
}

// A launch without a split.  `extra_tiles` workgroups are appended for the device-side tile list (a.dev_tiles), if any.
hipError_t launch_tiles(AttnTiles tiles, AttnArgs& a, bool log2_keys, const HeadRows& rows, const int64_t* k_off_host, int H, hipStream_t stream,
                        int extra_tiles = 0) {
  switch (tiles) {
    case AttnTiles::kGroups32: return launch_cfg<2, 4, 4>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
    case AttnTiles::kGroups64: return launch_cfg<2, 8, 4>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
    case AttnTiles::kGroups128: return launch_cfg<2, 8, 2>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
    case AttnTiles::kGroups128Wide: return launch_cfg<4, 8, 4>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
    case AttnTiles::kGroups256: return launch_cfg<4, 8, 2>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
    case AttnTiles::kTiles128: return launch_cfg<2, 4>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
    case AttnTiles::kTiles512: return launch_wide(a, rows, k_off_host, H, stream, extra_tiles);
    default: return launch_cfg<4, 4>(a, log2_keys, rows, k_off_host, H, stream, extra_tiles);
  }
}

AttnArgs attention_args(const void* q, const void* k, const void* v, void* o, int H, float scale, bool log2_keys, const UnmergeTarget* unmerge) {
  AttnArgs a;
  std::memset(&a, 0, sizeof(a));
  a.q = (const bf16_t*)q;
  a.k = (const bf16_t*)k;
  a.v = (const bf16_t*)v;
  a.o = (bf16_t*)o;
  a.scale_log2 = log2_keys ? 1.0f : scale * 1.4426950408889634f;
  a.H = H;
  if (unmerge) a.um = *unmerge;
  return a;
}

// `extra_tiles` of the device-side list go to the end of the (last) launch.
hipError_t launch_route(const AttnRoute& route, AttnArgs& a, bool log2_keys, const int64_t* q_off_host, const int64_t* k_off_host, int H,
                        int64_t cus, hipStream_t stream, void* scratch, int extra_tiles) {
  if (route.tiles == AttnTiles::kTiles256)
    return launch_cfg<4, 4>(a, log2_keys, all_rows(q_off_host, H), k_off_host, H, stream, extra_tiles, &route, (float*)scratch);
  if (route.tiles == AttnTiles::kTiles512)
    return launch_wide(a, all_rows(q_off_host, H), k_off_host, H, stream, extra_tiles, &route, (float*)scratch);
  if (route.tiles != AttnTiles::kRounds)
    return launch_tiles(route.tiles, a, log2_keys, all_rows(q_off_host, H), k_off_host, H, stream, extra_tiles);
  HeadRows whole, rest;
  split_rounds(q_off_host, H, cus, &whole, &rest);
  const hipError_t e = launch_cfg<4, 4>(a, log2_keys, whole, k_off_host, H, stream);
  if (e != hipSuccess) return e;
  return launch_tiles(route.rest, a, log2_keys, rest, k_off_host, H, stream, extra_tiles);
}

}  // namespace

int64_t attention_scratch_need(const int64_t* q_off_host, const int64_t* k_off_host, int H) {
  AttnRoute route;
  choose_attention_route(q_off_host, k_off_host, H, compute_units(), INT64_MAX, &route);
  return split_slots(route.split) * kAttnSlotWords * 4;
}

void choose_dev_tiles(int64_t rows, int64_t M_q, int64_t M_k, int H, bool log2_keys, int32_t* kind, int32_t* tile_rows) {
  // In the merged rows' tiles, behind them in the same launch, if all of them are still one round, and in 256-row tiles of one
  // key group always.  Otherwise in a launch of their own, in the tiles that are quickest: a launch of 256-row tiles of one key
  // group for both would be quicker behind whole rounds (3 to 7 %), but the merged rows' sums would not be those of the
  // separate stage call.  Layers with the outlier filter, us, all in 256-row tiles of one key group / always two launches /
  // so: 12 heads x 360 rows x 360 keys and 698 others 57 / 55 / 49, 16 x 1140 x 1140 and 441 69 / 67 / 56, 16 x 2676 x 2676 and 6790
  // 102 / 111 / 91, 24 x 2028 x 2028 and 10872 105 / 114 / 94, 8 x 6294 x 8726 and 3530 252 / 218 / 174, 24 x 1578 x 1578 and
  // 5736 86 / 93 / 78; two launches: 12 x 4962 x 4962 and 10522 184 / 169 / 169, 16 x 9914 x 1471 and 3988 163 / 172 / 172.
  int64_t q_off[kAttnMaxHeads + 1], k_off[kAttnMaxHeads + 1];
  for (int h = 0; h <= H; ++h) {
    q_off[h] = h * M_q;
    k_off[h] = h * M_k;
  }
  const int64_t cus = compute_units();
  AttnRoute route;
  choose_attention_route(q_off, k_off, H, cus, attention_scratch_bytes(H) / 4, &route, log2_keys);
  AttnTiles t = last_tiles(route);
  if (t == AttnTiles::kTiles512) {
    // Small tiles, which share the keys, if all of them are one round.  Else behind the merged rows in the same launch or in
    // 256-row tiles of their own, by the time in rounds of 512-row tiles (thousandths): whole rounds, what is left over next to the
    // merged rows' segments, and half a round of 256-row tiles takes 0.6 of one.  us a layer of 16 heads, all in 256-row tiles /
    // together / two launches: 28650 x 28650 and 65952 others 3369 / 3310 / -, 28700 x 28700 and 439680 5481 / 5362 / -, 25980 x 25980 and
    // 39571 2572 / 2565 / -, 2634 / - / 2543, and 131904 3145 / 3233 / -, 3108 / - / 3107, 17760 x 17760 and 42209 1347 / 1365 / -, 1410 / - / 1405;
    // in small tiles: 28650 x 28650 and 6595 2989 / - / 2832.
    const AttnTiles small = choose_key_groups([&](int n) { return rows / n + H; }, cus, (M_k + kAttnKeyTile - 1) / kAttnKeyTile, 0, rows).tiles;
    const int64_t dev = 1000 * (rows / kWideRows + H / 2) / cus, left = dev % 1000, segments = 1000 * route.split.n_tiles / cus;
    const int64_t together = left == 0 ? segments : std::max<int64_t>(1000, left + segments);
    const int64_t apart = segments + (left == 0 ? 0 : left <= 500 ? 600 : 1000);
    if (attention_tile_rows(small) < kAttnTileRows)
      t = small;
    else if (apart < together)
      t = AttnTiles::kTiles256;
  } else if (t != AttnTiles::kTiles256) {
    const int64_t extra = rows / attention_tile_rows(t) + (H + 1) / 2;     // (a partial tile per head at most: half of them, say)
    if (count_last_tiles(route, q_off, H, cus) + (extra + 7) / 8 * 8 > (t == AttnTiles::kTiles128 ? kSmallTileRound : cus))
      t = choose_key_groups([&](int n) { return rows / n + H; }, cus, (M_k + kAttnKeyTile - 1) / kAttnKeyTile, 0, rows).tiles;
  }
  *kind = (int32_t)t;
  *tile_rows = attention_tile_rows(t);
}

// Whether the 512-row tiles of a device-side list of `rows` rows run quicker in a launch of their own as two 256-row tiles each,
// which gives the same sums: in time per key tile, a round of 512-row tiles takes 1462, one of pairs of 256-row tiles 1517 and a
// last one with no more than one a CU 0.6 of that.  us, 512-row tiles / two 256-row tiles, 16 heads against 28650 keys: 32976 rows
// 557 / 393, 65952 562 / 593, 175872 1189 / 1016, 219840 1235 / 1293, 329760 1925 / 2003, 28700 keys: 131904 1188 / 958, 439680 2624 / 2458,
// 17760 keys: 70348 350 / 371.
bool dev_tiles_in_halves(int64_t rows, int H, int64_t cus) {
  const int64_t wide = rows / kWideRows + H / 2, narrow = rows / kAttnTileRows + H / 2, rest = narrow % (2 * cus);
  const int64_t time = (wide + cus - 1) / cus * 1462;
  return narrow / (2 * cus) * 1517 + (rest == 0 ? 0 : rest <= cus ? 910 : 1517) < time;
}

hipError_t launch_attention_dev_tiles(const void* q, const void* k, const void* v, void* o, const DevTiles& dev,
                                      const int64_t* k_off_host, int H, float scale, bool log2_keys,
                                      hipStream_t stream, const UnmergeTarget* unmerge) {
  if (dev.max_tiles <= 0) return hipSuccess;
  AttnArgs a = attention_args(q, k, v, o, H, scale, log2_keys, unmerge);
  a.dev_q_off = dev.q_off;
  a.dev_tiles = dev.tiles;
  a.q2 = a.q;
  a.o2 = a.o;
  HeadRows none = {};       // no whole tiles, no segments: every workgroup takes the device-side list
  if ((AttnTiles)dev.kind == AttnTiles::kTiles512 && dev_tiles_in_halves((int64_t)(dev.max_tiles - H) * kWideRows, H, compute_units())) {
    a.dev_halves = 1;
    return launch_tiles(AttnTiles::kTiles256, a, log2_keys, none, k_off_host, H, stream, 2 * dev.max_tiles);
  }
  return launch_tiles((AttnTiles)dev.kind, a, log2_keys, none, k_off_host, H, stream, dev.max_tiles);
}

hipError_t launch_attention_both(const void* q, const void* k, const void* v, void* o,
                                 const int64_t* q_off_host, const int64_t* k_off_host, int H, float scale,
                                 const void* q2, void* o2, const DevTiles& dev, bool log2_keys, hipStream_t stream,
                                 void* scratch, int64_t scratch_bytes, const UnmergeTarget* unmerge) {
  AttnArgs a = attention_args(q, k, v, o, H, scale, log2_keys, unmerge);
  const int64_t cus = compute_units();
  AttnRoute route;
  choose_attention_route(q_off_host, k_off_host, H, cus, scratch ? scratch_bytes / 4 : 0, &route, log2_keys);
  const bool together = dev.max_tiles > 0 && dev.kind == (int32_t)last_tiles(route);
  if (together) {
    a.dev_q_off = dev.q_off;
    a.dev_tiles = dev.tiles;
    a.q2 = (const bf16_t*)q2;
    a.o2 = (bf16_t*)o2;
  }
  const hipError_t e = launch_route(route, a, log2_keys, q_off_host, k_off_host, H, cus, stream, scratch, together ? dev.max_tiles : 0);
  if (e != hipSuccess || together) return e;
  return launch_attention_dev_tiles(q2, k, v, o2, dev, k_off_host, H, scale, log2_keys, stream, unmerge);
}

hipError_t launch_attention(const void* q, const void* k, const void* v, void* o,
                            const int64_t* q_off_host, const int64_t* k_off_host, int H,
                            float scale, bool log2_keys, hipStream_t stream, void* scratch, int64_t scratch_bytes,
                            const UnmergeTarget* unmerge) {
  AttnArgs a = attention_args(q, k, v, o, H, scale, log2_keys, unmerge);
  const int64_t cus = compute_units();
  AttnRoute route;
  choose_attention_route(q_off_host, k_off_host, H, cus, scratch ? scratch_bytes / 4 : 0, &route, log2_keys);
  return launch_route(route, a, log2_keys, q_off_host, k_off_host, H, cus, stream, scratch, 0);
}

// ---- scratch that belongs to the library -------------------------------------------------------
// For callers that cannot allocate device memory (code under HIP graph capture, serving loops, test
// harnesses that forbid it): the room for the partial results of the tiles that run in pieces, as a
// device array of fixed size.  Every GPU the library runs on holds its own copy at its own address
// until the process ends; the array's name is only a host-side handle, the address comes from
// hipGetSymbolAddress, once per device, and only that pointer is ever handed to a kernel.
// (More of it than kAttnStaticScratchBytes, by which launches are accepted: those of 512-row tiles take larger slots.)
static __device__ __align__(256) unsigned char g_static_scratch[kAttnScratchBytes];

hipError_t attention_static_scratch(void** ptr) {
  static std::mutex mu;
  static void* per_device[64] = {nullptr};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  return hipSuccess;
}

}  // namespace httm
