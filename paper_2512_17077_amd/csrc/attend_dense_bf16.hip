// Refresh-phase attention (Section 2.3, Eq. 3): dense bidirectional softmax attention, bf16 inputs,
// fp32 softmax state and accumulators, on the gfx950 matrix cores.  This path is a dense
// contraction (4*Lq*Lkv*D flop per head against O(L*D) bytes), so it is bound by MFMA throughput.
// This file holds the kernel for head_dim D = 128; attend_dense_paired_bf16.hip the one for 64.
//
// Shape of the kernel
//   - A workgroup is four waves, one per SIMD, and owns 256 query rows of one (sequence, head); a wave
//     owns 64 of them as two blocks of 32.  Every K operand (ds_read_b128) and every V^T operand
//     (ds_read_b64_tr_b16) fetched from LDS feeds two MFMAs, one per block, which halves the LDS
//     operand traffic per flop, and the two blocks give the wave independent work to interleave.
//   - Calls with too few query rows for the compute units take the split form (KS = 2): a workgroup owns 128 query
//     rows, wave pair 0 takes the first 32 keys of every tile and wave pair 1 the other 32, and the pairs merge
//     their (m, l, O) through LDS at the end.  Every step is then a tile's first: K rows are requested four tiles
//     ahead and V rows two (the rings hold four of each; scores run two steps ahead of the P V product), and the
//     step waits for all but the previous step's requests.  One layer of one request (32 heads x 128, 1024 keys):
//     29.7 -> 24.6 us.
//   - Queries come in and outputs go out through LDS in whole rows: lanes of an operand or accumulator register lie
//     in 32 different rows, and its 16- or 8-byte pieces cost the load and store paths one line each (the same
//     layer 31.0 -> 27.8 us unsplit, 25.2 -> 23.4 us split).
//   - K/V tiles of 64 keys go from global memory straight into LDS (global_load_lds, 16 bytes per
//     lane), two tiles ahead of their use, into rings of four tiles each (128 KB at D = 128); one
//     workgroup barrier per tile.  LDS tiles are XOR-swizzled by row; since the LDS side of such a load
//     is lane-contiguous, the swizzle is applied to the global chunk each lane fetches.
//   - Keys are walked in steps of 32 with a three-deep software pipeline.  Iteration j issues
//         S^T(j+1) = K(j+1) Q^T          16 MFMAs (D = 128), A by ds_read_b128 one iteration ahead
//         P(j)     = exp2(S(j) z - m z)   vector work on the scores of the previous iteration
//         O^T     += V(j-1)^T P(j-1)^T    16 MFMAs, A by ds_read_b64_tr_b16 in the same iteration
//     so the matrix work of an iteration does not depend on its vector work and the issue order can
//     alternate them freely (one MFMA, then a few vector and LDS instructions, and so on).
//   - Q is not pre-scaled (rounding the scaled queries to bf16 again costs 2e-2 of output accuracy at
//     logits around 20): scores leave the matrix core raw, and one fused multiply-add per score,
//     s * z - m * z with z = softmax_scale * log2(e), makes them base-2 logits relative to the running
//     maximum m.
//   - m is set 2^24 above the maximum and raised lazily (when a score exceeds it by more than 2^8, see kDenseHeadroom, and
//     before a ragged last step) behind one uniform branch per iteration.  When it is raised after iteration j, the accumulators,
//     row sums among them, still have to take P(j) V(j) and the sums of P(j) at the old scale during iteration j+1 and are
//     rescaled one iteration later.
//   - The loop is unrolled over one turn of the rings (eight steps, four in the split form), so every LDS address is a register
//     fixed before the loop plus an immediate offset.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>
#include <utility>

#include "attend_dense.h"
#include "attend_dense_step.inc"

namespace dllm {

constexpr int kDenseK = 64;          // keys per LDS tile
constexpr int kDenseRing = 4;        // K tiles, and V tiles, resident in LDS
constexpr int kDenseWaves = 4;       // waves per workgroup
constexpr int kDenseQB = 2;          // 32-query blocks per wave
constexpr uint32_t kDenseUnits = 256;   // compute units: the most workgroups of a launch whose workgroups stay (KS = 1)
// query rows per workgroup; with KS = 2 two wave pairs take the same rows and half of every tile's keys each
constexpr int dense_rows(int ks) { return kDenseWaves * kDenseQB * 32 / ks; }

typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// The state a wave carries through the key loop, bound to the registers the step text of
// attend_dense_step.inc names.
//   a[0 : 16*2*NDB)          acc   O^T accumulators [qb][db][16]
//   a[.. +  4*2*NT)          q     Q^T operands [qb][t][4]
//   v[96:127], v[128:159]    st_a, st_b   raw scores of two consecutive steps, [qb][16]
//   v[160:175], v[176:191]   pb_a, pb_b   packed probabilities of two consecutive steps, [qb][u][4]
//   v[192 : 192 + 4*NT)      kop   K operands of the next score chain, [t][4]
//   v[80:95]                 addr  LDS byte addresses: K operand [t], then V^T operand [rd][db] from +8
//   a[.. + 4*2)              ls    row sums [qb][4] (only the first register is used, see DLLM_LS_OUT)
//   v72 .. v75               nmz[2] (= -m z per block), mx[2] (lane maxima of the newest scores)
//   v[76:79], v[224:255]     scratch of a step (logits in flight, V^T operand buffers)
// C++ code may read and write the v-register variables between steps like any others, and may write q;
// the accumulators are only ever handed from one assembly block to the next (this compiler cannot take
// single elements out of an a-register tuple that an assembly block has written), so clearing,
// rescaling and reading them are assembly blocks too.

// What the first step of a tile needs to request the tile two ahead: the tile's first K and V row
// (wave-uniform), the byte offset of each of this lane's 16-byte chunks from there, and the LDS address
// of this wave's slice of a load round.
constexpr int NLD = 4;   // 16-byte loads per lane, tile and tensor
struct DenseTileLoad {
  const char *k, *v;
  uint32_t off[NLD];
  uint32_t off_v[NLD];   // split form only: there K and V rows of different tiles are requested
  uint32_t wave_lds;
};

#define DLLM_DENSE_SCRATCH                                                                                        \
  "v76", "v77", "v78", "v79", "v224", "v225", "v226", "v227", "v228", "v229", "v230", "v231", "v232", "v233", "v234", \
      "v235", "v236", "v237", "v238", "v239", "v240", "v241", "v242", "v243", "v244", "v245", "v246", "v247", "v248", \
      "v249", "v250", "v251", "v252", "v253", "v254", "v255"
#define DLLM_R16(k, x) "=v"(x[16 * (k) + 0]), "=v"(x[16 * (k) + 1]), "=v"(x[16 * (k) + 2]), "=v"(x[16 * (k) + 3]), \
      "=v"(x[16 * (k) + 4]), "=v"(x[16 * (k) + 5]), "=v"(x[16 * (k) + 6]), "=v"(x[16 * (k) + 7]),                  \
      "=v"(x[16 * (k) + 8]), "=v"(x[16 * (k) + 9]), "=v"(x[16 * (k) + 10]), "=v"(x[16 * (k) + 11]),               \
      "=v"(x[16 * (k) + 12]), "=v"(x[16 * (k) + 13]), "=v"(x[16 * (k) + 14]), "=v"(x[16 * (k) + 15])

// Row sums are taken on the matrix cores: the bf16 probabilities of the lane's query, the same values the P V
// product multiplies, added in fp32 like its terms.  A v_mfma_f32_16x16x32_bf16 does it for a block of 32 queries
// and 16 keys: read as its B operand, the registers of P^T hold query c in column c % 16, with keys in contraction
// slots 0..7 and 16..23 if c < 16, in the other slots if not.  The A operand (`ones`) has bf16 ones in row 0 for the
// first kind and in row 4 for the second, so the four accumulators (ls) hold the sum of query c in the first register of
// lane c and zeros elsewhere.  (A 32x32x16 product with one row of ones takes twice the matrix time: 494 -> 481 us on
// eight sequences of 2048, 32 heads x 128, and 28 a-registers more.)  Two queries share a column, so no probability may be
// infinite or NaN, see is_lost (4x4x4 products, in which every lane has a column, cost 0.7 to 1.9 % of the calls'
// time).  The vector form (unpack each packed pair with a
// shift and a mask, two adds) costs four vector instructions per pair of scores, a third of the step's vector work;
// v_dot2c_f32_bf16 does it in one but runs on the matrix pipe and holds back the MFMAs (+18 cycles per MFMA), and summing
// the unrounded values is off by up to 2^-8 of a row that one key rules.
#define DLLM_LS_OUT "={a[192:195]}"(ls[0]), "={a[196:199]}"(ls[1])
#define DLLM_LS_TIED(a, b) a(ls[0]), b(ls[1])

// One step: AB reads the scores st_a and the probabilities pb_b and leaves the next scores in st_b and its own
// probabilities in pb_a, BA the other way round.  Split: the texts in which every step requests a tile.
#define DLLM_STEP_FUNCTION(D)                                                                                       \
  template <bool AB, bool Split, int KOFF, int VOFF0, int VOFF1, int LK, int LV>                                    \
  __device__ __forceinline__ void step(float zs, const DenseTileLoad& tl, uint64_t& grow) {                    \
    if constexpr (AB && Split)                                                                                      \
      asm volatile(DLLM_DENSE_STEP_##D##_AB_SPLIT                                                                   \
                   : DLLM_STEP_OUT("={v[128:143]}"(st_b[0]), "={v[144:159]}"(st_b[1]), "={v[160:175]}"(pb_a))        \
                   : DLLM_STEP_IN("{v[96:111]}"(st_a[0]), "{v[112:127]}"(st_a[1]), "{v[176:191]}"(pb_b)),            \
                     DLLM_STEP_LOADS_SPLIT                                                                          \
                   : "memory", "m0", "scc", DLLM_DENSE_SCRATCH);                                                    \
    else if constexpr (Split)                                                                                       \
      asm volatile(DLLM_DENSE_STEP_##D##_BA_SPLIT                                                                   \
                   : DLLM_STEP_OUT("={v[96:111]}"(st_a[0]), "={v[112:127]}"(st_a[1]), "={v[176:191]}"(pb_b))         \
                   : DLLM_STEP_IN("{v[128:143]}"(st_b[0]), "{v[144:159]}"(st_b[1]), "{v[160:175]}"(pb_a)),           \
                     DLLM_STEP_LOADS_SPLIT                                                                          \
                   : "memory", "m0", "scc", DLLM_DENSE_SCRATCH);                                                    \
    else if constexpr (AB)                                                                                          \
      asm volatile(DLLM_DENSE_STEP_##D##_AB                                                                         \
                   : DLLM_STEP_OUT("={v[128:143]}"(st_b[0]), "={v[144:159]}"(st_b[1]), "={v[160:175]}"(pb_a))        \
                   : DLLM_STEP_IN("{v[96:111]}"(st_a[0]), "{v[112:127]}"(st_a[1]), "{v[176:191]}"(pb_b)),            \
                     DLLM_STEP_LOADS                                                                                \
                   : "memory", "m0", "scc", DLLM_DENSE_SCRATCH);                                                    \
    else                                                                                                            \
      asm volatile(DLLM_DENSE_STEP_##D##_BA                                                                         \
                   : DLLM_STEP_OUT("={v[96:111]}"(st_a[0]), "={v[112:127]}"(st_a[1]), "={v[176:191]}"(pb_b))         \
                   : DLLM_STEP_IN("{v[128:143]}"(st_b[0]), "{v[144:159]}"(st_b[1]), "{v[160:175]}"(pb_a))            \
                   : "memory", DLLM_DENSE_SCRATCH);                                                                 \
  }

struct DenseState {
  static constexpr int kAcc = 128;   // accumulator registers
  f32x16 acc[8], q[4], st_a[2], st_b[2], kop[2], pb_a, pb_b;
  f32x4 ls[2];   // row sums (a-registers behind the queries, see above)
  v4u ones;
  float nmz[2], mx[2];   // v72, v73 (= -m z per block); v74, v75 (lane maxima of the newest scores)
  i32x16 addr;
#define DLLM_ACC_OUT                                                                                          \
  "={a[0:15]}"(acc[0]), "={a[16:31]}"(acc[1]), "={a[32:47]}"(acc[2]), "={a[48:63]}"(acc[3]),                  \
      "={a[64:79]}"(acc[4]), "={a[80:95]}"(acc[5]), "={a[96:111]}"(acc[6]), "={a[112:127]}"(acc[7])
#define DLLM_ACC_TIED "0"(acc[0]), "1"(acc[1]), "2"(acc[2]), "3"(acc[3]), "4"(acc[4]), "5"(acc[5]), "6"(acc[6]), "7"(acc[7])
#define DLLM_ACC_IN                                                                                           \
  "{a[0:15]}"(acc[0]), "{a[16:31]}"(acc[1]), "{a[32:47]}"(acc[2]), "{a[48:63]}"(acc[3]), "{a[64:79]}"(acc[4]), \
      "{a[80:95]}"(acc[5]), "{a[96:111]}"(acc[6]), "{a[112:127]}"(acc[7])
#define DLLM_Q_IN "{a[128:143]}"(q[0]), "{a[144:159]}"(q[1]), "{a[160:175]}"(q[2]), "{a[176:191]}"(q[3])
#define DLLM_STEP_OUT(st0, st1, pb) DLLM_ACC_OUT, st0, st1, pb, "={v[192:207]}"(kop[0]), "={v[208:223]}"(kop[1]), \
      DLLM_LS_OUT, "={v74}"(mx[0]), "={v75}"(mx[1]), [grow] "=s"(grow)
#define DLLM_STEP_IN(st0, st1, pb) DLLM_ACC_TIED, "11"(kop[0]), "12"(kop[1]), DLLM_LS_TIED("13", "14"),          \
      [ones] "v"(ones), "{v72}"(nmz[0]), "{v73}"(nmz[1]), DLLM_Q_IN, st0, st1, pb, "{v[80:95]}"(addr),             \
      [zs] "s"(zs), [lazy] "s"(kLazyGrowthDense), [koff] "n"(KOFF), [voff0] "n"(VOFF0), [voff1] "n"(VOFF1)
#define DLLM_STEP_LOADS [kt] "s"(tl.k), [vt] "s"(tl.v), [lo0] "v"(tl.off[0]), [lo1] "v"(tl.off[1]),                \
      [lo2] "v"(tl.off[2]), [lo3] "v"(tl.off[3]), [wl] "s"(tl.wave_lds), [lk] "n"(LK), [lv] "n"(LV)
#define DLLM_STEP_LOADS_SPLIT DLLM_STEP_LOADS, [vo0] "v"(tl.off_v[0]), [vo1] "v"(tl.off_v[1]),                     \
      [vo2] "v"(tl.off_v[2]), [vo3] "v"(tl.off_v[3])
  DLLM_STEP_FUNCTION(128)
#undef DLLM_STEP_OUT
#undef DLLM_STEP_IN
#undef DLLM_STEP_LOADS
#undef DLLM_STEP_LOADS_SPLIT
  // the closing P V product, with the probabilities of pb_a; `ad`: addr with the V row
  // offset added to the V^T operand addresses (it is not a compile-time constant here)
  __device__ __forceinline__ void tail(i32x16 ad) {
    asm volatile(DLLM_DENSE_TAIL_128
                 : DLLM_ACC_OUT, DLLM_LS_OUT
                 : DLLM_ACC_TIED, DLLM_LS_TIED("8", "9"), [ones] "v"(ones), "{v[160:175]}"(pb_a), "{v[80:95]}"(ad), [voff0] "n"(0), [voff1] "n"(16 * 256)
                 : "memory", DLLM_DENSE_SCRATCH);
  }
  // S^T(0) into st_a from the K operands in kop
  __device__ __forceinline__ void score0() {
    asm volatile(DLLM_DENSE_SCORE0_128
                 : "={v[96:111]}"(st_a[0]), "={v[112:127]}"(st_a[1])
                 : "{v[192:207]}"(kop[0]), "{v[208:223]}"(kop[1]), DLLM_Q_IN);
  }
  // waits for the K operands that the last step has requested (nothing may take their registers before)
  __device__ __forceinline__ void drain() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::"{v[192:207]}"(kop[0]), "{v[208:223]}"(kop[1]) : "memory");
  }
  __device__ __forceinline__ void row_sums(float& l0, float& l1) {
    asm volatile("s_nop 15\n\ts_nop 15\n\tv_accvgpr_read_b32 %0, a192\n\tv_accvgpr_read_b32 %1, a196"
                 : "=v"(l0), "=v"(l1) : "{a[192:195]}"(ls[0]), "{a[196:199]}"(ls[1]));
  }
  __device__ __forceinline__ void acc_clear() { asm volatile(DLLM_DENSE_ACC_INIT_128 : DLLM_ACC_OUT, DLLM_LS_OUT); }
  // acc[qb] *= al[qb]; waits out the matrix pipe first (results may be read only 12 wait states after the
  // MFMA was issued, and nothing but software enforces it)
  __device__ __forceinline__ void acc_scale(float al0, float al1) {
    asm volatile(DLLM_DENSE_ACC_SCALE_128 : DLLM_ACC_OUT, DLLM_LS_OUT : DLLM_ACC_TIED, DLLM_LS_TIED("8", "9"), [al0] "v"(al0), [al1] "v"(al1) : DLLM_DENSE_SCRATCH);
  }
  // all accumulators of block qb, head_dim block db, after the matrix pipe has drained
  __device__ __forceinline__ void acc_read(float (&x)[kAcc]) {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    asm volatile(DLLM_DENSE_ACC_READ_0 : DLLM_R16(0, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_1 : DLLM_R16(1, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_2 : DLLM_R16(2, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_3 : DLLM_R16(3, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_4 : DLLM_R16(4, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_5 : DLLM_R16(5, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_6 : DLLM_R16(6, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_7 : DLLM_R16(7, x) : DLLM_ACC_IN);
  }
#undef DLLM_ACC_OUT
#undef DLLM_ACC_TIED
#undef DLLM_ACC_IN
#undef DLLM_Q_IN
  // element access (indices are compile-time constants after unrolling)
  __device__ __forceinline__ void q_set(int qb, int t, int c, float x) { q[2 * qb + t / 4][4 * (t % 4) + c] = x; }
  __device__ __forceinline__ void kop_set(int t, int c, float x) { kop[t / 4][4 * (t % 4) + c] = x; }
};

// f(integral_constant<int, 0>), f(integral_constant<int, 1>), ... in order
template <typename F, int... C>
__device__ __forceinline__ void for_each_round(F& f, std::integer_sequence<int, C...>) {
  (f(std::integral_constant<int, C>{}), ...);
}

// KS: wave groups that share the keys (1 or 2; see launch_attend_dense_bf16 for which calls take which)
// which: 1 = only sequences flagged dense in seq_mode; 2 = every sequence
//
// With KS = 1 a launch has at most one workgroup per compute unit, and each goes on to further tiles by itself: between the
// last step over one tile's keys and the first over the next one's, a workgroup that ends and one that starts spent
// 0.3 us on the dispatch, 0.7 to 1.2 until the new one knew its place, 2.4 to 4.3 until its queries and first K rows were
// there, 0.9 to 1.2 until the first step and 2.7 to 3.7 on the last product, the outputs and their stores, while a step
// takes 0.7 to 0.9.  A workgroup that stays knows its next tile in advance and requests what it needs before the last product
// and the outputs: about 6 us instead of 10.  32 heads, eight sequences of 2048 467 -> 459 us, eight of 1024 132 -> 127, 8 KV heads
// and 21 sequences of 83 to 472 56.7 -> 53.3 (then 48.2 with fewer visits to the careful path, see `stop`; eighteen of 652
// 174 -> 163, twelve of 323 with 16 heads 32.5 -> 28.8).  Tiles are dealt out in serpentine order (turn r: tile 256 r + i to workgroup i or 255 - i, within each
// XCD), so that ragged batches, whose tiles come longest sequences first, stay even.
template <int KS>
__global__ __launch_bounds__(kDenseWaves * 64, 1) void attend_dense_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv, const uint8_t* __restrict__ seq_mode,
    int which, uint16_t* __restrict__ o, Shape s DLLM_CHECK_PARAM) {
  DLLM_CHECK_EXIT();
  constexpr int NQB = kDenseQB;
  constexpr int D = 128;
  constexpr int CH = D / 8;
  constexpr int ROWB = 2 * D;
  constexpr int TILEB = kDenseK * ROWB;
  constexpr int VBASE = kDenseRing * TILEB;      // V ring follows the K ring
  constexpr int NTHREADS = kDenseWaves * 64;
  constexpr int NT = D / 16;
  constexpr int NDB = D / 32;
  constexpr int SPT = 2 / KS;                    // steps a wave takes per tile
  constexpr int ROUND = SPT * kDenseRing;        // steps in one turn of the rings
  constexpr int AHEAD_K = KS == 1 ? 2 : 4;       // a tile's first step requests the K rows of the tile this far ahead,
  constexpr int AHEAD_V = 2;                     // and the V rows of this one
  constexpr int kDenseRows = dense_rows(KS);
  static_assert(NLD * NTHREADS == kDenseK * CH, "the loads of a tile");
  static_assert(kDenseRing * TILEB <= 65536, "ring offsets must fit the 16-bit LDS offset field");
  static_assert(kDenseQB * 32 == kDenseK, "a wave's queries fill one slot");

  // K ring, V ring, and space for the queries that have no ring slot to come through (see below)
  constexpr int kSlots = 2 * kDenseRing + (KS == 1 ? 2 : 1);
  __shared__ __attribute__((aligned(16))) char smem[kSlots * TILEB];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int hf = lane >> 5;
  // the query blocks this wave takes, and which half of every tile's keys (0 when all waves take both)
  const int qwave = KS == 1 ? wave : wave & 1;
  const int part = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave >> 1);
  const int64_t pitch = s.kv_tok * 2, tile_bytes = int64_t(kDenseK) * pitch;

  // ---- the query tiles this workgroup takes
  DenseLanes lanes;
  DensePlace at;
  const bool stays = KS == 1 && gridDim.x == kDenseUnits && gridDim.y == 1 && gridDim.z == 1;
  uint32_t turn = 0;
  // the next tile with keys; outputs of sequences without any are zeros
  auto find = [&](DensePlace& p) __attribute__((always_inline)) -> bool {
    for (;;) {
      const uint32_t n = blockIdx.x;
      uint32_t mine = n;
      if (stays) mine = turn * kDenseUnits + ((turn & 1) != 0 ? (kDenseUnits / 8 - 1 - (n >> 3)) * 8 + (n & 7) : n);
      else if (turn != 0) return false;
      ++turn;
      if (!find_dense(s, lanes, mine, p)) return false;
      if (p.L != 0) return true;
      zero_dense_rows<D>(p.qtile * kDenseRows, kDenseRows, p, s.hq, o);
    }
  };
  if (gridDim.y == 1 && gridDim.z == 1) {
    lanes = gather_dense<kDenseRows>(s, cu_q, cu_kv, seq_mode, which);
    if (!find(at)) return;
  } else {
    if (!place_dense_grid<kDenseRows>(s, cu_q, cu_kv, seq_mode, which, at)) return;
    if (at.L == 0) {
      zero_dense_rows<D>(at.qtile * kDenseRows, kDenseRows, at, s.hq, o);
      return;
    }
  }

  // ---- what one tile's loads need.  Global side of the tile loads: this lane's chunk f = i * NTHREADS + tid of a K or V
  // tile lands at LDS byte 16 * f, i.e. row f / CH, chunk slot f % CH, and must hold chunk (slot ^ swizzle(row)) of
  // that row.  Rows past the end of the sequence re-read its last row (their keys are masked).
  uint32_t ld_off[NLD];   // byte offset of the chunk from the tile's first row (fits: checked on the host)
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int f = i * NTHREADS + tid, row = f / CH;
    ld_off[i] = uint32_t(row) * uint32_t(pitch) + uint32_t(((f % CH) ^ tile_swz<D>(row)) << 4);
  }
  // What is computed from the result cannot be moved out of the loop over tiles, where it would hold registers that the
  // steps do not leave (some twenty values went to scratch memory, whose loads wait for the tiles requested before them).
  auto anew = [](int x) __attribute__((always_inline)) -> int {
    asm volatile("" : "+v"(x));
    return x;
  };
  struct Keys {
    const char *k, *v;           // the sequence's first K and V row of this head
    int ntiles;
    uint32_t off_last[NLD];      // the offsets for the last tile, which the sequence may end inside of
  };
  auto keys_of = [&](const DensePlace& p) __attribute__((always_inline)) -> Keys {
    Keys x;
    const int mine = anew(tid);
    const int64_t first = int64_t(p.kv0) * s.kv_tok + int64_t(p.h / s.group) * s.kv_head;
    x.k = reinterpret_cast<const char*>(k + first);
    x.v = reinterpret_cast<const char*>(v + first);
    x.ntiles = (p.L + kDenseK - 1) / kDenseK;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int f = i * NTHREADS + mine, row = min(f / CH, p.L - 1 - (x.ntiles - 1) * kDenseK);
      x.off_last[i] = uint32_t(row) * uint32_t(pitch) + uint32_t(((f % CH) ^ tile_swz<D>(f / CH)) << 4);
    }
    return x;
  };
  // this wave's slice of each load round, as an LDS byte address
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(lds_addr(smem) + wave * 64 * 16);
  // (past the last tile the last one again, so that the number of loads in flight is always the same)
  auto load_tile = [&](const Keys& x, const char* base, int tile, auto lds_off) __attribute__((always_inline)) {
    constexpr int kLdsOff = decltype(lds_off)::value;
    const int t = min(tile, x.ntiles - 1);
    const char* tbase = base + t * tile_bytes;
    auto round = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      load16_to_lds<kLdsOff + i * NTHREADS * 16>(tbase, t == x.ntiles - 1 ? x.off_last[i] : ld_off[i], wave_lds);
    };
    for_each_round(round, std::make_integer_sequence<int, NLD>{});
  };
  // The wave's 64 query rows go through LDS, into ring slots that no tile needs yet and the slots behind the rings:
  // read straight into the operand layout, an instruction touches 32 rows of 32 bytes each, and the sixteen of them took
  // 3200 to 5200 cycles to issue.  Rows past the last query repeat it (their columns are never stored).
  const int qslot = KS == 1 ? (wave < 2 ? 2 + wave : 2 * kDenseRing - 2 + wave) : (qwave == 0 ? kDenseRing + 2 : 2 * kDenseRing);
  constexpr int NQLD = CH / KS;   // loads of 1 KB: with KS = 2 each wave of a pair that shares the queries brings half
  auto load_queries = [&](const DensePlace& p) __attribute__((always_inline)) {
    const uint32_t stage = __builtin_amdgcn_readfirstlane(lds_addr(smem) + qslot * TILEB + part * NQLD * 1024);
    // The rows of load i from the wave's first one on; their 16-byte chunk's swizzle depends on i % 4.
    const int mine = anew(lane), first = __builtin_amdgcn_readfirstlane(p.qtile * kDenseRows + qwave * 64 + part * NQLD * 4);
    const int row = mine / CH, left = p.nq - first;
    static_assert(64 / CH == 4, "four rows per load");
    const char* qh = reinterpret_cast<const char*>(q + int64_t(p.q0 + first) * s.q_tok + int64_t(p.h) * s.q_head);
    const int64_t qpitch = s.q_tok * 2;
    if (left >= NQLD * 4 && qpitch < (int64_t(1) << 30)) {
      auto round = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        load16_to_lds<i * 1024>(qh + i * 4 * qpitch, uint32_t(row) * uint32_t(qpitch) + (((mine % CH) ^ tile_swz<D>(i * 4 + row)) << 4), stage);
      };
      for_each_round(round, std::make_integer_sequence<int, NQLD>{});
      return;
    }
    auto round = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      const int r = i * 4 + row;
      load16_to_lds<i * 1024>(qh + min(r, left - 1) * qpitch + (((mine % CH) ^ tile_swz<D>(r)) << 4), stage);
    };
    for_each_round(round, std::make_integer_sequence<int, NQLD>{});
  };
#define DLLM_IC(x) std::integral_constant<int, (x)> {}

  DenseState w;
  const float zscale = s.scale * kLog2e;   // > 0; scores * zscale are base-2 logits
  // A operands of one step's score chain: rows = 32 keys at byte offset `koff` of the K ring
  auto k_operands = [&](int koff) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const v4u x = *reinterpret_cast<const v4u*>(smem + w.addr[t] + koff);
      w.kop_set(t, 0, __uint_as_float(x.x));
      w.kop_set(t, 1, __uint_as_float(x.y));
      w.kop_set(t, 2, __uint_as_float(x.z));
      w.kop_set(t, 3, __uint_as_float(x.w));
    }
  };
  auto mask_tail = [&](f32x16 (&st)[NQB], int nvalid) __attribute__((always_inline)) {   // keys past the end get no weight
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = 8 * (i / 4) + 4 * hf + (i % 4);
        if (key >= nvalid) st[qb][i] = -INFINITY;
      }
  };
  // largest score of a step per lane (a query's scores sit in the lane pair l, l ^ 32)
  auto lane_max = [&](const f32x16& st) __attribute__((always_inline)) -> float {
    float mx = maximum(st[0], st[1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) mx = maximum(maximum(mx, st[i]), st[i + 1]);
    return mx;
  };

  // ---- the first tile's requests: K rows of the first scores and the queries, then the rest
  Keys keys = keys_of(at);
  load_tile(keys, keys.k, 0, DLLM_IC(0));
  if constexpr (KS == 2) load_tile(keys, keys.k, 1, DLLM_IC(TILEB));
  load_queries(at);
  if constexpr (KS == 1) {
    load_tile(keys, keys.k, 1, DLLM_IC(TILEB));
    load_tile(keys, keys.v, 0, DLLM_IC(VBASE));
    load_tile(keys, keys.v, 1, DLLM_IC(VBASE + TILEB));
  } else {
    load_tile(keys, keys.k, 2, DLLM_IC(2 * TILEB));
    load_tile(keys, keys.v, 0, DLLM_IC(VBASE));
  }
  // Iteration 0 multiplies an all-zero P with the rows of ring slot 3 of V that the step "before the first" would
  // have used (the second half of the slot, or both halves when the keys are split): clear them, so that no stale
  // NaN pattern meets the zeros.  Tile 3 lands there later.
  {
    constexpr int kFrom = KS == 1 ? 32 * ROWB : 0;
    for (int e = kFrom + tid * 16; e < TILEB; e += NTHREADS * 16)
      *reinterpret_cast<v4u*>(smem + VBASE + 3 * TILEB + e) = v4u{0u, 0u, 0u, 0u};
  }

  for (;;) {   // over query tiles
    const int L = at.L, ntiles = keys.ntiles, qbase = at.qtile * kDenseRows;
    const int nsteps = KS == 1 ? (L + 31) / 32 : ntiles;
    // valid keys of this wave's last step: 32, or fewer when the sequence ends inside it (none at all is possible for
    // the second half of a tile)
    const int last_valid = KS == 1 ? L - 32 * (nsteps - 1) : max(0, min(32, L - kDenseK * (ntiles - 1) - 32 * part));
    // per query (lane pair l, l ^ 32): -m * z for the running maximum m of the raw scores (w.nmz), the factor
    // the accumulators (outputs and row sums) still have to take, and the accumulators
    float palpha[NQB];
    uint32_t pending = 0;   // 1: some palpha != 1 (uniform)
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) palpha[qb] = 1.0f;
    w.acc_clear();
    // LDS addresses, fixed for the whole pass; ring slot, 32-key half and 16-key quarter are immediates
    KAddr<D> kaddr;
    {
      const int mine = anew(lane);
      kaddr.init(mine);
      VtAddr<D> vaddr;
      vaddr.init(mine);
#pragma unroll
      for (int i = 0; i < 16; ++i) w.addr[i] = 0;
#pragma unroll
      for (int t = 0; t < NT; ++t) w.addr[t] = kaddr.off(t) + part * 32 * ROWB;
#pragma unroll
      for (int rd = 0; rd < 2; ++rd)
#pragma unroll
        for (int db = 0; db < NDB; ++db) w.addr[8 + NDB * rd + db] = VBASE + vaddr.off(rd, db) + part * 32 * ROWB;
      const uint32_t one2 = (mine & 31) == (mine & 4 ? 20 : 0) ? 0x3f803f80u : 0u;   // rows 0 and 4, see DLLM_LS_OUT
      w.ones = v4u{one2, one2, one2, one2};
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) w.pb_a[i] = w.pb_b[i] = 0.0f;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int i = 0; i < 16; ++i) w.st_b[qb][i] = 0.0f;
    // What the first step of each tile needs to request the tile two ahead (see the step text).  Past
    // the last tile the last one is requested again, into a ring slot nobody reads any more.
    DenseTileLoad tl;
    tl.wave_lds = wave_lds;
    int64_t advance_k, advance_v;   // what the pointers move by after a tile's first step; 0 once they reached the last tile
    auto aim_loads = [&](int tile) __attribute__((always_inline)) {   // for the requests of `tile`'s first step
      const int tk = min(tile + AHEAD_K, ntiles - 1), tv = min(tile + AHEAD_V, ntiles - 1);
      advance_k = tk < ntiles - 1 ? tile_bytes : 0;
      advance_v = tv < ntiles - 1 ? tile_bytes : 0;
      tl.k = keys.k + tk * tile_bytes;
      tl.v = keys.v + tv * tile_bytes;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        tl.off[i] = tk == ntiles - 1 ? keys.off_last[i] : ld_off[i];
        if constexpr (KS == 2) tl.off_v[i] = tv == ntiles - 1 ? keys.off_last[i] : ld_off[i];
      }
    };
    aim_loads(0);

    // The first scores need the queries and the K rows requested before them; the three (KS = 2: two) tiles requested after
    // those stay in flight (the first step waits for them, see its text).  Stores of the previous tile's outputs may have
    // been issued behind them: operations complete in order, so that is only a longer wait.
    wait_tile_loads_but<(KS == 1 ? 3 : 2) * NLD>();
    __syncthreads();
    // Q^T operands: lane (col = query, hf) holds Q[query][16t + 8hf .. +8) for every step t, as given
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const v4u x = *reinterpret_cast<const v4u*>(smem + qslot * TILEB + qb * 32 * ROWB + kaddr.off(t));
        w.q_set(qb, t, 0, __uint_as_float(x.x));
        w.q_set(qb, t, 1, __uint_as_float(x.y));
        w.q_set(qb, t, 2, __uint_as_float(x.z));
        w.q_set(qb, t, 3, __uint_as_float(x.w));
      }

    // scores of step 0, its maxima outright (they may be negative)
    k_operands(0);
    w.score0();
    if (nsteps == 1 && last_valid < 32) mask_tail(w.st_a, last_valid);
    const bool no_keys = KS == 2 && nsteps == 1 && last_valid == 0;   // this wave pair's half of the only tile is empty
    // (no lower than the lowest finite number: keys whose scores overflowed to minus infinity weigh nothing instead of
    // (-inf) - (-inf), also when they fill the first step)
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const float mx = maximum_across_halves(lane_max(w.st_a[qb])), mz = maximum(mx * zscale + kDenseHeadroom, -FLT_MAX);
      const bool lost = is_lost(mx, zscale, mz);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(lost) != 0, 0)) {
        drop_scores(w.st_a[qb], lost);
        if (lost) palpha[qb] = NAN;
        pending = 1;
      }
      w.nmz[qb] = no_keys ? 0.0f : lost ? FLT_MAX : -mz;
    }
    if constexpr (KS == 2) {   // what a step before the first would have requested, so that every step finds the same in flight
      load_tile(keys, keys.k, 3, DLLM_IC(3 * TILEB));
      load_tile(keys, keys.v, 1, DLLM_IC(VBASE + TILEB));
    }
    k_operands(KS == 1 ? 32 * ROWB : TILEB);   // step 1 (stale LDS if there is none; then unused)
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0) here, or the compiler waits for all LDS reads at every turn of the loop

    // Iteration j at position R = j % ROUND of the ring turn, which fixes every LDS offset.  Between two steps the common
    // path is one test and, after the first step of a tile, the advance of the tile pointers; everything else (the end of
    // the sequence, the ragged last step, a running maximum to raise, accumulators that still owe a factor) sits behind
    // that test.  `stop` is the number of steps done when the careful path is due without such a reason: when the next
    // tile to begin requests the last one, when the next step is a ragged last one, and at the end.  (Once the loads aim
    // at the last tile they stay there.  A visit costs some 280 cycles, and 1100 where it scales the accumulators; every step of the last one or two ring turns
    // used to make one, and a ragged last step scaled them by 1.)
    int j = 0;        // steps done
    int jb = 0;       // steps done at the start of the current ring turn
    const int aim_v = SPT * (ntiles - 1 - AHEAD_V) - (SPT - 1);   // ... for V rows, which the split form requests later
    int stop = SPT * (ntiles - 1 - AHEAD_K) - (SPT - 1);
    int left = 0;     // steps of this ring turn, and jb before it, that the common path may still take: stop - 1 - jb
    // ring offset of the rows of the step at ring position r
    constexpr auto step_off = [](int r) constexpr { return (r / SPT) * TILEB + (r % SPT) * 32 * ROWB; };
    // one step at ring position R (the text, with every offset it needs)
#define DLLM_RUN_STEP(R, grow)                                                                                  \
  w.template step<(R) % 2 == 0, KS == 2, step_off(((R) + 2) % ROUND), step_off(((R) + ROUND - 1) % ROUND),        \
                  step_off(((R) + ROUND - 1) % ROUND) + 16 * ROWB, (((R) / SPT + AHEAD_K) % kDenseRing) * TILEB,  \
                  VBASE + (((R) / SPT + AHEAD_V) % kDenseRing) * TILEB>(zscale, tl, grow)
    // what may need doing after step number j - 1 (at ring position R); true when the sequence is finished
    auto careful = [&](auto rc, uint64_t grow) __attribute__((always_inline)) -> bool {
      constexpr int R = decltype(rc)::value;
      if (pending) {   // hand the accumulators the factor they still owe
        w.acc_scale(palpha[0], palpha[1]);
        palpha[0] = palpha[1] = 1.0f;
        pending = 0;
      }
      if (j >= nsteps) return true;
      // tile requests near the end: the pointers stop at the last tile, whose rows may end early
      aim_loads((j + SPT - 1) / SPT);   // the next boundary is the first step of this tile
      // Keys past the end were scored from copies of the last row (the tile loads clamp the row), so they carry that
      // row's score and the lane maxima need no second look after masking.
      const int last_due = last_valid < 32 ? nsteps - 1 : nsteps;
      if (j == last_due) {
        if constexpr (R % 2 == 0) mask_tail(w.st_b, last_valid);
        else mask_tail(w.st_a, last_valid);
      }
      if (j >= stop) {
        stop = j < aim_v ? aim_v : j < last_due ? last_due : nsteps;
        left = stop - 1 - jb;
      }
      // Raise the running maxima for the scores of step j; before a ragged last step (last_due is nsteps otherwise, which j
      // is not here) always, since a key that sets its query's maximum has a probability that bf16 holds exactly.  Leaving
      // that out saved 0.9 us a call (eight heads, three sequences of 78 9.7 -> 8.8, 32 heads, 38 of 155 63.8 -> 59.9), but put
      // ragged batches further from 64 bits (six of 300 to 1500, 32 heads over 8 2.3206 -> 2.3259e-3).
      if (grow != 0 || j == last_due) {
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const float mz_old = -w.nmz[qb], mx = maximum_across_halves(w.mx[qb]);
          const float mz_new = maximum(mz_old, mx * zscale + kDenseHeadroom);
          const bool lost = is_lost(mx, zscale, mz_new);
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(lost) != 0, 0))
            drop_scores(R % 2 == 0 ? w.st_b[qb] : w.st_a[qb], lost);
          const float alpha = __builtin_amdgcn_exp2f(mz_old - mz_new);
          palpha[qb] = lost ? NAN : alpha;
          if (!lost) w.nmz[qb] = -mz_new;
        }
        pending = 1;
      }
      return false;
    };
#define DLLM_STEP(R)                                         \
  {                                                          \
    uint64_t grow;                                           \
    DLLM_RUN_STEP(R, grow);                                  \
    if ((R) % SPT == 0) {                                    \
      tl.k += advance_k;                                     \
      tl.v += advance_v;                                     \
    }                                                        \
    if (__builtin_expect((uint32_t(grow) | uint32_t(grow >> 32) | pending | uint32_t(left - (R) - 1) >> 31) != 0, 0)) { \
      j = jb + (R) + 1;                                      \
      if (careful(DLLM_IC(R), grow)) break;                  \
    }                                                        \
  }
    for (;;) {
      left = stop - 1 - jb;
      DLLM_STEP(0)
      DLLM_STEP(1)
      DLLM_STEP(2)
      DLLM_STEP(3)
      if constexpr (ROUND == 8) {
        DLLM_STEP(4)
        DLLM_STEP(5)
        DLLM_STEP(6)
        DLLM_STEP(7)
      }
      jb += ROUND;
    }
#undef DLLM_STEP
#undef DLLM_RUN_STEP
    w.drain();
    const DensePlace done = at;
    const bool more = stays && find(at);
    wait_tile_loads();   // the requests past the last tile still write to the rings
    __syncthreads();     // every wave is past its last K operands: the K ring is free
    if (more) {
      keys = keys_of(at);
      load_tile(keys, keys.k, 0, DLLM_IC(0));
      load_queries(at);
      load_tile(keys, keys.k, 1, DLLM_IC(TILEB));
    }
    // the last step's P V product: its probabilities are in pb_a after an odd number of steps, else in pb_b
    {
      const int last = nsteps - 1;
      const int voff = (last / SPT % kDenseRing) * TILEB + (last % SPT) * 32 * ROWB;
      i32x16 ad = w.addr;
#pragma unroll
      for (int i = 8; i < 16; ++i) ad[i] += voff;
      // (One tail for both cases, after moving sixteen registers: with a tail in either arm of a branch the
      // compiler carries all accumulators through vector registers and back where the arms meet, 2500 of the
      // 2900 cycles from the last step to the stores.)
      if (!(nsteps & 1)) w.pb_a = w.pb_b;
      w.tail(ad);
    }
    __syncthreads();     // ... and its last V rows: the V ring is free
    if (more) {
      load_tile(keys, keys.v, 0, DLLM_IC(VBASE));
      load_tile(keys, keys.v, 1, DLLM_IC(VBASE + TILEB));
    }
    float accv[DenseState::kAcc];   // [qb][db][16]
    w.acc_read(accv);
    float lrow[NQB];
    w.row_sums(lrow[0], lrow[1]);   // lanes 0..31: the query's sum; lanes 32..63: zero
    if constexpr (KS == 1) {
      // 32 rows of each wave at a time, through V ring slots 2 and 3
      char* stage = smem + VBASE + 2 * TILEB + wave * 32 * ROWB;
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
        store_dense_block<D>(accv + 16 * NDB * qb, sum_across_halves(lrow[qb]), stage, qbase + (wave * NQB + qb) * 32, done, s.hq, o);
    } else {
      static_assert(NQB == 2 && kDenseWaves == 4, "two wave pairs, two blocks each");
      static_assert(dense_merge_bytes<D>() <= 2 * kDenseRing * TILEB, "merge space");
      const float m[2] = {no_keys ? -INFINITY : -w.nmz[0], no_keys ? -INFINITY : -w.nmz[1]};
      merge_dense_halves<D>(accv, lrow, m, part, smem, qbase + qwave * NQB * 32, done, s.hq, o);
    }
    if (!more) break;
    // the rows that the next iteration 0 multiplies by zeros: the last wave's outputs came through them
    static_assert(kDenseWaves == 4, "the last wave stages its outputs in the second half of V ring slot 3");
    order_wave_lds();
    if (wave == kDenseWaves - 1)
#pragma unroll
      for (int i = 0; i < 32 * ROWB / 1024; ++i)
        *reinterpret_cast<v4u*>(smem + VBASE + 3 * TILEB + 32 * ROWB + (i * 64 + lane) * 16) = v4u{0u, 0u, 0u, 0u};
  }
}

// Whether a call splits every tile's keys between two wave pairs (2) or not (1).  The split form makes twice the
// workgroups, each half as long, for a call that would leave compute units idle; it costs a sixth more per score (every
// step requests a tile) and the same start and end per workgroup.  Measured (us, whole / split): 32 heads x 128, one
// sequence of 256 14.6 / 11.3, 512 19.6 / 15.0, 1024 29.7 / 24.6 (half the compute units); 2048 65.6 / 75.4 (all of them);
// three of 768 53.7 / 57.9 (two rounds against three); five of 300 35.4 / 27.1.
// head_dim 128, in shader cycles from the clock at the marks of both forms: 1440 per step and 13000 besides (split:
// 1660); one workgroup runs per compute unit at a time.  (Since workgroups stay for further tiles and the end of a sequence
// costs less, a step takes 1290 to 1460 and a further tile about 10000; over 80 batches measured in both forms since the
// choice is 0.2 % above the better one in the mean, 5 % at most.)
// head_dim 64 (two workgroups per compute unit), in ns, fitted to 101 batches measured in both forms (4 to 32 heads, one to 40
// sequences of 64 to 6000): a step takes 449 (split: 485) on a compute unit that the workgroup has for itself and 500 (525)
// of a shared one, where a workgroup costs 1000 (1500) besides; 3000 before the first step.  Ragged batches of up to 512
// workgroups keep the whole form unless the split one is estimated 1.3 times as fast: there the estimate knows least
// (8 heads, nine of 209 to 1073 22.5 / 19.3, six of 567 to 1601 29.8 / 28.3, thirteen of 370 to 446 13.8 / 14.1; with one
// wave per SIMD, as this kernel used to be, 21 to 23.5 / 25.2, 31.1 / 33.9, 14.9 / 21.0).  Over those batches the choice is 0.7 % above
// the better form in the mean (the whole form always: 11.6 %, the split one: 2.8 %).  16 heads: nine of 416 18.5 /
// 20.9, three of 600 15.3 / 11.6, four of 2048 70.0 / 74.6, two of 4400 190 / 176.  Even batches need
// the split form 3 % ahead and ragged ones beyond 512 workgroups 5 %: the two estimates came that near each other where the
// whole form is 3 to 13 % faster (8 heads, nineteen of 459 21.8 / 22.9; 32 heads, ten of 1183 to 1494 172 / 188, twenty of
// 580 to 628 88.7 / 96.0; 16 heads, seven of 537 to 2076 65.4 / 67.8, of 448 to 1804 65.5 / 68.3, of 422 to 2925 68.2 / 72.7, of 783 to 2873 99.9 / 106.8);
// not where most sequences fill no more than a split workgroup (32 heads, 25 of 70 to 133 19.3 / 17.6).
// The lengths themselves are on the device.  With the mean and the longest known, they are taken to be spread evenly
// around the mean (up to 64 of them, for the batch), and the workgroups to start longest first: at head_dim 128, in a second
// round that is not full, a workgroup then follows one of about the length at which the first round ended.  Counting such
// a round by its share of the mean instead took the split form where it loses (8 heads x 128, fifteen of 109 to 834 29.2 /
// 32.1).  More than a round is estimated to within a few per cent, so there the split form has to be 6 % ahead (of 1500
// simulated batches 3 then lose more than 2 %, 14 without).
int dense_key_splits(const Shape& s, int which) {
  constexpr int kUnits = 256;   // compute units
  // the densely attended sequences of a mixed call are not known here: as many as total_q can have of the longest
  const int64_t n = which == 2 ? s.batch : std::max<int64_t>(1, (int64_t(s.total_q) + s.max_q - 1) / s.max_q);
  const double longest_q = s.max_q, mean_q = double(s.total_q) / n;
  const double longest_kv = which == 2 ? s.max_kv : std::min(s.max_kv, s.max_q);
  const double mean_kv = which == 2 ? double(s.total_kv) / n : std::min(longest_kv, mean_q);
  const bool even = mean_kv * 8 >= longest_kv * 7 && mean_q * 8 >= longest_q * 7;
  const int reps = int(std::min<int64_t>(n, 64));
  const bool shared = s.d == 64;   // two workgroups per compute unit
  auto cost = [&](int ks) -> double {
    const double step = shared ? (ks == 1 ? 500 : 525) : (ks == 1 ? 1440 : 1660);
    const double fixed = shared ? (ks == 1 ? 1000 : 1500) : 13000, start = shared ? 3000 : 0;
    const double per_key = step / (32 * ks), one = longest_kv * per_key + fixed;
    double workgroups = 0, work = 0, second = 0;   // second: what the first workgroup of the second round takes
    for (int i = 0; i < reps; ++i) {
      const double t = reps > 1 ? 2.0 * i / (reps - 1) : 0.0;
      const double q = std::max(1.0, longest_q - (longest_q - mean_q) * t), kv = std::max(1.0, longest_kv - (longest_kv - mean_kv) * t);
      const double k = double(n) / reps * s.hq * std::ceil(q / dense_rows(ks)), length = kv * per_key + fixed;
      if (workgroups <= kUnits && workgroups + k > kUnits) second = length;
      workgroups += k;
      work += k * length;
    }
    if (shared) {
      const double alone = longest_kv * (ks == 1 ? 449 : 485) / (32 * ks) + 1000;
      if (workgroups <= kUnits) return start + alone;
      if (even) return (ks == 2 ? 1.03 : 1.0) * (start + std::ceil(workgroups / kUnits) * one);
      if (workgroups <= 2 * kUnits) return (ks == 2 ? 1.3 : 1.0) * (start + std::max(alone, work / kUnits));
      return (ks == 2 && mean_q > dense_rows(2) ? 1.05 : 1.0) * (start + std::max(one, work / kUnits + work / workgroups / 2));
    }
    if (workgroups <= kUnits) return one;
    const double doubt = ks == 2 ? 1.06 : 1.0;
    if (even) return doubt * std::ceil(workgroups / kUnits) * one;   // equal workgroups: whole rounds
    if (workgroups <= 2 * kUnits) return doubt * std::max(one, 2 * second);
    return doubt * std::max(one, work / kUnits + work / workgroups / 2);
  };
  return cost(2) < cost(1) ? 2 : 1;
}

hipError_t launch_attend_dense_bf16(const Shape& s, const void* q, const void* k, const void* v,
                                    const int32_t* cu_q, const int32_t* cu_kv, const uint8_t* seq_mode, int which,
                                    void* o, hipStream_t st) {
  if (s.max_q == 0) return hipSuccess;   // no sequence has a query: nothing to write
  const int ks = dense_key_splits(s, which);
  const int rows = dense_rows(ks);
  const int64_t nx = (s.max_q + rows - 1) / rows;
  dim3 grid(unsigned(nx), s.hq, s.batch);
  if (s.batch <= 64) {
    // the workgroups place themselves (see the kernel): as many as the batch can have query tiles, times the heads
    const int64_t tiles = std::min<int64_t>(int64_t(s.total_q) / rows + s.batch, nx * s.batch);
    if (tiles * s.hq < (int64_t(1) << 31)) grid = dim3(unsigned(tiles * s.hq), 1, 1);
    // at head_dim 128 workgroups stay for further tiles (see the kernel)
    if (s.d == 128 && ks == 1 && grid.y == 1 && grid.z == 1) grid.x = std::min(grid.x, unsigned(kDenseUnits));
  }
  auto launch = [&](auto kernel) -> hipError_t {
    kernel<<<grid, kDenseWaves * 64, 0, st>>>(static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),
                                              static_cast<const uint16_t*>(v), cu_q, cu_kv, seq_mode, which,
                                              static_cast<uint16_t*>(o), s DLLM_CHECK_PASS);
    return hipGetLastError();
  };
  if (s.d == 64) return launch_attend_dense_paired(s, ks, grid, q, k, v, cu_q, cu_kv, seq_mode, which, o, st);
  return ks == 2 ? launch(attend_dense_bf16_kernel<2>) : launch(attend_dense_bf16_kernel<1>);
}

}  // namespace dllm
