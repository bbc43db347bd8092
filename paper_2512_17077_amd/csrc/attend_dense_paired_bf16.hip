// Refresh-phase attention at head_dim 64 with two waves per SIMD (bf16 inputs, fp32 softmax state and accumulators).
//
// At head_dim 64 a 32-key step of 64 queries needs 576 cycles of the matrix pipe and about 780 of the vector units (32
// exponentials take 512), and a wave that is alone on its SIMD issues both, its LDS reads and its scalar instructions one
// after the other and sits out every wait: 1070 to 1165 cycles per step.  Here a wave keeps its 64 queries (an LDS
// operand read still feeds two products) but lives in half of the registers, so two workgroups of four waves share a
// compute unit: one wave's matrix and LDS instructions, waits, start and end run beside the other's vector work.
// What makes it fit:
//   - probabilities overwrite the scores they come from, and are multiplied with V in the step that makes them;
//   - K and V^T operands take turns in four buffers of four a-registers, which LDS reads fill directly;
//   - registers are split evenly, 128 v and 128 a, which is how this compiler divides a budget of 256.
// Everything else is as in attend_dense_bf16.hip: the step text comes from the same generator, K/V tiles of 64 keys go
// straight into LDS rings of four (64 KB per workgroup) and are requested three tiles ahead, the running maximum is
// raised lazily, row sums are matrix products, queries and outputs pass through LDS in whole rows.
#include <cfloat>
#include <type_traits>
#include <utility>

#include "attend_dense.h"
#include "attend_dense_step.inc"

namespace dllm {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

constexpr int D = 64;
constexpr int kWaves = 4;
constexpr int rows_of(int ks) { return kWaves * 64 / ks; }   // query rows per workgroup
constexpr int kRing = 4;                        // K tiles, and V tiles, resident in LDS
constexpr int CH = D / 8, ROWB = 2 * D, TILEB = 64 * ROWB, VBASE = kRing * TILEB;
constexpr int kThreads = kWaves * 64;
constexpr int NLD = 64 * CH / kThreads;         // 16-byte loads per lane, tile and tensor
static_assert(NLD == 2 && kWaves * 64 * ROWB == 4 * TILEB, "the step text requests two rounds; the queries fill four ring slots");

// What a step requests: the first K and V row of the tiles (wave-uniform), the byte offset of each of this lane's 16-byte
// chunks from there, and the LDS address of this wave's slice of a load round.
struct TileLoads {
  const char *k, *v;
  uint32_t off[NLD], off_v[NLD];   // off_v: split form only (there K and V rows of different tiles are requested)
  uint32_t wave_lds;
};

// The state of a wave in the registers that the step text names:
//   a[0:63] acc  O^T accumulators [qb][db][16]     a[64:95] q  Q^T operands [qb][t][4]     a[96:103] ls  row sums [qb][4]
//   a[104:119] kop  operand buffers (between steps: K operands of the next score chain, on their way)
//   v48, v49 nmz (= -m z per block)   v50, v51 mx (lane maxima of the newest scores)   v52..v55 scratch
//   v[56:63] addr  LDS byte addresses: K operand [t], V^T operand [rd][db]     v[64:95], v[96:127] st_a, st_b  scores of
//   two consecutive steps, [qb][16]; a step leaves its probabilities in place of its scores
// As in attend_dense_bf16.hip the accumulators go from one assembly block to the next.
struct PairedState {
  f32x16 acc[4], q[2], st_a[2], st_b[2], kop;
  f32x4 ls[2];
  v4u ones;   // the A operand of the row sums
  float nmz[2], mx[2];
  i32x8 addr;

#define DLLM_ACC_OUT "={a[0:15]}"(acc[0]), "={a[16:31]}"(acc[1]), "={a[32:47]}"(acc[2]), "={a[48:63]}"(acc[3])
#define DLLM_ACC_TIED "0"(acc[0]), "1"(acc[1]), "2"(acc[2]), "3"(acc[3])
#define DLLM_ACC_IN "{a[0:15]}"(acc[0]), "{a[16:31]}"(acc[1]), "{a[32:47]}"(acc[2]), "{a[48:63]}"(acc[3])
#define DLLM_LS_OUT "={a[96:99]}"(ls[0]), "={a[100:103]}"(ls[1])
#define DLLM_STEP_OUT DLLM_ACC_OUT, DLLM_LS_OUT, "={a[104:119]}"(kop), "={v[64:79]}"(st_a[0]), "={v[80:95]}"(st_a[1]),  \
      "={v[96:111]}"(st_b[0]), "={v[112:127]}"(st_b[1]), "={v50}"(mx[0]), "={v51}"(mx[1]), [grow] "=s"(grow)
#define DLLM_STEP_IN DLLM_ACC_TIED, "4"(ls[0]), "5"(ls[1]), "6"(kop), "7"(st_a[0]), "8"(st_a[1]), "9"(st_b[0]),         \
      "10"(st_b[1]), "{v48}"(nmz[0]), "{v49}"(nmz[1]), "{a[64:79]}"(q[0]), "{a[80:95]}"(q[1]), [ones] "v"(ones), \
      "{v[56:63]}"(addr), [zs] "s"(zs), [lazy] "s"(kLazyGrowthDense), [koff] "n"(KOFF), [voff0] "n"(VOFF),               \
      [voff1] "n"(VOFF + 16 * ROWB)
#define DLLM_SCRATCH "v52", "v53", "v54", "v55"
#define DLLM_STEP_LOADS [kt] "s"(tl.k), [vt] "s"(tl.v), [lo0] "v"(tl.off[0]), [lo1] "v"(tl.off[1]),                 \
      [wl] "s"(tl.wave_lds), [lk] "n"(LK), [lv] "n"(LV)
  // One step; AB: scores in st_a (a tile's first step, if waves take both halves of it), otherwise in st_b.
  template <bool AB, bool Split, int KOFF, int VOFF, int LK, int LV>
  __device__ __forceinline__ void step(float zs, const TileLoads& tl, uint64_t& grow) {
    if constexpr (AB && Split)
      asm volatile(DLLM_DENSE_PAIRED_STEP_AB_SPLIT
                   : DLLM_STEP_OUT
                   : DLLM_STEP_IN, DLLM_STEP_LOADS, [vo0] "v"(tl.off_v[0]), [vo1] "v"(tl.off_v[1])
                   : "memory", "m0", "scc", DLLM_SCRATCH);
    else if constexpr (Split)
      asm volatile(DLLM_DENSE_PAIRED_STEP_BA_SPLIT
                   : DLLM_STEP_OUT
                   : DLLM_STEP_IN, DLLM_STEP_LOADS, [vo0] "v"(tl.off_v[0]), [vo1] "v"(tl.off_v[1])
                   : "memory", "m0", "scc", DLLM_SCRATCH);
    else if constexpr (AB)
      asm volatile(DLLM_DENSE_PAIRED_STEP_AB
                   : DLLM_STEP_OUT : DLLM_STEP_IN, DLLM_STEP_LOADS : "memory", "m0", "scc", DLLM_SCRATCH);
    else
      asm volatile(DLLM_DENSE_PAIRED_STEP_BA : DLLM_STEP_OUT : DLLM_STEP_IN : "memory", DLLM_SCRATCH);
  }
#undef DLLM_STEP_LOADS
  // The K operands of the rows at byte offset OFF of the K ring.  Like the accumulators, the buffers only ever go from one
  // assembly block to the next: between two steps their reads are still in flight, so nothing may copy them.
  template <int OFF>
  __device__ __forceinline__ void k_operands() {
    asm volatile(
        "ds_read_b128 a[104:107], %1 offset:%5\n\tds_read_b128 a[108:111], %2 offset:%5\n\t"
        "ds_read_b128 a[112:115], %3 offset:%5\n\tds_read_b128 a[116:119], %4 offset:%5\n\ts_waitcnt lgkmcnt(0)"
        : "={a[104:119]}"(kop) : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "n"(OFF) : "memory");
  }
  // waits for the operands that the last step has requested
  __device__ __forceinline__ void drain() { asm volatile("s_waitcnt lgkmcnt(0)" ::"{a[104:119]}"(kop) : "memory"); }
  // S^T(0) into st_a from the K operands in kop
  __device__ __forceinline__ void score0() {
    asm volatile(DLLM_DENSE_PAIRED_SCORE0
                 : "={v[64:79]}"(st_a[0]), "={v[80:95]}"(st_a[1])
                 : "{a[104:119]}"(kop), "{a[64:79]}"(q[0]), "{a[80:95]}"(q[1]));
  }
  __device__ __forceinline__ void acc_clear() { asm volatile(DLLM_DENSE_ACC_INIT_64 : DLLM_ACC_OUT, DLLM_LS_OUT); }
  // accumulators and row sums of block qb times al<qb>; waits out the matrix pipe first
  __device__ __forceinline__ void acc_scale(float al0, float al1) {
    asm volatile(DLLM_DENSE_PAIRED_ACC_SCALE
                 : DLLM_ACC_OUT, DLLM_LS_OUT
                 : DLLM_ACC_TIED, "4"(ls[0]), "5"(ls[1]), [al0] "v"(al0), [al1] "v"(al1)
                 : DLLM_SCRATCH);
  }
  __device__ __forceinline__ void row_sums(float& l0, float& l1) {
    asm volatile("s_nop 15\n\ts_nop 15\n\tv_accvgpr_read_b32 %0, a96\n\tv_accvgpr_read_b32 %1, a100"
                 : "=v"(l0), "=v"(l1) : "{a[96:99]}"(ls[0]), "{a[100:103]}"(ls[1]));
  }
#define DLLM_R16(k, x) "=v"(x[16 * (k) + 0]), "=v"(x[16 * (k) + 1]), "=v"(x[16 * (k) + 2]), "=v"(x[16 * (k) + 3]), \
      "=v"(x[16 * (k) + 4]), "=v"(x[16 * (k) + 5]), "=v"(x[16 * (k) + 6]), "=v"(x[16 * (k) + 7]),                  \
      "=v"(x[16 * (k) + 8]), "=v"(x[16 * (k) + 9]), "=v"(x[16 * (k) + 10]), "=v"(x[16 * (k) + 11]),               \
      "=v"(x[16 * (k) + 12]), "=v"(x[16 * (k) + 13]), "=v"(x[16 * (k) + 14]), "=v"(x[16 * (k) + 15])
  // all accumulators, [qb][db][16], after the matrix pipe has drained
  __device__ __forceinline__ void acc_read(float (&x)[64]) {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    asm volatile(DLLM_DENSE_ACC_READ_0 : DLLM_R16(0, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_1 : DLLM_R16(1, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_2 : DLLM_R16(2, x) : DLLM_ACC_IN);
    asm volatile(DLLM_DENSE_ACC_READ_3 : DLLM_R16(3, x) : DLLM_ACC_IN);
  }
#undef DLLM_R16
#undef DLLM_SCRATCH
#undef DLLM_STEP_IN
#undef DLLM_STEP_OUT
#undef DLLM_LS_OUT
#undef DLLM_ACC_IN
#undef DLLM_ACC_TIED
#undef DLLM_ACC_OUT
};

template <typename F, int... C>
__device__ __forceinline__ void for_each_round(F& f, std::integer_sequence<int, C...>) {
  (f(std::integral_constant<int, C>{}), ...);
}

#define DLLM_IC(x) std::integral_constant<int, (x)> {}

// KS: wave groups that share the keys (1 or 2), as in attend_dense_bf16.hip: with 2, wave pair 0 takes the first 32 keys
// of every tile and wave pair 1 the others.
template <int KS>
__global__ __launch_bounds__(kThreads, 2) void attend_dense_paired_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv, const uint8_t* __restrict__ seq_mode,
    int which, uint16_t* __restrict__ o, Shape s DLLM_CHECK_PARAM) {
  DLLM_CHECK_EXIT();
  constexpr int kRows = rows_of(KS);
  constexpr int SPT = 2 / KS;                  // steps a wave takes per tile
  constexpr int kRound = SPT * kRing;          // steps in one turn of the rings
  // A tile's first step requests the K rows of the tile kAheadK further on and the V rows of the one kAheadV further on:
  // K rows are read two steps before their products and V rows in the step of theirs, so those slots are free.
  constexpr int kAheadK = KS == 1 ? 3 : 4, kAheadV = 3;
  __shared__ __attribute__((aligned(16))) char smem[2 * kRing * TILEB];   // K ring, V ring
  DensePlace at;
  if (gridDim.y == 1 && gridDim.z == 1) {
    if (!find_dense(s, gather_dense<kRows>(s, cu_q, cu_kv, seq_mode, which), blockIdx.x, at)) return;
  } else if (!place_dense_grid<kRows>(s, cu_q, cu_kv, seq_mode, which, at)) {
    return;
  }
  const int L = at.L, qbase = at.qtile * kRows;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hf = lane >> 5;
  // the query blocks this wave takes, and which half of every tile's keys (0 when all waves take both)
  const int qwave = KS == 1 ? wave : wave & 1;
  const int part = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave >> 1);
  if (L == 0) {   // nothing to attend to
    zero_dense_rows<D>(qbase, kRows, at, s.hq, o);
    return;
  }
  const int64_t head = int64_t(at.h / s.group) * s.kv_head;
  const char* kbase = reinterpret_cast<const char*>(k + int64_t(at.kv0) * s.kv_tok + head);
  const char* vbase = reinterpret_cast<const char*>(v + int64_t(at.kv0) * s.kv_tok + head);
  const int64_t pitch = s.kv_tok * 2, tile_bytes = 64 * pitch;
  const int ntiles = (L + 63) / 64, nsteps = KS == 1 ? (L + 31) / 32 : ntiles;
  // valid keys of this wave's last step (the second half of a tile may have none)
  const int last_valid = KS == 1 ? L - 32 * (nsteps - 1) : max(0, min(32, L - 64 * (ntiles - 1) - 32 * part));
  const bool no_keys = KS == 2 && nsteps == 1 && last_valid == 0;

  // This lane's chunk f = i * kThreads + tid of a tile lands at LDS byte 16 * f, row f / CH, slot f % CH, and must hold
  // chunk (slot ^ swizzle(row)) of that row.  Rows past the end of the sequence re-read its last row.
  uint32_t ld_off[NLD], ld_off_last[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int f = i * kThreads + tid, row = f / CH;
    const uint32_t chunk = uint32_t(((f % CH) ^ tile_swz<D>(row)) << 4);
    ld_off[i] = uint32_t(row) * uint32_t(pitch) + chunk;
    ld_off_last[i] = uint32_t(min(row, L - 1 - (ntiles - 1) * 64)) * uint32_t(pitch) + chunk;
  }
  // What the next tile's first step requests.  Past the last tile the last one is requested again, into slots nobody
  // reads any more.
  TileLoads tl;
  tl.wave_lds = __builtin_amdgcn_readfirstlane(lds_addr(smem) + wave * 64 * 16);
  int64_t advance_k, advance_v;   // what the pointers move by after a tile's first step; 0 once they reached the last tile
  auto aim = [&](int tile_k, int tile_v) __attribute__((always_inline)) {
    const int tk = min(tile_k, ntiles - 1), tv = min(tile_v, ntiles - 1);
    advance_k = tk < ntiles - 1 ? tile_bytes : 0;
    advance_v = tv < ntiles - 1 ? tile_bytes : 0;
    tl.k = kbase + tk * tile_bytes;
    tl.v = vbase + tv * tile_bytes;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      tl.off[i] = tk == ntiles - 1 ? ld_off_last[i] : ld_off[i];
      if constexpr (KS == 2) tl.off_v[i] = tv == ntiles - 1 ? ld_off_last[i] : ld_off[i];
    }
  };
  auto request = [&](const char* base, int tile, auto lds_off) __attribute__((always_inline)) {
    constexpr int kLdsOff = decltype(lds_off)::value;
    const int t = min(tile, ntiles - 1);
    const char* row0 = base + t * tile_bytes;
    load16_to_lds<kLdsOff>(row0, t == ntiles - 1 ? ld_off_last[0] : ld_off[0], tl.wave_lds);
    load16_to_lds<kLdsOff + kThreads * 16>(row0, t == ntiles - 1 ? ld_off_last[1] : ld_off[1], tl.wave_lds);
  };

  // K rows of the first scores, then the queries (64 rows per wave or wave pair, into ring slots that no tile needs yet;
  // rows past the last query repeat it), then what else the first steps need
  request(kbase, 0, DLLM_IC(0));
  const char* qstage = smem + (KS == 1 ? (wave < 2 ? 2 + wave : kRing + wave) : (qwave == 0 ? 3 : kRing + 3)) * TILEB;
  constexpr int NQLD = CH / KS;   // loads of 1 KB: each wave of a pair that shares the queries brings half
  {
    const uint32_t stage = __builtin_amdgcn_readfirstlane(lds_addr(qstage) + part * NQLD * 1024);
    const uint16_t* qh = q + int64_t(at.q0) * s.q_tok + int64_t(at.h) * s.q_head;
    auto round = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      const int f = (part * NQLD + i) * 64 + lane, r = f / CH;
      const int qi = min(qbase + qwave * 64 + r, at.nq - 1);
      load16_to_lds<i * 1024>(qh + int64_t(qi) * s.q_tok + (((f % CH) ^ tile_swz<D>(r)) << 3), stage);
    };
    for_each_round(round, std::make_integer_sequence<int, NQLD>{});
  }
  if constexpr (KS == 1) {
    request(vbase, 0, DLLM_IC(VBASE));
    request(kbase, 1, DLLM_IC(TILEB));
    request(vbase, 1, DLLM_IC(VBASE + TILEB));
  } else {
    request(kbase, 1, DLLM_IC(TILEB));
    request(vbase, 0, DLLM_IC(VBASE));
    request(kbase, 2, DLLM_IC(2 * TILEB));
  }

  PairedState w;
  const float zscale = s.scale * kLog2e;   // > 0; scores * zscale are base-2 logits
  KAddr<D> kaddr;
  kaddr.init(lane);
  VtAddr<D> vaddr;
  vaddr.init(lane);
#pragma unroll
  for (int t = 0; t < 4; ++t) w.addr[t] = kaddr.off(t) + part * 32 * ROWB;
#pragma unroll
  for (int n = 0; n < 4; ++n) w.addr[4 + n] = VBASE + vaddr.off(n >> 1, n & 1) + part * 32 * ROWB;
  {
    const uint32_t one2 = (lane & 31) == (lane & 4 ? 20 : 0) ? 0x3f803f80u : 0u;   // rows 0 and 4
    w.ones = v4u{one2, one2, one2, one2};
  }
  w.acc_clear();
  auto mask_tail = [&](f32x16 (&st)[2]) __attribute__((always_inline)) {   // keys past the end get no weight
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i / 4) + 4 * hf + (i % 4) >= last_valid) st[qb][i] = -INFINITY;
  };
  auto lane_max = [&](const f32x16& st) __attribute__((always_inline)) -> float {
    float mx = maximum(st[0], st[1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) mx = maximum(maximum(mx, st[i]), st[i + 1]);
    return mx;
  };

  wait_tile_loads_but<3 * NLD>();   // the first K rows and the queries are in
  __syncthreads();
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const v4u x = *reinterpret_cast<const v4u*>(qstage + qb * 32 * ROWB + kaddr.off(t));
#pragma unroll
      for (int c = 0; c < 4; ++c) w.q[qb][4 * t + c] = __uint_as_float(x[c]);
    }
  w.k_operands<0>();
  w.score0();
  if constexpr (KS == 2) wait_tile_loads_but<2 * NLD>();   // K rows of step 1 are in
  __syncthreads();   // every wave has its queries: their slots are free
  if constexpr (KS == 1) {
    request(kbase, 2, DLLM_IC(2 * TILEB));
    request(vbase, 2, DLLM_IC(VBASE + 2 * TILEB));
  } else {   // what the two steps before the first would have requested last
    request(vbase, 1, DLLM_IC(VBASE + TILEB));
    request(kbase, 3, DLLM_IC(3 * TILEB));
    request(vbase, 2, DLLM_IC(VBASE + 2 * TILEB));
  }
  if (nsteps == 1 && last_valid < 32) mask_tail(w.st_a);
  // (no lower than the lowest finite number: keys whose scores overflowed to minus infinity weigh nothing instead of
  // (-inf) - (-inf), also when they fill the first step)
  bool lost[2];   // see is_lost
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float mx = maximum_across_halves(lane_max(w.st_a[qb])), mz = maximum(mx * zscale + kDenseHeadroom, -FLT_MAX);
    lost[qb] = is_lost(mx, zscale, mz);
    w.nmz[qb] = no_keys ? 0.0f : lost[qb] ? FLT_MAX : -mz;
  }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(lost[0] || lost[1]) != 0, 0)) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) drop_scores(w.st_a[qb], lost[qb]);
    w.acc_scale(lost[0] ? NAN : 1.0f, lost[1] ? NAN : 1.0f);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) w.st_b[0][i] = w.st_b[1][i] = 0.0f;
  w.k_operands<KS == 1 ? 32 * ROWB : TILEB>();   // step 1 (copies of the last row if there is none; then unused)
  aim(kAheadK, kAheadV);

  // Iteration j at position R = j % kRound of the ring turn, which fixes every LDS offset.  Between two steps the common
  // path is one test and, after a tile's first step, the advance of the tile pointers.  `stop` is the number of steps done
  // when the careful path is due although no score has outgrown its maximum: when the next tile to begin requests the last
  // one (once the loads aim at it they stay there), when the next step is a ragged last one, and at the end.
  int j = 0, jb = 0;   // steps done; steps done at the start of the current ring turn
  const int aim_v = SPT * (ntiles - 1 - kAheadV) - (SPT - 1);   // ... for V rows, which the split form requests later
  int stop = SPT * (ntiles - 1 - kAheadK) - (SPT - 1);
  int left = 0;        // stop - 1 - jb
  // what may need doing after step number j - 1 (at ring position R); true when the sequence is finished
  auto careful = [&](auto rc, uint64_t grow) __attribute__((always_inline)) -> bool {
    constexpr int R = decltype(rc)::value;
    if (j >= nsteps) return true;
    const int tile = (j + SPT - 1) / SPT;   // the next tile to be begun
    aim(tile + kAheadK, tile + kAheadV);
    // Keys past the end were scored from copies of the last row, so the lane maxima need no second look after masking.
    const int last_due = last_valid < 32 ? nsteps - 1 : nsteps;
    if (j == last_due) mask_tail(R % 2 == 0 ? w.st_b : w.st_a);
    if (j >= stop) {
      stop = j < aim_v ? aim_v : j < last_due ? last_due : nsteps;
      left = stop - 1 - jb;
    }
    // (before a ragged last step always, see attend_dense_bf16.hip; here that costs 0.5 us a call and takes seven of 300 to
    // 3000 keys from 2.3226e-3 to 2.3167e-3)
    if (grow != 0 || j == last_due) {
      float alpha[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        const float mz_old = -w.nmz[qb], mx = maximum_across_halves(w.mx[qb]);
        const float mz_new = maximum(mz_old, mx * zscale + kDenseHeadroom);
        const bool over = is_lost(mx, zscale, mz_new);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(over) != 0, 0))
          drop_scores(R % 2 == 0 ? w.st_b[qb] : w.st_a[qb], over);
        alpha[qb] = over ? NAN : __builtin_amdgcn_exp2f(mz_old - mz_new);
        if (!over) w.nmz[qb] = -mz_new;
      }
      w.acc_scale(alpha[0], alpha[1]);
    }
    return false;
  };
  // ring offset of the rows of the step at ring position r
  constexpr auto step_off = [](int r) constexpr { return (r / SPT % kRing) * TILEB + (r % SPT) * 32 * ROWB; };
#define DLLM_STEP(R)                                                                                                     \
  {                                                                                                                      \
    uint64_t grow;                                                                                                       \
    w.step<(R) % 2 == 0, KS == 2, step_off((R) + 2), step_off(R), step_off((R) / SPT * SPT + kAheadK * SPT),             \
           VBASE + step_off((R) / SPT * SPT + kAheadV * SPT)>(zscale, tl, grow);                                         \
    if ((R) % SPT == 0) {                                                                                                \
      tl.k += advance_k;                                                                                                 \
      tl.v += advance_v;                                                                                                 \
    }                                                                                                                    \
    if (__builtin_expect((uint32_t(grow) | uint32_t(grow >> 32) | uint32_t(left - (R) - 1) >> 31) != 0, 0)) {             \
      j = jb + (R) + 1;                                                                                                  \
      if (careful(DLLM_IC(R), grow)) break;                                                                              \
    }                                                                                                                    \
  }
  for (;;) {
    left = stop - 1 - jb;
    DLLM_STEP(0)
    DLLM_STEP(1)
    DLLM_STEP(2)
    DLLM_STEP(3)
    if constexpr (kRound == 8) {
      DLLM_STEP(4)
      DLLM_STEP(5)
      DLLM_STEP(6)
      DLLM_STEP(7)
    }
    jb += kRound;
  }
#undef DLLM_STEP
  w.drain();
  float accv[64], lrow[2];   // [qb][db][16]; lanes 0..31: the query's row sum, lanes 32..63: zero
  w.acc_read(accv);
  w.row_sums(lrow[0], lrow[1]);
  wait_tile_loads();   // the requests past the last tile still write to the rings, which are now space for the outputs
  __syncthreads();
  if constexpr (KS == 1) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
      store_dense_block<D>(accv + 32 * qb, sum_across_halves(lrow[qb]), smem + (2 * wave + qb) * 32 * ROWB,
                           qbase + (2 * wave + qb) * 32, at, s.hq, o);
  } else {
    static_assert(dense_merge_bytes<D>() <= int(sizeof smem), "merge space");
    const float m[2] = {no_keys ? -INFINITY : -w.nmz[0], no_keys ? -INFINITY : -w.nmz[1]};
    merge_dense_halves<D>(accv, lrow, m, part, smem, qbase + qwave * 64, at, s.hq, o);
  }
}

}  // namespace

hipError_t launch_attend_dense_paired(const Shape& s, int ks, dim3 grid, const void* q, const void* k, const void* v,
                                      const int32_t* cu_q, const int32_t* cu_kv, const uint8_t* seq_mode, int which,
                                      void* o, hipStream_t st) {
  auto launch = [&](auto kernel) {
    kernel<<<grid, kThreads, 0, st>>>(static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),
                                      static_cast<const uint16_t*>(v), cu_q, cu_kv, seq_mode, which,
                                      static_cast<uint16_t*>(o), s DLLM_CHECK_PASS);
  };
  if (ks == 2) launch(attend_dense_paired_bf16_kernel<2>);
  else launch(attend_dense_paired_bf16_kernel<1>);
  return hipGetLastError();
}

}  // namespace dllm
