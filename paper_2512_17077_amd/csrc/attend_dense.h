// What the two dense Refresh kernels (bf16) share: where a workgroup works, and how a block of outputs is written.
#pragma once
#include <type_traits>

#include "attn_tile.h"

namespace dllm {

// The larger of the two, or not a number if one of them is not (v_max_f32 would drop it).
__device__ __forceinline__ float maximum(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float maximum_across_halves(float x) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return maximum(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// What a step may not see.  Queries share the row-sum products, whose columns hold two of them told apart by zeros, so a
// probability that is infinite or NaN would reach another query's sum as 0 * NaN.  A query whose scores are infinite or NaN, or
// so large (2^31 and beyond) that the rounding of its maximum leaves them far above it, is lost: its scores of the
// step are taken out, and its accumulators, which are its own, are multiplied by NaN.
// mx: the query's largest score of a step, mz: the base-2 logit that stands for its running maximum
__device__ __forceinline__ bool is_lost(float mx, float zscale, float mz) { return !(fmaf(mx, zscale, -mz) <= 64.0f); }
__device__ __forceinline__ void drop_scores(f32x16& st, bool lost) {
#pragma unroll
  for (int i = 0; i < 16; ++i) st[i] = lost ? -INFINITY : st[i];
}

struct DensePlace {
  int qtile, h;            // query tile, query head
  int q0, nq, kv0, L;      // the sequence's first query, number of queries, first key, number of keys
};

// Which query tile of which (sequence, head) a workgroup takes.
//
// Batches of up to 64 sequences are launched as a one-dimensional grid with just enough workgroups for the
// query tiles the batch can have (the host bounds their number from total_q), and every workgroup finds
// its tile itself: lane i looks at sequence i, a prefix sum over the tiles of the sequences that are
// attended densely places the workgroup.  A mixed batch then starts no workgroups for its sparse
// sequences, and a ragged one none for the query tiles short sequences do not have (an empty workgroup
// holds a whole compute unit until it has found out that it is empty).  Larger batches use the
// three-dimensional grid (query tile, head, sequence) with an early exit.
//
// Workgroups are handed to the eight XCDs round-robin by launch order, and each XCD has its own L2.
// The numbering is such that the workgroups that stream the same K/V -- the query tiles of the query
// heads that share one KV head of one sequence -- land on one XCD (launch ids equal modulo 8) and
// share its L2, while consecutive (sequence, KV head) pairs go to different XCDs.

// A batch of up to 64 sequences: lane i holds one of them, those that are attended densely in order of their lengths.
struct DenseLanes {
  int q0, nq, kv0, L, tiles;
  int incl, total;   // tiles of the sequences up to this one; of all
};
// which: see launch_attend_dense_bf16
template <int Rows>
__device__ __forceinline__ DenseLanes gather_dense(const Shape& s, const int32_t* __restrict__ cu_q,
                                                   const int32_t* __restrict__ cu_kv, const uint8_t* __restrict__ seq_mode,
                                                   int which) {
  const int lane = threadIdx.x & 63;
  DenseLanes w{0, 0, 0, 0, 0, 0, 0};
  if (lane < s.batch) {
    w.q0 = cu_q[lane];
    w.nq = cu_q[lane + 1] - w.q0;
    w.kv0 = cu_kv[lane];
    w.L = cu_kv[lane + 1] - w.kv0;
    const bool dense = which == 2 || (seq_mode != nullptr && seq_mode[lane] == DLLM_SEQ_DENSE);
    w.tiles = dense ? (w.nq + Rows - 1) / Rows : 0;
  }
  // Longest sequences first: a workgroup lasts as long as its sequence has keys, and with the long ones at the
  // end of the launch most compute units wait for a few (seven sequences of 537 to 2076 keys, 16 heads x 64:
  // 82.9 us in batch order, 81.2 us longest first; 83.1 and 79.2 on another card).  Lane i goes on with the sequence of
  // rank i among the densely attended ones; equal lengths need no ranking.
  const uint64_t with_tiles = __builtin_amdgcn_ballot_w64(w.tiles != 0);
  const int first_L = with_tiles != 0 ? __builtin_amdgcn_readlane(w.L, __builtin_ctzll(with_tiles)) : 0;
  if (__builtin_amdgcn_ballot_w64(w.tiles != 0 && w.L != first_L) != 0) {
    const int rank = rank_longest_first(w.tiles != 0 ? w.L : -1, s.batch);   // lanes past the batch stay where they are
    w.q0 = __builtin_amdgcn_ds_permute(rank * 4, w.q0);
    w.nq = __builtin_amdgcn_ds_permute(rank * 4, w.nq);
    w.kv0 = __builtin_amdgcn_ds_permute(rank * 4, w.kv0);
    w.L = __builtin_amdgcn_ds_permute(rank * 4, w.L);
    w.tiles = __builtin_amdgcn_ds_permute(rank * 4, w.tiles);
  }
  w.incl = int(wave_inclusive_sum(uint32_t(w.tiles)));
  w.total = __builtin_amdgcn_readlane(w.incl, 63);
  return w;
}

// Tile number n of such a batch; false if it has no more than n.
__device__ __forceinline__ bool find_dense(const Shape& s, const DenseLanes& w, uint32_t n, DensePlace& at) {
  int b;
  if ((s.hkv & 7) == 0) {
    // XCD x = n % 8 takes KV heads x, x + 8, ...; within the XCD: sequence, KV head, query head of its group, tile
    const int per_seq = s.group * (s.hkv >> 3), place = int(n >> 3);
    if (place >= w.total * per_seq) return false;
    b = __builtin_ctzll(__builtin_amdgcn_ballot_w64(w.incl * per_seq > place));
    const int tb = __builtin_amdgcn_readlane(w.tiles, b);
    const int rem = place - (__builtin_amdgcn_readlane(w.incl, b) - tb) * per_seq;
    const int per_head_group = tb * s.group;
    const int kvh = (rem / per_head_group) * 8 + int(n & 7), r = rem % per_head_group;
    at.qtile = r % tb;
    at.h = kvh * s.group + r / tb;
  } else {
    const int place = int(n / uint32_t(s.hq));
    at.h = int(n % uint32_t(s.hq));
    if (place >= w.total) return false;
    b = __builtin_ctzll(__builtin_amdgcn_ballot_w64(w.incl > place));
    at.qtile = place - (__builtin_amdgcn_readlane(w.incl, b) - __builtin_amdgcn_readlane(w.tiles, b));
  }
  at.q0 = __builtin_amdgcn_readlane(w.q0, b);
  at.nq = __builtin_amdgcn_readlane(w.nq, b);
  at.kv0 = __builtin_amdgcn_readlane(w.kv0, b);
  at.L = __builtin_amdgcn_readlane(w.L, b);
  return true;
}

// The tile of this workgroup in the three-dimensional grid of a larger batch; false if there is none.
template <int Rows>
__device__ __forceinline__ bool place_dense_grid(const Shape& s, const int32_t* __restrict__ cu_q,
                                                 const int32_t* __restrict__ cu_kv, const uint8_t* __restrict__ seq_mode,
                                                 int which, DensePlace& at) {
  const int nx = gridDim.x, units = s.hkv * gridDim.z;
  const int n = blockIdx.x + nx * (blockIdx.y + gridDim.y * blockIdx.z);
  int b = blockIdx.z;
  at.qtile = blockIdx.x;
  at.h = blockIdx.y;
  if ((units & 7) == 0) {
    const int per_unit = s.group * nx;
    const int j = n >> 3;   // position in this XCD's own launch sequence
    const int r = j % per_unit, unit = (j / per_unit) * 8 + (n & 7);
    at.qtile = r % nx;
    at.h = (unit % s.hkv) * s.group + r / nx;
    b = unit / s.hkv;
  }
  if (which == 1 && !(seq_mode != nullptr && seq_mode[b] == DLLM_SEQ_DENSE)) return false;
  at.q0 = cu_q[b];
  at.nq = cu_q[b + 1] - at.q0;
  at.kv0 = cu_kv[b];
  at.L = cu_kv[b + 1] - at.kv0;
  return at.qtile * Rows < at.nq;
}

// LDS accesses of this wave before this point come before those behind it, whichever lanes make them (a lane's own
// addresses may be provably different ones).  No instruction: LDS serves a wave in order.
__device__ __forceinline__ void order_wave_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Writes 32 query rows: accumulators `a` ([db][16], as the matrix cores leave them) over the row sum l.  A lane holds
// four elements of one row at a time, so the block goes through LDS (`stage`, 32 rows that are this wave's alone) and out
// in whole rows.  first: the block's first query; rows past the last query are not written.  Lane offsets fit 32 bits: 32
// rows of at most 65535 heads span 512 MB.
template <int D>
__device__ __forceinline__ void store_dense_block(const float* a, float l, char* stage, int first, const DensePlace& at,
                                                  int hq, uint16_t* __restrict__ o) {
  constexpr int CH = D / 8;
  const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;
  const float inv = 1.0f / l;
  order_wave_lds();   // the rows may be read from until here: by the block before, or as the other wave's block
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      v2u w2;
      const float* x = a + 16 * db + 4 * i4;
      w2.x = cvt_pk_bf16(x[0] * inv, x[1] * inv);
      w2.y = cvt_pk_bf16(x[2] * inv, x[3] * inv);
      *reinterpret_cast<v2u*>(stage + tile_off<D>(col, 4 * db + i4) + 8 * hf) = w2;
    }
  order_wave_lds();
  first = __builtin_amdgcn_readfirstlane(first);
  const uint32_t row_bytes = uint32_t(hq) * (2 * D);
  char* base = reinterpret_cast<char*>(o + (int64_t(at.q0 + first) * hq + at.h) * D);
  const int left = at.nq - first;   // rows there are
  constexpr int kStep = 64 / CH;    // rows per store
  const uint32_t r0 = lane / CH, off = r0 * row_bytes + (lane % CH) * 16;
  auto put = [&](int i) __attribute__((always_inline)) {
    *reinterpret_cast<v4u*>(base + uint32_t(i * kStep) * row_bytes + off) =
        *reinterpret_cast<const v4u*>(stage + tile_off<D>(i * kStep + r0, lane % CH));
  };
  if (left >= 32) {
#pragma unroll
    for (int i = 0; i < 32 / kStep; ++i) put(i);
  } else {
#pragma unroll
    for (int i = 0; i < 32 / kStep; ++i)
      if (int(i * kStep + r0) < left) put(i);
  }
}

// The end of a workgroup whose waves w and w ^ 2 hold (m, l, O) of the same 64 queries over different keys: each finishes
// the block with its own number (`part`) and hands the other one over through LDS (`space`).  acc: [block][db][16]; l: row
// sums as the row-sum products leave them; m: running maxima, minus infinity for a wave without keys (one of the two has
// seen one).  All waves call it; nothing else may be in `space` any more.
template <int D>
constexpr int dense_merge_bytes() { return 4 * (D / 32) * 4 * 64 * 16 + 4 * 64 * 4; }
template <int D>
__device__ __forceinline__ void merge_dense_halves(const float* acc, const float* l, const float* m, int part, char* space,
                                                   int first, const DensePlace& at, int hq, uint16_t* __restrict__ o) {
  constexpr int NB = 16 * (D / 32), kBlock = NB / 4 * 64;   // accumulators, and float4s of LDS, of one block
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 31, other = wave ^ 2;
  float4* mrg = reinterpret_cast<float4*>(space);                       // [wave][db][i4][lane]
  float* ml = reinterpret_cast<float*>(space + 4 * kBlock * 16);        // [wave][m: 32 | l: 32]
  auto hand_over = [&](auto qc) __attribute__((always_inline)) {
    constexpr int QB = decltype(qc)::value;
#pragma unroll
    for (int n = 0; n < NB / 4; ++n) {
      const float* x = acc + NB * QB + 4 * n;
      mrg[wave * kBlock + n * 64 + lane] = make_float4(x[0], x[1], x[2], x[3]);
    }
    const float sum = sum_across_halves(l[QB]);
    if (lane < 32) {
      ml[wave * 64 + col] = m[QB];
      ml[wave * 64 + 32 + col] = sum;
    }
  };
  auto finish = [&](auto qc) __attribute__((always_inline)) {
    constexpr int QB = decltype(qc)::value;
    const float m_other = ml[other * 64 + col], top = fmaxf(m[QB], m_other);
    const float f_mine = __builtin_amdgcn_exp2f(m[QB] - top), f_other = __builtin_amdgcn_exp2f(m_other - top);
    float x[NB];
#pragma unroll
    for (int n = 0; n < NB / 4; ++n) {
      const float4 y = mrg[other * kBlock + n * 64 + lane];
      const float* a = acc + NB * QB + 4 * n;
      x[4 * n + 0] = a[0] * f_mine + y.x * f_other;
      x[4 * n + 1] = a[1] * f_mine + y.y * f_other;
      x[4 * n + 2] = a[2] * f_mine + y.z * f_other;
      x[4 * n + 3] = a[3] * f_mine + y.w * f_other;
    }
    // (the space the other wave's block came through is this wave's alone now)
    store_dense_block<D>(x, sum_across_halves(l[QB]) * f_mine + ml[other * 64 + 32 + col] * f_other,
                         space + other * kBlock * 16, first + QB * 32, at, hq, o);
  };
  constexpr std::integral_constant<int, 0> b0{};
  constexpr std::integral_constant<int, 1> b1{};
  if (part == 0) hand_over(b1); else hand_over(b0);
  __syncthreads();
  if (part == 0) finish(b0); else finish(b1);
}

// Zeros for `rows` query rows from `first` on: a sequence without keys.
template <int D>
__device__ __forceinline__ void zero_dense_rows(int first, int rows, const DensePlace& at, int hq, uint16_t* __restrict__ o) {
  for (int e = threadIdx.x; e < rows * D; e += blockDim.x) {
    const int r = first + e / D;
    if (r < at.nq) o[(int64_t(at.q0 + r) * hq + at.h) * D + e % D] = 0;
  }
}

}  // namespace dllm
