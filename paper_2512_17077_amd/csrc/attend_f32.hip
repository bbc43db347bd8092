// fp32 attention (Section 2.3, Eq. 3 and Eq. 4) in fp32 throughout, on the fp32 matrix instructions of gfx950.
//
// fp32 inputs are held to 1e-5 absolute, which rules out the reduced-precision matrix paths, but
// v_mfma_f32_16x16x4_f32 multiplies and adds in fp32 at twice the rate of the vector units (157 TFLOP/s on
// the chip) and needs no operand broadcast, so both products run on it:
//   - A workgroup of eight waves owns NQ blocks of 16 queries of one (sequence, head); the waves deal the
//     keys out in tiles of 16 and merge their (m, l, O) through LDS at the end.  Splitting the keys and not
//     the queries is what fills the chip: these batches have few heads and blocks of 32 queries.
//   - S^T = K Q^T (16 keys x 16 queries) and O^T += V^T P^T.  The contraction order inside a 16-byte chunk is
//     free, so lane (key, j) simply loads chunk 4c + j of its own K row, and the score accumulators are,
//     unchanged, the B operand of the second product (step i contracts keys i, 4+i, 8+i, 12+i).  For V the
//     lane (r, j) loads chunk r of row 4j + i: one instruction fetches four whole 256-byte row parts.  No tile
//     goes through LDS.
//   - K of the next tile is requested when this tile's score product has read it, V likewise, and the row
//     ids one tile further ahead, so every load has a product's time (512 NQ cycles at D = 64) to arrive.
// Bound: matrix time where the keys are many, the chain launch -> offsets -> ids -> rows, about 5 us, where they are few.
// 8 heads x 64, a sequence of 700 tokens beside three Reuse blocks over up to 630 kept rows: 1.08 GFLOP, 6.9 us at the full
// rate, 9.4 us because 200 workgroups leave 56 compute units out; measured 22 us in one launch: by clock marks 0.8 us
// until a workgroup knows its place, 1.6 to 3.3 until its queries and first keys are there, 13.6 in the loop (six tiles a
// wave, whose products, softmax and row sums follow one another), 1.2 in the merge, launch and drain around them.  One wave per
// query row with vector arithmetic took 630 us in two launches; one sequence with 4 heads and 64 kept rows takes 5.5 us
// instead of 14.6.
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "attn_tile.h"

namespace dllm {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kF32Waves = 8;

// max / sum over the four lanes that hold one query's scores (lane, lane ^ 16, lane ^ 32, lane ^ 48)
__device__ __forceinline__ float quad_max(float x) {
  const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_across_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quad_sum(float x) {
  const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return sum_across_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// which: 0 = every sequence as its flag says (kept rows, or all rows if flagged dense); 1 = only sequences
//        flagged dense; 2 = every sequence, treated as dense
template <int D, int NQ>
__global__ __launch_bounds__(kF32Waves * 64, 2) void attend_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cu_k, int32_t total_k, const uint8_t* __restrict__ seq_mode, int which,
    float* __restrict__ o, Shape s DLLM_CHECK_PARAM) {
  DLLM_CHECK_EXIT();
  constexpr int QT = 16 * NQ;      // queries per workgroup
  constexpr int NC = D / 16;       // groups of four 16-byte chunks per row
  constexpr int NH = D / 64;       // 64-wide parts of head_dim
  constexpr int UNITS = NQ * NH * 4;
  __shared__ f32x4 mrg[kF32Waves][UNITS][64];          // (m, l, O) of the waves
  __shared__ float sm_m[kF32Waves][QT], sm_l[kF32Waves][QT];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, j = lane >> 4;
  {   // every kernel argument is fetched now, next to the offsets, not one by one where it is first used
    auto fetch_now = [](auto x) { asm volatile("" ::"s"(x)); };
    fetch_now(q); fetch_now(k); fetch_now(v); fetch_now(idx); fetch_now(o); fetch_now(total_k);
    fetch_now(s.hq); fetch_now(s.group); fetch_now(s.q_tok); fetch_now(s.q_head); fetch_now(s.kv_tok);
    fetch_now(s.kv_head); fetch_now(s.scale);
  }
  // Which query tile: with up to 64 sequences the grid has one dimension and just enough workgroups, and a
  // prefix sum over the sequences' tiles (lane i looks at sequence i) places this one; otherwise (tile,
  // head, sequence).  Heads are numbered fastest, so workgroups that read one head's rows share an XCD.
  int b, h, qtile, q0, nq, kv0, L, ko0 = 0, kb = 0;
  bool dense;
  if (gridDim.y == 1 && gridDim.z == 1) {
    int my_q0 = 0, my_nq = 0, my_kv0 = 0, my_L = 0, my_ko0 = 0, my_kb = 0, my_tiles = 0, my_dense = 0;
    if (lane < s.batch) {
      my_q0 = cu_q[lane];
      my_nq = cu_q[lane + 1] - my_q0;
      my_kv0 = cu_kv[lane];
      my_L = cu_kv[lane + 1] - my_kv0;
      if (cu_k != nullptr) {
        my_ko0 = cu_k[lane];
        my_kb = cu_k[lane + 1] - my_ko0;
      }
      my_dense = which == 2 || (seq_mode != nullptr && seq_mode[lane] == DLLM_SEQ_DENSE);
      my_tiles = which == 1 && !my_dense ? 0 : (my_nq + QT - 1) / QT;
    }
    const int incl = int(wave_inclusive_sum(uint32_t(my_tiles)));
    const int place = int(blockIdx.x / uint32_t(s.hq));
    h = int(blockIdx.x) - place * s.hq;
    if (place >= __builtin_amdgcn_readlane(incl, 63)) return;
    b = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl > place));
    qtile = place - (__builtin_amdgcn_readlane(incl, b) - __builtin_amdgcn_readlane(my_tiles, b));
    q0 = __builtin_amdgcn_readlane(my_q0, b);
    nq = __builtin_amdgcn_readlane(my_nq, b);
    kv0 = __builtin_amdgcn_readlane(my_kv0, b);
    L = __builtin_amdgcn_readlane(my_L, b);
    ko0 = __builtin_amdgcn_readlane(my_ko0, b);
    kb = __builtin_amdgcn_readlane(my_kb, b);
    dense = __builtin_amdgcn_readlane(my_dense, b) != 0;
  } else {
    qtile = blockIdx.x; h = blockIdx.y; b = blockIdx.z;
    dense = which == 2 || (seq_mode != nullptr && seq_mode[b] == DLLM_SEQ_DENSE);
    if (which == 1 && !dense) return;
    q0 = cu_q[b]; nq = cu_q[b + 1] - q0;
    kv0 = cu_kv[b]; L = cu_kv[b + 1] - kv0;
    if (cu_k != nullptr) { ko0 = cu_k[b]; kb = cu_k[b + 1] - ko0; }
  }
  const int qbase = qtile * QT;
  if (qbase >= nq) return;
  const int n = dense ? L : kb;   // rows attended to
  const int g = h / s.group;
  if (n == 0) {   // nothing to attend to: zeros
    for (int e = tid; e < QT * (D / 4); e += kF32Waves * 64) {
      const int r = qbase + e / (D / 4);
      if (r < nq) *reinterpret_cast<f32x4*>(o + (int64_t(q0 + r) * s.hq + h) * D + 4 * (e % (D / 4))) = f32x4{0, 0, 0, 0};
    }
    return;
  }
  // a NULL idx stands for the identity lists (kept rows 0 .. k_b-1): then a row is its own list position
  const int32_t* __restrict__ rows = (dense || idx == nullptr) ? nullptr : idx + int64_t(h) * total_k + ko0;
  const char* kbase = reinterpret_cast<const char*>(k + int64_t(kv0) * s.kv_tok + int64_t(g) * s.kv_head + 4 * j);
  const char* vbase = reinterpret_cast<const char*>(v + int64_t(kv0) * s.kv_tok + int64_t(g) * s.kv_head + 4 * c16);
  const uint64_t pitch = uint64_t(s.kv_tok) * 4;   // bytes from one token to the next (any number: 64 bits throughout)
  auto row_at = [&](const char* base, int row) -> const f32x4* {
    return reinterpret_cast<const f32x4*>(base + uint64_t(uint32_t(row)) * pitch);
  };
  const int ntiles = (n + 15) >> 4;
  const float zscale = s.scale * kLog2e;   // > 0: (score - maximum) * zscale is a base-2 logit
  // The running maximum starts at the lowest finite number, not at minus infinity: a wave may meet a whole tile of keys
  // whose scores overflowed to minus infinity, and those weigh nothing instead of (-inf) - (-inf).
  float m_used[NQ], lsum[NQ];
  f32x4 acc[NQ][4 * NH];
#pragma unroll
  for (int nb = 0; nb < NQ; ++nb) {
    m_used[nb] = -FLT_MAX;
    lsum[nb] = 0.0f;
#pragma unroll
    for (int db = 0; db < 4 * NH; ++db) acc[nb][db] = f32x4{0, 0, 0, 0};
  }

  // The walk over this wave's tiles, compiled for lists and for rows in place: with every load of the loop
  // unconditional (past the end the last row again) the compiler can count them, and waits for K, V and ids
  // separately; a load behind a branch makes it wait for everything at the top of the loop.
  auto walk = [&](auto gather) {
    auto row_of = [&](int tile) -> int {   // row of this lane's key of a tile; positions past the end repeat the last one
      const int t = min(tile * 16 + c16, n - 1);
      return decltype(gather)::value ? rows[t] : t;
    };
    // Loads issued ahead must stay ahead: without a (possible) store behind them the compiler turns "loaded
    // before the loop or at the end of the last iteration" into "loaded at the top of this one".
    auto stay = []() { asm volatile("" ::: "memory"); };
    f32x4 kf[NC], vf[4][NH];
    auto fetch_k = [&](int row) {
      const f32x4* p = row_at(kbase, row);
#pragma unroll
      for (int c = 0; c < NC; ++c) kf[c] = p[4 * c];
    };
    auto fetch_v = [&](int row) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4* p = row_at(vbase, __shfl(row, 4 * j + i));
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) vf[i][hh] = p[16 * hh];
      }
    };
    const int row = row_of(wave);
    int row_next = row_of(wave + kF32Waves);
    fetch_k(row);
    fetch_v(row);
    stay();
    f32x4 qf[NQ][NC];
#pragma unroll
    for (int nb = 0; nb < NQ; ++nb) {
      const int qi = min(qbase + 16 * nb + c16, nq - 1);   // past the last query: the last one again, never stored
      const float* qp = q + int64_t(q0 + qi) * s.q_tok + int64_t(h) * s.q_head + 4 * j;
#pragma unroll
      for (int c = 0; c < NC; ++c) qf[nb][c] = *reinterpret_cast<const f32x4*>(qp + 16 * c);
    }

    for (int tile = wave; tile < ntiles; tile += kF32Waves) {
      f32x4 st[NQ];
#pragma unroll
      for (int nb = 0; nb < NQ; ++nb) st[nb] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int nb = 0; nb < NQ; ++nb)
            st[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[nb][c][e], st[nb], 0, 0, 0);
      fetch_k(row_next);
      stay();
      const int nvalid = n - tile * 16;
      if (nvalid < 16) {
#pragma unroll
        for (int nb = 0; nb < NQ; ++nb)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (4 * j + i >= nvalid) st[nb][i] = -INFINITY;
      }
      // The maximum is exact, so probabilities never exceed 1 and sums stay below the number of keys times the largest
      // |V|.  Raising it only past 2^32 overflows from |V| of about 2^80 on and gains 0.6 us on the batch above.
      float tmax[NQ];
      bool grown = false;
#pragma unroll
      for (int nb = 0; nb < NQ; ++nb) {
        tmax[nb] = quad_max(fmaxf(fmaxf(st[nb][0], st[nb][1]), fmaxf(st[nb][2], st[nb][3])));
        grown = grown || tmax[nb] > m_used[nb];
      }
      if (__builtin_amdgcn_ballot_w64(grown) != 0) {
#pragma unroll
        for (int nb = 0; nb < NQ; ++nb) {
          const float m_new = fmaxf(m_used[nb], tmax[nb]);
          const float alpha = __builtin_amdgcn_exp2f((m_used[nb] - m_new) * zscale);   // first tile: 0, or times sums that are 0
          m_used[nb] = m_new;
          lsum[nb] *= alpha;
#pragma unroll
          for (int db = 0; db < 4 * NH; ++db) acc[nb][db] *= alpha;
        }
      }
      float p[NQ][4];
#pragma unroll
      for (int nb = 0; nb < NQ; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[nb][i] = __builtin_amdgcn_exp2f((st[nb][i] - m_used[nb]) * zscale);   // exactly 1 at the maximum
          lsum[nb] += p[nb][i];
        }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int hh = 0; hh < NH; ++hh)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int nb = 0; nb < NQ; ++nb)
              acc[nb][4 * hh + e] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][hh][e], p[nb][i], acc[nb][4 * hh + e], 0, 0, 0);
      const int row_after = row_of(tile + 2 * kF32Waves);
      fetch_v(row_next);
      stay();
      row_next = row_after;
    }
  };
  if (rows != nullptr) walk(std::true_type{});
  else walk(std::false_type{});

  // ---- merge: every wave leaves its maxima, sums and unscaled accumulators; a unit is (query block, part of
  // head_dim, register i), whose four accumulators are neighbours in head_dim
#pragma unroll
  for (int nb = 0; nb < NQ; ++nb) {
    const float l = quad_sum(lsum[nb]);
    if (j == 0) {
      sm_m[wave][16 * nb + c16] = m_used[nb];
      sm_l[wave][16 * nb + c16] = l;
    }
#pragma unroll
    for (int hh = 0; hh < NH; ++hh)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        mrg[wave][(nb * NH + hh) * 4 + i][lane] =
            f32x4{acc[nb][4 * hh][i], acc[nb][4 * hh + 1][i], acc[nb][4 * hh + 2][i], acc[nb][4 * hh + 3][i]};
  }
  __syncthreads();
  const int busy = min(kF32Waves, ntiles);   // waves that saw a tile
  for (int u = wave; u < UNITS; u += kF32Waves) {
    const int i = u & 3, hh = (u >> 2) % NH, nb = (u >> 2) / NH, col = 16 * nb + c16;
    float m_all = sm_m[0][col];
    for (int w = 1; w < busy; ++w) m_all = fmaxf(m_all, sm_m[w][col]);
    float l_all = 0.0f;
    f32x4 a = f32x4{0, 0, 0, 0};
    for (int w = 0; w < busy; ++w) {
      const float f = __builtin_amdgcn_exp2f((sm_m[w][col] - m_all) * zscale);
      l_all += sm_l[w][col] * f;
      a += mrg[w][u][lane] * f;
    }
    const int qi = qbase + col;
    if (qi < nq)
      *reinterpret_cast<f32x4*>(o + (int64_t(q0 + qi) * s.hq + h) * D + 64 * hh + 16 * j + 4 * i) = a * (1.0f / l_all);
  }
}

// o rows of the sequences not flagged dense := 0 (what attention over an empty kept list is defined as);
// used when a call passes no cu_k at all.  es: element bytes.
__global__ __launch_bounds__(256) void zero_sparse_outputs_kernel(const int32_t* __restrict__ cu_q,
                                                                  const uint8_t* __restrict__ seq_mode,
                                                                  char* __restrict__ o, int row_bytes DLLM_CHECK_PARAM) {
  DLLM_CHECK_EXIT();
  const int b = blockIdx.y;
  if (seq_mode != nullptr && seq_mode[b] == DLLM_SEQ_DENSE) return;
  const int64_t lo = int64_t(cu_q[b]) * row_bytes, hi = int64_t(cu_q[b + 1]) * row_bytes;   // multiples of 16
  for (int64_t e = lo + (int64_t(blockIdx.x) * 256 + threadIdx.x) * 16; e < hi; e += int64_t(gridDim.x) * 256 * 16)
    *reinterpret_cast<v4u*>(o + e) = v4u{0u, 0u, 0u, 0u};
}

hipError_t launch_zero_sparse_outputs(const Shape& s, dllm_dtype dt, const int32_t* cu_q, const uint8_t* seq_mode,
                                      void* o, hipStream_t st) {
  if (s.max_q == 0) return hipSuccess;
  const int row_bytes = s.hq * s.d * (dt == DLLM_F32 ? 4 : 2);
  const int64_t per_seq = int64_t(s.max_q) * row_bytes / (256 * 16) + 1;
  zero_sparse_outputs_kernel<<<dim3(unsigned(per_seq < 64 ? per_seq : 64), s.batch), 256, 0, st>>>(
      cu_q, seq_mode, static_cast<char*>(o), row_bytes DLLM_CHECK_PASS);
  return hipGetLastError();
}

template <int D, int NQ>
static hipError_t launch_f32(const Shape& s, const float* q, const float* k, const float* v, const int32_t* cu_q,
                             const int32_t* cu_kv, const int32_t* idx, const int32_t* cu_k, int32_t total_k,
                             const uint8_t* seq_mode, int which, float* o, hipStream_t st) {
  constexpr int QT = 16 * NQ;
  const int64_t nx = (s.max_q + QT - 1) / QT;
  dim3 grid(unsigned(nx), s.hq, s.batch);
  if (s.batch <= 64) {   // the workgroups place themselves (see the kernel)
    const int64_t tiles = std::min<int64_t>(int64_t(s.total_q) / QT + s.batch, nx * s.batch);
    if (tiles * s.hq < (int64_t(1) << 31)) grid = dim3(unsigned(tiles * s.hq), 1, 1);
  }
  attend_f32_kernel<D, NQ><<<grid, kF32Waves * 64, 0, st>>>(q, k, v, cu_q, cu_kv, idx, cu_k, total_k, seq_mode, which, o,
                                                            s DLLM_CHECK_PASS);
  return hipGetLastError();
}

hipError_t launch_attend_f32(const Shape& s, const void* q, const void* k, const void* v, const int32_t* cu_q,
                             const int32_t* cu_kv, const int32_t* idx, const int32_t* cu_k, int32_t total_k,
                             const uint8_t* seq_mode, int which, void* o, hipStream_t st) {
  if (s.max_q == 0) return hipSuccess;   // no sequence has a query: nothing to write
  const float *qf = static_cast<const float*>(q), *kf = static_cast<const float*>(k), *vf = static_cast<const float*>(v);
  float* of = static_cast<float*>(o);
  // Two query blocks per workgroup halve the K and V traffic per flop (21 against 24 us on the batch above);
  // one makes twice as many workgroups, which is what a batch of few queries lacks (5.5 against 6.2 us for one
  // block of 32 queries with 4 heads).  The line: 128 workgroups of two blocks, half the chip.
  const bool wide = int64_t(s.total_q) * s.hq >= 32 * 128;
  auto go = [&](auto launch) { return launch(s, qf, kf, vf, cu_q, cu_kv, idx, cu_k, total_k, seq_mode, which, of, st); };
  if (s.d == 128) return wide ? go(launch_f32<128, 2>) : go(launch_f32<128, 1>);
  return wide ? go(launch_f32<64, 2>) : go(launch_f32<64, 1>);
}

}  // namespace dllm
