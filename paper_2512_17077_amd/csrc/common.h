// Internal declarations shared by the HIP translation units of libdllm_hcsa (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dllm_hcsa.h"

namespace dllm {

constexpr int kWave = 64;

// 16 bytes as a native vector: loads and stores of it stay plain vector moves in every address
// space, so register tiles built from it are always promoted out of private memory
typedef __attribute__((ext_vector_type(4))) unsigned int v4u;
typedef __attribute__((ext_vector_type(2))) unsigned int v2u;

// Element strides and sizes every kernel needs; built once per call on the host.
struct Shape {
  int32_t batch, hq, hkv, group, d;
  int64_t q_tok, q_head, kv_tok, kv_head;  // element strides
  int32_t total_q, total_kv, max_q, max_kv;
  float scale;
};

// Whether K rows are better read with the non-temporal hint (load_once).  A Reuse step streams K for the scores
// and then gathers rows of the same K: while K is small, lines left in the caches by the first are found by the
// second.  Measured per selection / per step of selection and attention, hint against no hint in both: K of 10 MB
// 9.66 / 19.0 against 9.23 / 18.65 us, 21 MB 12.6 / 22.3 against 12.2 / 21.2, 42 MB 16.3 / 26.7 against 16.2 / 25.8, 34 MB
// under grouped queries 16.9 / 29.4 against 16.7 / 28.0; but the stream itself loses from 100 MB on (34.1 against 35.1 us;
// at 168 MB 38.4 against 41.8), the gather from 260 MB on (33.1 against 36.2 us on the kept rows of 264 MB of K, while 101 MB
// gains 55.4 -> 53.5 us a step, 168 MB 59.0 -> 57.4).  The two other kernels that read K always take the hint: the
// one-launch selection (hint / none: K of 17 MB 19.3 / 19.3 us, 67 MB 37.3 / 39.9, 134 MB 59.2 / 65.1; a step 41.3 / 40.9, 89.5 /
// 90.6, 157.1 / 154.4) and the Reuse kernel that walks several lists (attention / step over K of 25 MB 12.8 / 29.1
// against 13.0 / 28.2, 50 MB 14.0 / 34.3 against 14.2 / 33.3, 126 MB 22.7 / 55.6 against 21.3 / 54.0, 264 MB 33.4 / 85.7
// against 36.5 / 89.0: up to 3 % of a step are left there below 128 MB).
inline int64_t k_bytes(const Shape& s, int es) { return int64_t(s.total_kv) * s.hkv * s.d * es; }
inline bool streams_once(const Shape& s, int es) { return k_bytes(s, es) > (int64_t(64) << 20); }
inline bool gathers_once(const Shape& s, int es) { return k_bytes(s, es) > (int64_t(128) << 20); }

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// ---- selection (select_kernels.hip)
struct SelectPlan {
  size_t off_scores, off_summed, bytes;
};
SelectPlan plan_select(const Shape& s);
hipError_t launch_select(const Shape& s, dllm_dtype dt, const void* q, const void* k, const int32_t* cu_q,
                         const int32_t* cu_kv, const int32_t* cu_k, int32_t total_k, int32_t max_k,
                         int32_t pool_w, int32_t forced_tail, int32_t head_sum, int32_t* idx_out, void* ws,
                         hipStream_t st);

// the form a selection call of this shape takes under the current setting (ONE_LAUNCH or TWO_LAUNCHES)
int32_t select_form_of(const Shape& s, dllm_dtype dt, int32_t pool_w, int32_t head_sum);
int32_t set_select_form(int32_t form);   // DLLM_SELECT_FORM_*; returns the previous one, -1 if form is not one of them

// ---- packing of the kept rows (pack_kernels.hip)
hipError_t launch_pack(const Shape& s, dllm_dtype dt, const void* k, const void* v, const int32_t* cu_kv,
                       const int32_t* idx, const int32_t* cu_k, int32_t total_k, int32_t max_k, void* kp, void* vp,
                       hipStream_t st);

// ---- attention over kept rows / all rows (attend_*.hip)
struct AttendPlan {
  int32_t chunk_rows;  // kept rows one workgroup walks
  int32_t n_chunks;    // upper bound on chunks per (sequence, head)
  int32_t max_k;       // the caller's bound on kept rows per (sequence, head)
  int32_t v_split;     // workgroups per list that share out head_dim of V and O (1, 2 or 4; n_chunks is 1 if more than one)
  size_t off_po, off_pm, off_pl, bytes;
};
AttendPlan plan_attend(const Shape& s, dllm_dtype dt, int32_t max_k, int64_t total_k);
// Wave groups that share the keys of a densely attended sequence in the bf16 kernel (1 or 2); `which` as below.
int dense_key_splits(const Shape& s, int which);

// `which` selects the sequences a launch works on: 0 = all, each as its flag in seq_mode says (fp32 only);
// 1 = those flagged dense; 2 = every sequence, as dense.
hipError_t launch_attend_f32(const Shape& s, const void* q, const void* k, const void* v, const int32_t* cu_q,
                             const int32_t* cu_kv, const int32_t* idx, const int32_t* cu_k, int32_t total_k,
                             const uint8_t* seq_mode, int which, void* o, hipStream_t st);
hipError_t launch_zero_sparse_outputs(const Shape& s, dllm_dtype dt, const int32_t* cu_q, const uint8_t* seq_mode,
                                      void* o, hipStream_t st);
hipError_t launch_attend_sparse_bf16(const Shape& s, const AttendPlan& p, const void* q, const void* k,
                                     const void* v, const int32_t* cu_q, const int32_t* cu_kv, const int32_t* idx,
                                     const int32_t* cu_k, int32_t total_k, const uint8_t* seq_mode, void* o,
                                     void* ws, hipStream_t st);
hipError_t launch_attend_dense_bf16(const Shape& s, const void* q, const void* k, const void* v,
                                    const int32_t* cu_q, const int32_t* cu_kv, const uint8_t* seq_mode, int which,
                                    void* o, hipStream_t st);
hipError_t launch_attend_dense_paired(const Shape& s, int ks, dim3 grid, const void* q, const void* k, const void* v,
                                      const int32_t* cu_q, const int32_t* cu_kv, const uint8_t* seq_mode, int which,
                                      void* o, hipStream_t st);

// ---- optional device-side precondition checks (checks.hip; built with -DDLLM_CHECK_PRECONDITIONS)
// In that build every entry point first runs validators over the offset arrays and the index lists, which
// set bits in an error word, and every kernel takes that word's address as its last argument and returns
// at once if it is not zero: a violating input is reported and nothing is read or written through it.
#ifdef DLLM_CHECK_PRECONDITIONS
#define DLLM_CHECK_PARAM , const uint32_t* __restrict__ check_word
#define DLLM_CHECK_PASS , dllm::check_word()
#define DLLM_CHECK_EXIT() \
  if (*check_word != 0) return
uint32_t* check_word();   // device address of the current GPU's error word; NULL if it cannot be had
#else
#define DLLM_CHECK_PARAM
#define DLLM_CHECK_PASS
#define DLLM_CHECK_EXIT()
#endif
// Runs the validators (a no-op in the release build).  cu_k, idx and seq_mode may be NULL.
hipError_t validate_inputs(const Shape& s, const int32_t* cu_q, const int32_t* cu_kv, const int32_t* cu_k,
                           const int32_t* idx, const uint8_t* seq_mode, int32_t total_k, int32_t max_k,
                           int32_t forced_tail, hipStream_t st);

// ---- device helpers
// 16-byte load of data that is read once per launch (K/V rows streamed or gathered from HBM).  With Once set it
// carries the non-temporal hint, which keeps such lines from displacing reusable data in the caches and
// measurably raises the HBM read rate on MI355X (selection over 264 MB of K: 52.0 against 57.7 us); without it the
// lines may stay, for a call whose K is small enough to be found again (streams_once, gathers_once).
template <bool Once = true>
__device__ __forceinline__ v4u load_once(const void* p) {
  if constexpr (Once) return __builtin_nontemporal_load(static_cast<const v4u*>(p));
  else return *static_cast<const v4u*>(p);
}
// Inclusive prefix sum over the 64 lanes of a wave (all lanes active) through the data-parallel
// primitives: shifts by 1, 2, 4, 8 within each row of 16 lanes, then the last lane of row 0 (2) is
// added to row 1 (3), then lane 31 to rows 2 and 3.  A lane without a source adds zero.
template <int Ctrl, int RowMask>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {
  return x + uint32_t(__builtin_amdgcn_update_dpp(0, int(x), Ctrl, RowMask, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
  x = dpp_add<0x111, 0xf>(x);   // row_shr:1
  x = dpp_add<0x112, 0xf>(x);   // row_shr:2
  x = dpp_add<0x114, 0xf>(x);   // row_shr:4
  x = dpp_add<0x118, 0xf>(x);   // row_shr:8
  x = dpp_add<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  x = dpp_add<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Rank of this lane's sequence among those of lanes 0 .. batch-1 (batch <= 64) by descending length, ties to the lower lane;
// lanes past the batch get a rank past it.  length >= -1.  The keys are all different, so one comparison per sequence does,
// and sequences are taken eight at a time (a loop over single ones with a second comparison for equal lengths took 1.1 to
// 2.4 us at the start of the dense kernel's workgroups on a batch of 25); lengths from 2^25 on count as equal.
__device__ __forceinline__ int rank_longest_first(int length, int batch) {
  const int lane = int(threadIdx.x & 63u);
  const uint32_t key = lane < batch ? uint32_t(min(length, (1 << 25) - 2) + 1) << 6 | uint32_t(63 - lane) : uint32_t(63 - lane);
  int rank = 0;
  for (int i = 0; i < batch; i += 8)
#pragma unroll
    for (int c = 0; c < 8; ++c) rank += uint32_t(__builtin_amdgcn_readlane(int(key), i + c)) > key ? 1 : 0;
  return lane < batch ? rank : lane;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16, round to nearest even (inputs are finite here)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

}  // namespace dllm
