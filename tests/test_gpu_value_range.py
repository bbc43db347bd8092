"""Values near the ends of the number range, where the online softmax keeps a running maximum that lags behind: outputs
are means of V rows, so V scaled by a power of two must give outputs scaled by it, and keys whose score overflows to
minus infinity must simply carry no weight."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2512_17077_amd import hcsa, synth, workload

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-5, torch.bfloat16: 2e-2}


def growing_workload(dtype, hq, hkv, D, lens, qlens, keep, dense, growth=31.0):
    """One key near the middle and one near the end of every sequence stand 2^growth above all others, whose base-2 logits
    stay near zero: a maximum raised late leaves probabilities of 2^growth in the sums."""
    w = synth.make_workload("range", synth.SEED_BASE + 2000, dtype, hq, hkv, D, lens, qlens, keep,
                            seq_mode=np.full(len(lens), 1 if dense else 0, np.uint8))
    w.q.fill_(1.0)
    k = 0.01 * w.k.float()
    for b in range(len(lens)):
        lo, hi = int(w.cu_kv[b]), int(w.cu_kv[b + 1])
        for pos in (lo + (hi - lo) // 2, hi - 1 - (hi - lo) // 20):
            k[pos] = growth / (w.softmax_scale * math.log2(math.e) * D)
    w.k.copy_(k.to(dtype))
    return w


def attend_both_ways(w, log2_scale):
    """Outputs of the library on V * 2^log2_scale, scaled back, and the oracle's on V (the scaling is exact in both types)."""
    idx = oracle.select(synth.to_bits(w.q), synth.to_bits(w.k), w.cu_q, w.cu_kv, w.cu_k)
    ref = oracle.attend(synth.to_bits(w.q), synth.to_bits(w.k), synth.to_bits(w.v), w.cu_q, w.cu_kv, idx, w.cu_k, w.seq_mode,
                        w.softmax_scale)
    w.v.copy_((w.v.double() * 2.0 ** log2_scale).to(w.v.dtype))
    dw = workload.DeviceWorkload(w)
    dw.attend(torch.from_numpy(np.ascontiguousarray(idx)).to(dw.device))
    return dw.o.double().cpu().numpy() * 2.0 ** -log2_scale, ref


def check_values(w, log2_scale):
    got, ref = attend_both_ways(w, log2_scale)
    assert np.isfinite(got).all(), "an accumulator overflowed"
    assert np.abs(got - ref).max() <= TOL[w.dtype]


# bf16 inputs: probabilities reach 2^8, so sums over 2^9 keys of |V| up to 2^2 * 2^100 stay below 2^120
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("hq,hkv,lens,keep", [(4, 2, [400], [300]), (32, 8, [2900], [2600]),
                                              (32, 8, [40 + 30 * b for b in range(16)], [30 + 25 * b for b in range(16)])])
@pytest.mark.parametrize("log2_scale", [100, -110])
def test_large_and_small_values_in_kept_lists(hq, hkv, lens, keep, D, log2_scale):
    """One workgroup per list, lists cut into chunks, and many lists per workgroup."""
    check_values(growing_workload(torch.bfloat16, hq, hkv, D, lens, [32] * len(lens), keep, dense=False), log2_scale)


# fp32 inputs: the maximum is exact, probabilities stay at or below 1
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("hq,hkv,lens,keep", [(4, 2, [400], [300]), (8, 4, [900, 500, 700], [800, 300, 650])])
@pytest.mark.parametrize("dense", [False, True])
def test_large_values_in_fp32(hq, hkv, lens, keep, D, dense):
    keep = [0] * len(lens) if dense else keep
    qlens = lens if dense else [32] * len(lens)
    check_values(growing_workload(torch.float32, hq, hkv, D, lens, qlens, keep, dense), 112)


# bf16 dense sequences: split over wave pairs with few heads, whole with many
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("hq,hkv,lens", [(4, 2, [400]), (4, 2, [33]), (32, 8, [330] * 8), (32, 8, [700, 450, 290, 530, 801, 333])])
@pytest.mark.parametrize("growth", [6.0, 31.0])
@pytest.mark.parametrize("log2_scale", [100, -110])
def test_large_and_small_values_in_dense_sequences(hq, hkv, lens, D, growth, log2_scale):
    """(Small: products with probabilities of 2^-24 are below the smallest normal number.)"""
    check_values(growing_workload(torch.bfloat16, hq, hkv, D, lens, lens, [0] * len(lens), True, growth), log2_scale)


def masked_outputs(dtype, hq, hkv, D, L, first, last):
    """Dense attention of one sequence whose keys first .. last-1 score minus infinity (their products with the queries
    overflow, all inputs are finite), and the same over the other keys in fp64."""
    w = synth.make_workload("masked", synth.SEED_BASE + 2100, dtype, hq, hkv, D, [L], [40], [0], seq_mode=np.ones(1, np.uint8))
    w.q.copy_((2.0 ** 64 * (1.0 + w.q.float().abs())).to(dtype))
    w.k.copy_((2.0 ** -64 * w.k.float()).to(dtype))
    w.k[first:last] = -2.0 ** 70
    rest = [i for i in range(L) if not first <= i < last]
    q = w.q.double().transpose(0, 1)
    k, v = (x.double()[rest].repeat_interleave(hq // hkv, 1).transpose(0, 1) for x in (w.k, w.v))
    ref = torch.matmul(torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * w.softmax_scale, -1), v)
    dw = workload.DeviceWorkload(w)
    dw.dense_refresh()
    return dw.o.double().cpu(), ref.transpose(0, 1)


@pytest.mark.parametrize("first,last", [(0, 16), (16, 32), (0, 32), (32, 64), (64, 96), (0, 64), (96, 200)])
@pytest.mark.parametrize("dtype,hq,hkv,D", [(torch.bfloat16, 4, 2, 128), (torch.bfloat16, 4, 2, 64), (torch.float32, 4, 2, 64),
                                            (torch.float32, 4, 2, 128)])
def test_keys_whose_score_overflows_to_minus_infinity(dtype, hq, hkv, D, first, last):
    got, ref = masked_outputs(dtype, hq, hkv, D, 200, first, last)
    assert torch.isfinite(got).all()
    assert (got - ref).abs().max() <= TOL[dtype]


@pytest.mark.parametrize("hq,hkv,D,form", [(2, 1, 128, 2), (2, 1, 64, 2), (16, 8, 128, 1), (16, 8, 64, 1)])
def test_a_ragged_last_step_raises_the_maximum(hq, hkv, D, form):
    """Two keys carry each sequence: one in the first 32, the largest in the ragged last step, with values that nearly cancel.
    Both set their query's running maximum, so both probabilities are powers of two and what is left of the output is exact
    but for its own rounding and fp32: logits up to 32 are rounded to 2^-20 twice on either side, which leaves 2^-18 of values up
    to 2.  A probability rounded to bf16 leaves up to 2^-9 of them."""
    n, extra = 20, [1, 7, 16, 31]
    lens = [64 * (1 + b // 4) + extra[b % 4] for b in range(n)]
    qlens = [40] * n if form == 2 else [256] * n
    w = synth.make_workload("last", synth.SEED_BASE + 2300, torch.bfloat16, hq, hkv, D, lens, qlens, [0] * n,
                            seq_mode=np.ones(n, np.uint8))
    rng = np.random.default_rng(5)
    w.q.fill_(0.0)
    w.q[:, :, 0] = 1.0
    w.k.fill_(0.0)
    w.k[:, :, 0] = -60.0 / (w.softmax_scale * math.log2(math.e))
    w.v.fill_(0.0)
    ref = torch.empty(w.q.shape, dtype=torch.float64)
    for b in range(n):
        lo, hi, unit = int(w.cu_kv[b]), int(w.cu_kv[b + 1]), 1.0 / (w.softmax_scale * math.log2(math.e))
        first, last = lo + int(rng.integers(0, 32)), hi - 1 - int(rng.integers(0, extra[b % 4]))
        below = float(rng.uniform(0.05, 0.95))
        w.k[last, :, 0], w.k[first, :, 0] = 3.0 * unit, (3.0 - below) * unit
        ratio = torch.exp2((w.k[first, :, 0].double() - w.k[last, :, 0].double()) / unit)
        w.v[last], w.v[first] = 1.0, (-1.0 / ratio[:, None]).to(w.v.dtype).expand(-1, D)
        each = (1.0 + ratio * w.v[first, :, 0].double()) / (1.0 + ratio)
        ref[int(w.cu_q[b]):int(w.cu_q[b + 1])] = each.repeat_interleave(hq // hkv)[None, :, None]
    dw = workload.DeviceWorkload(w)
    assert hcsa.dllm_hcsa_attend_form_of(dw.batch, all_dense=True)[2] == form
    dw.dense_refresh()
    err = (dw.o.double().cpu() - ref).abs()
    assert (err <= 2.0 ** -8 * ref.abs() + 2.0 ** -16).all(), float(err.max())


@pytest.mark.parametrize("first,last", [(0, 1), (40, 41), (199, 200), (64, 128)])
@pytest.mark.parametrize("bad_value", [-1.0, -2.0 ** -74, float("nan")])
@pytest.mark.parametrize("hq,hkv,n,D,form", [(4, 2, 1, 128, 2), (4, 2, 1, 64, 2), (16, 8, 20, 128, 1), (16, 8, 20, 64, 1)])
def test_scores_that_overflow_spoil_their_own_query_only(hq, hkv, n, D, form, first, last, bad_value):
    """Keys that score plus infinity for a few queries (or 2^66, far beyond what logits can tell apart; or queries that hold
    NaN) and minus infinity for all others, which must come out as if those keys were not there: queries share matrix
    products, but none may see another's values.  The few are NaN where they scored infinity or hold NaN."""
    L, nq, bad = 200, 70 if form == 2 else 256, [3, 17, 36, 52, 69]
    w = synth.make_workload("contained", synth.SEED_BASE + 2200, torch.bfloat16, hq, hkv, D, [L] * n, [nq] * n, [0] * n,
                            seq_mode=np.ones(n, np.uint8))
    w.q.copy_((2.0 ** 64 * (1.0 + w.q.float().abs())).to(w.q.dtype))
    w.k.copy_((2.0 ** -64 * w.k.float()).to(w.k.dtype))
    for b in range(n):
        w.q[[b * nq + i for i in bad]] *= bad_value
        w.k[b * L + first:b * L + last] = -2.0 ** 70
    rest = [i for i in range(L) if not first <= i < last]
    good = [i for i in range(nq) if i not in bad]
    q = w.q.double().view(n, nq, hq, D).transpose(1, 2)
    k, v = (x.double().view(n, L, hkv, D)[:, rest].repeat_interleave(hq // hkv, 2).transpose(1, 2) for x in (w.k, w.v))
    ref = torch.matmul(torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) * w.softmax_scale, -1), v)
    dw = workload.DeviceWorkload(w)
    assert hcsa.dllm_hcsa_attend_form_of(dw.batch, all_dense=True)[2] == form
    dw.dense_refresh()
    got = dw.o.double().cpu().view(n, nq, hq, D).transpose(1, 2)
    assert bad_value == -2.0 ** -74 or torch.isnan(got[:, :, bad]).all()
    assert torch.isfinite(got[:, :, good]).all()
    assert (got - ref)[:, :, good].abs().max() <= TOL[torch.bfloat16]


@pytest.mark.parametrize("pos", [0, 40, 64, 130, 199])
@pytest.mark.parametrize("hq,hkv,n,D,form", [(4, 2, 1, 128, 2), (4, 2, 1, 64, 2), (16, 8, 20, 128, 1), (16, 8, 20, 64, 1)])
def test_a_key_that_is_no_number_shows(hq, hkv, n, D, form, pos):
    """One NaN in a key: all outputs of its KV head's query heads are NaN, whichever step meets it; no others are."""
    L, nq = 200, 70 if form == 2 else 256
    w = synth.make_workload("nan", synth.SEED_BASE + 2201, torch.bfloat16, hq, hkv, D, [L] * n, [nq] * n, [0] * n,
                            seq_mode=np.ones(n, np.uint8))
    w.k[[b * L + pos for b in range(n)], 1, 5] = float("nan")
    dw = workload.DeviceWorkload(w)
    assert hcsa.dllm_hcsa_attend_form_of(dw.batch, all_dense=True)[2] == form
    dw.dense_refresh()
    group = hq // hkv
    assert torch.isnan(dw.o[:, group:2 * group]).all()
    assert torch.isfinite(dw.o[:, :group]).all() and torch.isfinite(dw.o[:, 2 * group:]).all()


@pytest.mark.parametrize("first,last", [(0, 1), (40, 41), (199, 200), (64, 128)])
@pytest.mark.parametrize("dtype,D,dense", [(torch.bfloat16, 128, False), (torch.bfloat16, 64, False), (torch.float32, 64, False),
                                           (torch.float32, 128, True)])
def test_overflow_stays_with_its_query_in_kept_lists_and_fp32(dtype, D, dense, first, last):
    """The same over kept lists (of all positions) and in fp32."""
    L, nq, hq, hkv, bad = 200, 40, 4, 2, [3, 17, 36]
    w = synth.make_workload("contained", synth.SEED_BASE + 2202, dtype, hq, hkv, D, [L], [nq], [0 if dense else L],
                            seq_mode=np.full(1, 1 if dense else 0, np.uint8))
    w.q.copy_((2.0 ** 64 * (1.0 + w.q.float().abs())).to(dtype))
    w.k.copy_((2.0 ** -64 * w.k.float()).to(dtype))
    w.q[bad] *= -1.0
    w.k[first:last] = -2.0 ** 70
    rest = [i for i in range(L) if not first <= i < last]
    good = [i for i in range(nq) if i not in bad]
    q = w.q.double().transpose(0, 1)
    k, v = (x.double()[rest].repeat_interleave(hq // hkv, 1).transpose(0, 1) for x in (w.k, w.v))
    ref = torch.matmul(torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * w.softmax_scale, -1), v).transpose(0, 1)
    dw = workload.DeviceWorkload(w)
    dw.attend(torch.arange(0 if dense else L, dtype=torch.int32).repeat(hq, 1).to(dw.device))
    got = dw.o.double().cpu()
    assert torch.isnan(got[bad]).all() and torch.isfinite(got[good]).all()
    assert (got - ref)[good].abs().max() <= TOL[dtype]
