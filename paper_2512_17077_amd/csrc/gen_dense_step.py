#!/usr/bin/env python3
"""Writes attend_dense_step.inc: the instruction stream of one 32-key step of the dense Refresh kernel
(attend_dense_bf16.hip) as inline-assembly text with a fixed register map.

Why text and not builtins: with one wave per SIMD the kernel has 512 registers, but only the lower 256
(v0..v255) can feed vector instructions; the upper 256 (a0..a255) can only feed the matrix cores.  The
compiler, once it uses the upper half at all, puts every MFMA result there, the scores included, and
then copies them down one register at a time for the softmax: +60 % vector instructions.  Here the
output accumulators and the queries live in a-registers, the scores, probabilities and LDS operands in
v-registers, and the order of issue is exactly the order written: one MFMA, then the few vector and
LDS instructions that fit under it, and so on.

Run `python3 gen_dense_step.py` in this folder after changing the schedule; the .inc file is committed.

One step (iteration j) at D = 128, NQB = 2 blocks of 32 queries per wave:
    slots  0..15   S^T(j+1) = K(j+1) Q^T         MFMA(t, qb), K operand t shared by the two blocks
    slots 16..31   O^T += V(j-1)^T P(j-1)^T      MFMA(u, db, qb), V^T operand (u, db) shared likewise
    slots 32..35   l += ones P(j-1)^T             row sums of the same probabilities, 16x16x32 MFMA(u, qb), half as long
    all slots      P(j) = exp2(S(j) z - m z)      on the scores of the previous step: per pair of scores
                                                   2 fma, 2 exp, 1 cvt_pk (-> bf16 x 2)
    slots 20..31   row maxima of S(j+1)           16 max / max3
    LDS            16 transposing reads (V^T operands, four slots ahead of their MFMAs),
                   8 ds_read_b128 (K operands of step j+2, after the S chain has consumed the old ones)
Maxima are taken with NaN kept (v_maximum3_f32), and a maximum that is no number asks for the raise too: scores that are
infinite or NaN never reach the exponentials (see drop_scores).
Matrix results are read by vector instructions no sooner than four MFMAs after they were issued (the
hardware does not interlock that; 12 wait states are required), and a transcendental's result is not
read by the next instruction.
"""
import os
import sys

# ---- register map (v-registers; a-registers are numbered separately)
ST_A, ST_B = 96, 128          # scores, [qb][16]
PB_A, PB_B = 160, 176         # packed probabilities, [qb][u][4]
KOP = 192                     # K operands [t][4]
VOP = 224                     # V^T operand buffers [NBUF][4]
TMP = 76                      # [2][2] logits / probabilities in flight
SM = 70                       # two unused, nmz0, nmz1, mx0, mx1
ADDR = 80                     # ka[8], va[2][4]
NBUF = 8
ACC = 0                       # a: acc[qb][db][16]


def vr(base, n=1):
    return f"v{base}" if n == 1 else f"v[{base}:{base + n - 1}]"


def ar(base, n=1):
    return f"a{base}" if n == 1 else f"a[{base}:{base + n - 1}]"


def gen_step(D, cur, nxt, pnew, pold, with_scores=True, with_softmax=True, with_loads=False, split=False):
    """Instruction list of one step.  with_scores/with_softmax False: the closing P V product only.  split: the form
    in which two wave pairs share a tile's keys, so every step is a tile's first and requests K and V rows of
    different tiles, each from offsets of its own."""
    NT, NDB = D // 16, D // 32
    QR = 16 * 2 * NDB                      # a: q[qb][t][4] after the accumulators
    ROWB = 2 * D
    n_s = NT * 2 if with_scores else 0     # score MFMAs
    n_pv = 2 * NDB * 2                     # P V MFMAs
    n_ls = 4                               # row-sum MFMAs
    nslots = n_s + n_pv + n_ls
    LS = QR + 4 * NT * 2                   # a: ls[qb][4] after the queries
    # matrix-pipe time before each slot, in halves of a 32x32x16 product (a row-sum product takes one half)
    at = [2 * s if s <= n_s + n_pv else n_s + n_pv + s for s in range(nslots + 1)]

    # ---- MFMAs per slot
    mfma = []
    if with_scores:
        for t in range(NT):
            for qb in range(2):
                c = "0" if t == 0 else vr(nxt + 16 * qb, 16)
                mfma.append((f"v_mfma_f32_32x32x16_bf16 {vr(nxt + 16 * qb, 16)}, {vr(KOP + 4 * t, 4)}, "
                             f"{ar(QR + 4 * (NT * qb + t), 4)}, {c}", None))
    for u in range(2):
        for db in range(NDB):
            p = u * NDB + db
            for qb in range(2):
                a = ACC + 16 * (NDB * qb + db)
                mfma.append((f"v_mfma_f32_32x32x16_bf16 {ar(a, 16)}, {vr(VOP + 4 * (p % NBUF), 4)}, "
                             f"{vr(pold + 4 * (2 * qb + u), 4)}, {ar(a, 16)}", ("v", p) if qb == 0 else None))
    # row sums: rows 0 and 4 of ones * P^T, accumulated like the outputs (four a-registers each, after the queries)
    for u in range(2):
        for qb in range(2):
            a = LS + 4 * qb
            mfma.append((f"v_mfma_f32_16x16x32_bf16 {ar(a, 4)}, %[ones], {vr(pold + 4 * (2 * qb + u), 4)}, {ar(a, 4)}", None))

    # ---- LDS reads per slot: (text, tag)
    ds = [[] for _ in range(nslots)]
    npairs = 2 * NDB

    def vread(p, rd):
        u, db = divmod(p, NDB)
        return (f"ds_read_b64_tr_b16 {vr(VOP + 4 * (p % NBUF) + 2 * rd, 2)}, {vr(ADDR + 8 + NDB * rd + db)} "
                f"offset:%[voff{u}]", ("v", p))

    # the first NBUF operand pairs are fetched ahead of the P V phase, the others as their buffer frees up
    first = min(NBUF, npairs)
    if with_scores:
        lead = n_s - 2 * first
        for p in range(first):
            ds[lead + 2 * p].append(vread(p, 0))
            ds[lead + 2 * p + 1].append(vread(p, 1))
    else:
        for p in range(first):   # nothing to hide behind: all at once, in front
            ds[0].append(vread(p, 0))
            ds[0].append(vread(p, 1))
    for p in range(first, npairs):
        s0 = n_s + 2 * (p - NBUF) + 2   # after both MFMAs that read this buffer have been issued
        ds[s0].append(vread(p, 0))
        ds[s0 + 1].append(vread(p, 1))
    if with_scores:
        free = [s for s in range(n_s, n_s + n_pv) if not ds[s]]
        assert len(free) >= NT, (len(free), NT)
        for t in range(NT):
            ds[free[t]].append((f"ds_read_b128 {vr(KOP + 4 * t, 4)}, {vr(ADDR + t)} offset:%[koff]", ("k", t)))

    # ---- vector work
    valu = [[] for _ in range(nslots)]
    if with_softmax:
        ops = []
        pairs = [(qb, u, jj) for qb in range(2) for u in range(2) for jj in range(4)]

        # Row sums: the four extra MFMAs above add up the probabilities as rounded to bf16, the values the
        # matrix cores multiply with V, so the vector units only convert.
        def finish(i):
            qb, u, jj = pairs[i]
            t0 = TMP + 2 * (i % 2)
            w = pnew + 4 * (2 * qb + u) + jj
            return [f"v_cvt_pk_bf16_f32 {vr(w)}, {vr(t0)}, {vr(t0 + 1)}"]

        for i, (qb, u, jj) in enumerate(pairs):
            t0 = TMP + 2 * (i % 2)
            s0 = cur + 16 * qb + 8 * u + 2 * jj
            ops += [f"v_fma_f32 {vr(t0)}, {vr(s0)}, %[zs], {vr(SM + 2 + qb)}",
                    f"v_fma_f32 {vr(t0 + 1)}, {vr(s0 + 1)}, %[zs], {vr(SM + 2 + qb)}"]
            ops += [f"v_exp_f32_e32 {vr(t0 + c)}, {vr(t0 + c)}" for c in range(2)]
            ops += finish(i - 1) if i > 0 else []
        ops += ["s_nop 0"] + finish(len(pairs) - 1)   # the nop keeps the last exp's result from being read at once
        for s in range(nslots):   # evenly over the matrix pipe's time: about three per MFMA at D = 128
            valu[s] += ops[at[s] * len(ops) // at[-1]:at[s + 1] * len(ops) // at[-1]]
        # row maxima of the new scores, well after the S chain
        mops = []
        for i in range(8):
            for qb in range(2):
                s0 = nxt + 16 * qb + 2 * i
                m = vr(SM + 4 + qb)
                mops.append(f"v_maximum3_f32 {m}, {vr(s0) if i == 0 else m}, {vr(s0)}, {vr(s0 + 1)}")
        start = n_s + 4
        span = nslots - start
        for i, op in enumerate(mops):
            valu[start + i * span // len(mops)].append(op)

    # ---- tile loads (first step of a tile only): K then V rows of the tile two ahead, global memory
    # straight into LDS, one load every other MFMA so that their issue (about 50 cycles each when issued
    # back to back) hides under the matrix work.  m0 holds the LDS destination of the wave's slice.
    loads = [[] for _ in range(nslots)]
    if with_loads:
        nld = 64 * (D // 8) // 256
        vo = "vo" if split else "lo"
        seq = [("%[kt]", "%[lk]", "lo", i) for i in range(nld)] + [("%[vt]", "%[lv]", vo, i) for i in range(nld)]
        for n, (base, lds, off, i) in enumerate(seq):
            loads[2 + 2 * n] = [f"s_add_u32 m0, %[wl], {lds}+{i * 256 * 16}",
                                f"global_load_lds_dwordx4 %[{off}{i}], {base}"]

    # ---- emit, with the waits for LDS data: reads return in order, so a consumer waits until no more
    # reads are outstanding than were issued after the one it needs (steady state: the previous step's
    # tail is the same as this step's)
    order = []   # DS tags in issue order over this step
    for s in range(nslots):
        for _, tag in ds[s]:
            order.append(tag)
    lines = []
    issued = []   # tags issued so far in this step

    def wait_for(tag_pred, from_prev):
        if from_prev:
            # needed read was issued in the previous step: everything after it there, plus all issued here
            idx = max(i for i, t in enumerate(order) if tag_pred(t))
            n = (len(order) - 1 - idx) + len(issued)
        else:
            idx = max(i for i, t in enumerate(issued) if tag_pred(t))
            n = len(issued) - 1 - idx
        return n

    if not with_scores:   # the closing product: its first operand fetches come before its first MFMA
        for dtext, tag in ds[0]:
            lines.append(dtext)
            issued.append(tag)
        ds[0] = []
    for s in range(nslots):
        text, need = mfma[s]
        if with_scores and s < n_s and s % 2 == 0:
            t = s // 2
            n = wait_for(lambda tag: tag == ("k", t), True)
            lines.append(f"s_waitcnt lgkmcnt({min(n, 15)})")
        if need is not None:
            p = need[1]
            n = wait_for(lambda tag: tag == ("v", p), False)
            lines.append(f"s_waitcnt lgkmcnt({min(n, 15)})")
        lines.append(text)
        if with_loads and s == 1:
            # Tile boundary: the loads issued a tile ago (the next tile) have landed in every wave, and every
            # wave is done with the tile before last, whose ring slots the loads below refill.  Two MFMAs
            # are in the pipe while the waves meet.  (split: a tile lasts one step, so the previous step's loads
            # stay in flight and those before them have landed.)
            lines += [f"s_waitcnt vmcnt({len(seq) if split else 0})", "s_barrier"]
        if loads[s]:
            lines.append(loads[s][0])
        for dtext, tag in ds[s]:
            lines.append(dtext)
            issued.append(tag)
        lines += valu[s][:1]
        if loads[s]:
            lines.append(loads[s][1])
        lines += valu[s][1:]
    if with_softmax:
        # does any new score exceed its running maximum by more than the lazy step?  (lanes as a mask)
        lines += [f"v_fma_f32 {vr(TMP)}, {vr(SM + 4)}, %[zs], {vr(SM + 2)}",
                  f"v_fma_f32 {vr(TMP + 1)}, {vr(SM + 5)}, %[zs], {vr(SM + 3)}",
                  f"v_maximum3_f32 {vr(TMP)}, {vr(TMP)}, {vr(TMP)}, {vr(TMP + 1)}",
                  f"v_cmp_nle_f32_e64 %[grow], {vr(TMP)}, %[lazy]"]
    return lines


# ---- the form with two waves per SIMD (head_dim 64): half the registers, so probabilities take the place of the scores
# they come from, and K and V^T operands take turns in four a-register buffers
P2 = dict(NMZ=48, MX=50, TMP=52, ADDR=56, ST_A=64, ST_B=96, OPND=104)


def gen_paired_step(cur, nxt, with_loads, split=False):
    """One step of the form that runs two waves per SIMD (head_dim 64; split as in gen_step): in iteration j
        slots  0..7    S^T(j+1) = K(j+1) Q^T         beside them P(j), keys 0..15 of the step
        slots  8..13   O^T += V(j)^T P(j)^T, row sums  of keys 0..15; beside them P(j), keys 16..31
        slots 14..19   the same of keys 16..31        beside them the row maxima of S(j+1)
    K operands of step j+2 are fetched once the buffers' V^T operands are used up, and the other way round."""
    D, NT, NDB = 64, 4, 2
    QR, LS = 64, 96
    r = P2
    opnd = [ar(r["OPND"] + 4 * i, 4) for i in range(4)]
    prob = [[vr(cur + 16 * qb + 8 * u, 4) for u in range(2)] for qb in range(2)]
    mfma, need, reads = [], [], []   # per slot: text, operand it waits for, LDS reads issued behind it
    for t in range(NT):
        for qb in range(2):
            st = vr(nxt + 16 * qb, 16)
            mfma.append(f"v_mfma_f32_32x32x16_bf16 {st}, {opnd[t]}, {ar(QR + 4 * (NT * qb + t), 4)}, {'0' if t == 0 else st}")
            need.append(("k", t) if qb == 0 else None)
            u, db = divmod(t, NDB)
            reads.append([] if qb == 0 else
                         [(f"ds_read_b64_tr_b16 {ar(r['OPND'] + 4 * t + 2 * rd, 2)}, {vr(r['ADDR'] + 4 + NDB * rd + db)} "
                           f"offset:%[voff{u}]", ("v", t)) for rd in range(2)])
    for u in range(2):
        for db in range(NDB):
            for qb in range(2):
                a, n = ar(16 * (NDB * qb + db), 16), NDB * u + db
                mfma.append(f"v_mfma_f32_32x32x16_bf16 {a}, {opnd[n]}, {prob[qb][u]}, {a}")
                need.append(("v", n) if qb == 0 else None)
                reads.append([] if qb == 0 else [(f"ds_read_b128 {opnd[n]}, {vr(r['ADDR'] + n)} offset:%[koff]", ("k", n))])
        for qb in range(2):
            a = ar(LS + 4 * qb, 4)
            mfma.append(f"v_mfma_f32_16x16x32_bf16 {a}, %[ones], {prob[qb][u]}, {a}")
            need.append(None)
            reads.append([])

    # vector work: the pairs of scores, keys 0..15 of both query blocks first
    ops, done = [], {}
    pairs = [(qb, u, jj) for u in range(2) for qb in range(2) for jj in range(4)]

    def convert(i):
        qb, u, jj = pairs[i]
        t0 = r["TMP"] + 2 * (i % 2)
        ops.append(f"v_cvt_pk_bf16_f32 {vr(cur + 16 * qb + 8 * u + jj)}, {vr(t0)}, {vr(t0 + 1)}")
        done[i] = len(ops)

    for i, (qb, u, jj) in enumerate(pairs):
        t0 = r["TMP"] + 2 * (i % 2)
        s0 = cur + 16 * qb + 8 * u + 2 * jj
        ops += [f"v_fma_f32 {vr(t0 + c)}, {vr(s0 + c)}, %[zs], {vr(r['NMZ'] + qb)}" for c in range(2)]
        ops += [f"v_exp_f32_e32 {vr(t0 + c)}, {vr(t0 + c)}" for c in range(2)]
        if i > 0:
            convert(i - 1)
    ops.append("s_nop 0")   # the last exp's result is not read at once
    convert(15)
    tops = []
    for i in range(8):
        for qb in range(2):
            s0, m = nxt + 16 * qb + 2 * i, vr(r["MX"] + qb)
            tops.append(f"v_maximum3_f32 {m}, {vr(s0) if i == 0 else m}, {vr(s0)}, {vr(s0 + 1)}")
    # a product reads a converted probability no sooner than two instructions later
    cut = done[7] + 2
    phases = [(range(0, 8), ops[:cut]), (range(8, 14), ops[cut:] + tops[:2]), (range(14, 20), tops[2:])]
    valu = [[] for _ in mfma]
    for slots, work in phases:
        for n, s in enumerate(slots):
            valu[s] = work[n * len(work) // len(slots):(n + 1) * len(work) // len(slots)]

    order = [tag for rd in reads for _, tag in rd]
    lines, issued = [], []
    seq = [("%[kt]", "%[lk]", "lo", i) for i in range(2)] + [("%[vt]", "%[lv]", "vo" if split else "lo", i) for i in range(2)]
    for s, text in enumerate(mfma):
        if need[s] is not None:
            if need[s][0] == "k":   # fetched in the previous step
                n = len(order) - 1 - max(i for i, t in enumerate(order) if t == need[s]) + len(issued)
            else:
                n = len(issued) - 1 - max(i for i, t in enumerate(issued) if t == need[s])
            lines.append(f"s_waitcnt lgkmcnt({min(n, 15)})")
        lines.append(text)
        if with_loads and s == 1:
            # Tile boundary: the next tile has landed in every wave (the one after it stays in flight), and every wave
            # is done with the previous tile, whose ring slots the loads below refill.  (split: K rows of the step after
            # next have landed; what stays in flight are the V rows requested with them and the previous step's loads.)
            lines += [f"s_waitcnt vmcnt({6 if split else 4})", "s_barrier"]
        load = seq[(s - 2) // 2] if with_loads and s in (2, 4, 6, 8) else None
        if load:
            lines.append(f"s_add_u32 m0, %[wl], {load[1]}+{load[3] * 256 * 16}")
        for text, tag in reads[s]:
            lines.append(text)
            issued.append(tag)
        lines += valu[s][:1]
        if load:
            lines.append(f"global_load_lds_dwordx4 %[{load[2]}{load[3]}], {load[0]}")
        lines += valu[s][1:]
    t, m, z = r["TMP"], r["MX"], r["NMZ"]
    lines += [f"v_fma_f32 {vr(t)}, {vr(m)}, %[zs], {vr(z)}", f"v_fma_f32 {vr(t + 1)}, {vr(m + 1)}, %[zs], {vr(z + 1)}",
              f"v_maximum3_f32 {vr(t)}, {vr(t)}, {vr(t)}, {vr(t + 1)}", f"v_cmp_nle_f32_e64 %[grow], {vr(t)}, %[lazy]"]
    return lines


def as_macro(name, lines):
    body = " \\\n".join(f'  "{l}\\n\\t"' for l in lines)
    return f"#define {name} \\\n{body}\n"


def gen_score0(D, st=ST_A, kop=lambda t: vr(KOP + 4 * t, 4)):
    """S^T(0) into st_a from the K operands in kop, then enough wait states for any reader"""
    NT, NDB = D // 16, D // 32
    QR = 16 * 2 * NDB
    lines = []
    for t in range(NT):
        for qb in range(2):
            c = "0" if t == 0 else vr(st + 16 * qb, 16)
            lines.append(f"v_mfma_f32_32x32x16_bf16 {vr(st + 16 * qb, 16)}, {kop(t)}, "
                         f"{ar(QR + 4 * (NT * qb + t), 4)}, {c}")
    return lines + ["s_nop 15", "s_nop 15"]


def gen_acc_init(D):
    regs = list(range(16 * 2 * (D // 32)))
    ls = 16 * 2 * (D // 32) + 4 * (D // 16) * 2
    regs += list(range(ls, ls + 8))         # the row sums behind the queries
    return [f"v_accvgpr_write_b32 a{i}, 0" for i in regs]


def gen_acc_scale(D, TMP=TMP):
    """acc[qb] *= %[al<qb>] for both blocks, well after the last MFMA and before the next one."""
    n = 16 * (D // 32)
    lines = ["s_nop 15", "s_nop 15"]
    for qb in range(2):
        for i in range(0, n, 4):
            regs = [qb * n + i + c for c in range(4)]
            lines += [f"v_accvgpr_read_b32 {vr(TMP + c)}, a{r}" for c, r in enumerate(regs)]
            lines += [f"v_mul_f32_e32 {vr(TMP + c)}, %[al{qb}], {vr(TMP + c)}" for c in range(4)]
            lines += [f"v_accvgpr_write_b32 a{r}, {vr(TMP + c)}" for c, r in enumerate(regs)]
    ls = 2 * n + 4 * (D // 16) * 2   # the row sums: only the first register of each four is ever non-zero
    for qb in range(2):
        lines += [f"v_accvgpr_read_b32 {vr(TMP)}, a{ls + 4 * qb}", f"v_mul_f32_e32 {vr(TMP)}, %[al{qb}], {vr(TMP)}",
                  f"v_accvgpr_write_b32 a{ls + 4 * qb}, {vr(TMP)}"]
    lines += ["s_nop 7"]
    return lines


def gen_acc_read(k):
    """sixteen accumulator registers a[16k .. 16k+15] into operands %0 .. %15"""
    return [f"v_accvgpr_read_b32 %{i}, a{16 * k + i}" for i in range(16)]


def main():
    out = ["// Generated by gen_dense_step.py -- do not edit by hand.  One 32-key step of the dense Refresh kernel as",
           "// inline-assembly text over a fixed register map; see the generator for the schedule and the map.",
           "// Named operands: %[ones] (four v-registers: the A operand of the row sums), %[zs] (softmax_scale * log2 e, scalar), %[koff] (byte offset of the K rows fetched",
           "// for step j+2), %[voff0], %[voff1] (byte offsets of the V rows of step j-1, keys 0..15 and 16..31),",
           "// %[grow] (out, scalar pair: lanes whose newest scores outgrew the running maximum by more than %[lazy]);",
           "// in the _AB text (the first step of a tile) also %[kt], %[vt] (scalar pairs: first K / V row of the tile",
           "// to load), %[lo0..] (per-lane byte offsets of the 16-byte chunks), %[wl] (LDS address of the wave's",
           "// slice of a load round), %[lk], %[lv] (byte offsets of the K / V ring slots to fill).  The _SPLIT texts are",
           "// the steps of the form that splits a tile's keys between two wave pairs: both request tiles, the V rows at",
           "// offsets %[vo0..] of their own.",
           ""]
    for D in (128,):
        out.append(as_macro(f"DLLM_DENSE_STEP_{D}_AB", gen_step(D, ST_A, ST_B, PB_A, PB_B, with_loads=True)))
        out.append(as_macro(f"DLLM_DENSE_STEP_{D}_BA", gen_step(D, ST_B, ST_A, PB_B, PB_A)))
        out.append(as_macro(f"DLLM_DENSE_STEP_{D}_AB_SPLIT", gen_step(D, ST_A, ST_B, PB_A, PB_B, with_loads=True, split=True)))
        out.append(as_macro(f"DLLM_DENSE_STEP_{D}_BA_SPLIT", gen_step(D, ST_B, ST_A, PB_B, PB_A, with_loads=True, split=True)))
        out.append(as_macro(f"DLLM_DENSE_TAIL_{D}", gen_step(D, 0, 0, 0, PB_A, False, False)))
        out.append(as_macro(f"DLLM_DENSE_SCORE0_{D}", gen_score0(D)))
        out.append(as_macro(f"DLLM_DENSE_ACC_INIT_{D}", gen_acc_init(D)))
        out.append(as_macro(f"DLLM_DENSE_ACC_SCALE_{D}", gen_acc_scale(D)))
    out.append(as_macro("DLLM_DENSE_ACC_INIT_64", gen_acc_init(64)))
    st_a, st_b = P2["ST_A"], P2["ST_B"]
    out.append(as_macro("DLLM_DENSE_PAIRED_STEP_AB", gen_paired_step(st_a, st_b, True)))
    out.append(as_macro("DLLM_DENSE_PAIRED_STEP_BA", gen_paired_step(st_b, st_a, False)))
    out.append(as_macro("DLLM_DENSE_PAIRED_STEP_AB_SPLIT", gen_paired_step(st_a, st_b, True, True)))
    out.append(as_macro("DLLM_DENSE_PAIRED_STEP_BA_SPLIT", gen_paired_step(st_b, st_a, True, True)))
    out.append(as_macro("DLLM_DENSE_PAIRED_SCORE0", ["s_nop 1"] + gen_score0(64, st_a, lambda t: ar(P2["OPND"] + 4 * t, 4))))
    out.append(as_macro("DLLM_DENSE_PAIRED_ACC_SCALE", gen_acc_scale(64, P2["TMP"])))
    for k in range(8):
        out.append(as_macro(f"DLLM_DENSE_ACC_READ_{k}", gen_acc_read(k)))
    outdir = os.path.dirname(os.path.abspath(__file__))
    for a in sys.argv[1:]:
        if a.startswith("--out="):
            outdir = a[6:]
    path = os.path.join(outdir, "attend_dense_step.inc")
    with open(path, "w") as f:
        f.write("\n".join(out))
    print("wrote", path)


if __name__ == "__main__":
    main()
