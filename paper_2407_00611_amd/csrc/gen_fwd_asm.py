#!/usr/bin/env python3
"""Generates the gfx950 assembly of the forward main loop (head_dim 128, or 64) as a C string literal.

    python gen_fwd_asm.py > st_fwd_asm.inc          (build.py does this before compiling)
    python gen_fwd_asm.py 64 > st_fwd64_asm.inc     (head_dim 64: half the contraction steps and half the
                                                     O^T row blocks per key block, tiles of 128-byte rows)

Body of ONE `asm volatile` statement in st_fwd_fast.hip.  A workgroup (4 wavefronts) owns 256 queries of
one head, 64 per wavefront as two 32-query blocks, and walks 64-key tiles: first the ones that every one of
its rows sees in full, then the ones that a mask edge crosses (the causal diagonal, the ragged end of a chunk).
It writes O = acc / l, lse and, where asked for, O rounded to bf16; query rows beyond the shard are not stored.

Masked tiles are the last S_NM of the walk.  The loop exists twice: the first copy has no masks and leaves for the
second where a block of a masked tile comes up (the compare that ends a loop without masks does it, so whole tiles
pay nothing; a test of its own in every 32-key block cost 1.4 % at head size 64); the second copy tests every block
and calls an out-of-line routine that overwrites the invisible exponents with -inf before their exponentials are.
The ragged end of a chunk is read as the chunk's last 64 rows, with the rows of the tile before it masked, so no
load leaves the chunk.  Where no tile is visible to all rows, a row may meet its first visible key late: its
reference starts at zero and is set to its first finite block maximum by the mask routine (its accumulators are
still zero), since a lazy reference never moves down.

MFMA C layout "lane = query column": the exponent reference r (log2 units) and the row sum are one
register per lane and query block.  The Q fragments are multiplied by scale * log2(e) once (and rounded
to bf16 again), and every S^T accumulator starts from -r instead of zero, so the MFMAs deliver the
exponent S c - r directly and no VALU instruction is spent on it.  The reference starts as the row's maximum over the
first tile, so that the P of that key is 1 and carries no rounding: a row that sees few keys (the first ones of a causal
sequence) is mostly that key.  Rounded up to whole log2 units it made O of the first rows of a sequence 1.6e-3 wrong where
one key is seen and the result is exact, of rows 1 to 31 2.0e-3 instead of 1.5e-3, of 2000 rows together 2.19e-3 instead of
1.91e-3.  From there it is lazy: it only moves, by a whole number of log2 units, when a block's maximum exceeds it by more
than GAP, so the rescale factor is an exact power of two and the common path never touches the accumulators.  That is
noticed by the block's row sums, which are there anyway: while they stay below a limit no exponent was too large, and
beyond it, infinities included, nothing of the block has been used yet and its exponents still stand where the MFMAs put
them.  A maximum of its own, 17 of 97 VALU instructions per block, cost the loop 2 % at head size 128 (6.03 ms, now 5.90)
and 5 % at 64 (11.7 ms, now 11.1), where it waits for VALU issue.

Per 32-key block i and wavefront two groups of 16 MFMAs, software-pipelined two blocks deep:
    group B   O^T += V^T P^T(i)          A: V^T of block i by LDS transpose reads, B: packed P(i)
    group A   S^T(i+2) = K Q^T           A: K rows of block i+2 from LDS,          B: Q fragments (AGPRs)
    VALU      slots 3..30: P(i+1) = exp2(S c - r), bf16 pack, row sums of the block; behind slot 30 the test of the sums
              (rare: call the rescale routine), then their addition to the running ones
K / V tiles (64 keys) arrive by direct global->LDS loads into a 4-stage ring, three tiles ahead; one
barrier per tile.  The chunk table (base pointers, tiles per chunk) sits in LDS, written by the C++ side.
"""
import os
import sys

from st_asmgen import Emitter, ar, sr, vr, write_inc

D = 64 if "64" in sys.argv[1:] else 128              # head_dim
KS, DB, QB, NS = D // 16, D // 32, 2, 4
ROW = 2 * D                                          # bytes of one K / V row in LDS
TILE = 64 * ROW                                      # one 64-key tile
NDMA = TILE // 4096                                  # direct-to-LDS loads per wavefront and tile (4 wavefronts x 1 KiB each)
NSLOT = 4 * DB + 2 * KS                              # MFMAs per key block and wavefront
SPLIT = 4 * 2 * TILE > 65536                         # ring beyond the 16-bit offset field: second set of base registers
                                                     # (the limit of a block sum, 2^(GAP + 4), arrives in s46)

# ---- AGPRs
def ACC(db, qb): return 16 * (2 * db + qb)
def QF(qb, ks): return 128 + 4 * (KS * qb + ks)

# ---- VGPRs
def SBUF(buf, qb): return 32 * buf + 16 * qb        # two score buffers (S, then P in fp32)
def P16(buf, qb, m): return 64 + 16 * buf + 8 * qb + 4 * m
def NL(qb): return 240 - 16 * qb                     # sixteen copies of -r (minus the exponent reference, log2 units):
                                                     # the C operand that starts every S^T accumulator
                                                     # (NL(1) reuses the input registers once the prologue has read them)
def LSUM(qb): return 98 + qb                        # row sum over the blocks before (this lane's key rows)
def BSUM(qb, c): return 100 + 2 * qb + c             # of the block in hand, two chains
LIMR, SMAX = 105, 106                                # what a block sum may be; largest block sum of both query blocks
def MX(qb): return 194 + qb                         # row maximum (prologue, rescale routine)
TMP = 108                                            # 108..119
POOL0 = 120                                          # 2 rings x 4 fragments x 4 registers
XL, XH = 152, 160
TRLO_L, TRHI_L, TRLO_H, TRHI_H = 168, 172, 176, 180
KOFF, VOFF = 184, 188
OOFF, LSEOFF = 192, 193
RT = 200                                             # 200..223: probabilities on their way to the pack; temporaries of the
                                                     # out-of-line routines, which are called when none is
def QREL(qb): return 198 + qb                        # the row's position relative to the tile's first row, less 4 * (lane / 32)
def SEEN(qb): return 104 if qb == 0 else 107         # 0: the row has met no visible key yet
# inputs (pinned by the C++ side): v[224:239]
I_QROW0, I_QROW1, I_XBASE, I_GF16, I_TRBASE, I_LF16, I_KOFF0, I_VOFF0, I_OOFF, I_LSEOFF, I_QREL, I_LIVE = (
    224, 226, 228, 229, 230, 231, 232, 233, 234, 235, 236, 238)       # I_LIVE: bit qb = the lane's row of block qb exists
S_LIMIT = 46
(S_LDS, S_WAVE, S_NT, S_KRS16, S_VRS16, S_SCALE, S_OPTR, S_OQB, S_TBL, S_KTILE, S_VTILE, S_LSEPTR) = (
    32, 33, 34, 35, 36, 37, 38, 40, 41, 42, 43, 44)
# scalar temporaries
S_CEXP, T_M0, T_REM, D_KPTR, D_VPTR, D_LEFT, D_IDX, D_TBL, T_X = 47, 64, 65, 66, 68, 70, 71, 72, 73
T_RET, T_RARE = 76, 78                               # return address; address of rescale routine b at 78 + 2 b
# set by the prologue, from the parameter block behind the chunk table in LDS
S_LIVE = 48                                          # 48:49, 50:51: lanes whose row of block qb exists
S_NM, S_NM1, S_MTBL, S_FRESH, S_OLOW = 52, 53, 54, 55, 56   # masked tiles, + 1; their first table entry; 1: no tile is visible
                                                     # to all rows; 56:57: bf16 copy of O, or null
M_LEFT, M_REL, M_LO, T_MRET, T_CMP, T_MASK = 58, 59, 60, 62, 82, 90   # masked walk; four compare results; mask routine kb at 90 + 2 kb

# ---- LDS map
def KT(s): return 2 * TILE * s
def VT(s): return 2 * TILE * s + TILE
TBL = 2 * TILE * NS                                  # at most three entries per chunk: whole tiles, masked tiles, ragged end
PARAMS = 3 * 64 * 32                                 # offset of the parameter block from the table
LDS_BYTES = TBL + PARAMS + 64

LAT = int(os.environ.get("ST_GEN_FWD_LAT", 3))
# issue units of side work per MFMA slot: 0 = spread evenly; otherwise as many as fit, from the first slot on, the rest in one lump
# ahead of the test.  24 heads of 64 x 16384 rows x 131072 keys: 11.30 ms evenly, 11.10 by sixes, 11.15 by sevens, 11.4 by nines and
# more; 32/8 heads of 128 x 4096 rows x 32 chunks of 4096: 5.90 ms evenly, 5.93 by sixes, 6.0 and 6.1 by sevens and eights.
BUDGET = int(os.environ.get("ST_GEN_FWD_BUDGET", 0 if D == 128 else 6))
BRANCH_SLOT = NSLOT - 2                              # the test of the row sums sits behind this MFMA slot


NEXT_STUBS = []                                      # (label, return label) of every switch to the next chunk
STUBS = []                                           # (call label, return label, P buffer) of every reference test
MASK_STUBS = []                                      # (call label, return label, score buffer) of every mask test


class Pipe:
    def __init__(self, e):
        self.e = e
        self.frag_reg, self.uses_left, self.owner = {}, {}, {}

    def alloc(self, ring, idx, tag, uses):
        slot = 4 * ring + idx % 4
        old = self.owner.get(slot)
        assert old is None or self.uses_left[old] == 0, f"fragment {old} overwritten by {tag} before its last use"
        self.owner[slot] = tag
        self.uses_left[tag] = uses
        self.frag_reg[tag] = POOL0 + 4 * slot
        return POOL0 + 4 * slot

    def use(self, tag):
        assert self.uses_left[tag] > 0, tag
        self.uses_left[tag] -= 1
        return self.frag_reg[tag]

    def snapshot(self):
        return list(self.e.ds), dict(self.frag_reg), dict(self.uses_left), dict(self.owner)

    def restore(self, snap):
        self.e.ds, self.frag_reg, self.uses_left, self.owner = list(snap[0]), dict(snap[1]), dict(snap[2]), dict(snap[3])


def upper(stage): return SPLIT and stage >= 2
def xreg(stage, ks): return (XH if upper(stage) else XL) + ks
def trregs(stage): return (TRLO_H, TRHI_H) if upper(stage) else (TRLO_L, TRHI_L)
def imm(stage, base): return base - (65536 if upper(stage) else 0)


def read_k(p, blk, ks, seq):
    stage, kb = blk
    tag = f"k{seq}_{ks}"
    r = p.alloc(0, ks, tag, QB)
    p.e.ds_read(f"ds_read_b128 {vr(r, 4)}, {vr(xreg(stage, ks))} offset:{imm(stage, KT(stage)) + 32 * ROW * kb}", tag)


def read_vt(p, blk, m, db, seq):
    """V^T fragment (32 d rows x 16 keys) of a block: A operand of O^T += V^T P^T."""
    stage, kb = blk
    tag = f"t{seq}_{m}_{db}"
    r = p.alloc(1, DB * m + db, tag, QB)
    lo, hi = trregs(stage)
    off = imm(stage, VT(stage)) + 32 * ROW * kb + 16 * ROW * m
    p.e.ds_read(f"ds_read_b64_tr_b16 {vr(r, 2)}, {vr(lo + db)} offset:{off}", tag + "lo")
    p.e.ds_read(f"ds_read_b64_tr_b16 {vr(r + 2, 2)}, {vr(hi + db)} offset:{off}", tag)


def valu_exchange(reg=MX, op="v_max_f32"):
    """The two halves of the wavefront hold different key rows of the same query column: combine them in both."""
    out = []
    for qb in range(QB):
        out.append(f"v_mov_b32 {vr(TMP + qb)}, {vr(reg(qb))}")
    out.append("s_nop 1")
    for qb in range(QB):
        out.append(f"v_permlane32_swap_b32 {vr(TMP + qb)}, {vr(reg(qb))}")
    out.append("s_nop 1")
    for qb in range(QB):
        out.append(f"{op} {vr(reg(qb))}, {vr(reg(qb))}, {vr(TMP + qb)}")
    return out


def valu_exp(sbuf, pbuf):
    """P = exp2(exponent), packed to bf16 into P buffer `pbuf`, and the block's row sums of the fp32 values (plain adds
    in two chains per query block: measured cheaper than v_dot2c_f32_bf16 on the packed values against ones).  The
    exponents stay where they are: the rescale routine starts from them again."""
    out = []
    for qb in range(QB):
        for m in range(2):
            es = [SBUF(sbuf, qb) + 8 * m + i for i in range(8)]
            rs = [RT + 8 * ((2 * qb + m) % 3) + i for i in range(8)]
            for x, r in zip(es, rs):
                out.append((f"v_exp_f32 {vr(r)}, {vr(x)}", (), 2))
            for i in range(4):
                d = P16(pbuf, qb, m) + i
                out.append((f"v_cvt_pk_bf16_f32 {vr(d)}, {vr(rs[2 * i])}, {vr(rs[2 * i + 1])}", (d,), 1))
            for c in range(2):
                s = BSUM(qb, c)
                out.append((f"v_add_f32 {vr(s)}, {vr(rs[c])}, {vr(rs[2 + c])}" if m == 0 else f"v_add_f32 {vr(s)}, {vr(s)}, {vr(rs[c])}", (), 1))
                if m:
                    out.append((f"v_add_f32 {vr(s)}, {vr(s)}, {vr(rs[2 + c])}", (), 1))
            for i in range(4, 8):
                s = BSUM(qb, i % 2)
                out.append((f"v_add_f32 {vr(s)}, {vr(s)}, {vr(rs[i])}", (), 1))
    for qb in range(QB):
        out.append((f"v_add_f32 {vr(BSUM(qb, 0))}, {vr(BSUM(qb, 0))}, {vr(BSUM(qb, 1))}", (), 1))
    return out


def valu_take():
    """The block's row sums into the running ones."""
    return [f"v_add_f32 {vr(LSUM(qb))}, {vr(LSUM(qb))}, {vr(BSUM(qb, 0))}" for qb in range(QB)]


def gen_iter(p, cur, nxt, nxt2, par, seq, do_a=True, do_valu=True, head=None, prefetch=True, side=None, masked=False):
    """Block i = cur, i+1 = nxt (its V^T is prefetched at the tail), i+2 = nxt2 (its K feeds group A).
    par = i % 2: P(i) sits in P buffer par, S(i+1) in score buffer 1 - par, S(i+2) goes to score buffer par."""
    e = p.e
    e.comment(f"======== block {cur}: O^T += V^T P^T{cur} | S^T{nxt2} -> buffer {par} | softmax of {nxt}")
    reads = {k: [] for k in range(-1, NSLOT)}

    def plan(first_use, fn, n):                           # n LDS reads, LAT slots ahead
        reads[max(first_use - LAT, -1)].append((fn, n))

    slots = []
    for m in range(2):
        for db in range(DB):
            k = 2 * (DB * m + db)
            if not (m == 0 and db < 2):                   # requested at the tail of the block before
                plan(k, (lambda m=m, db=db: read_vt(p, cur, m, db, seq)), 2)
            for qb in range(QB):
                slots.append(("B", m, db, qb))
    if do_a:
        for ks in range(KS):
            plan(4 * DB + 2 * ks, (lambda ks=ks: read_k(p, nxt2, ks, seq)), 1)
            for qb in range(QB):
                slots.append(("A", ks, qb))
    else:
        slots += [None] * (2 * KS)
    if prefetch and nxt is not None:
        for db in range(2):
            reads[NSLOT - 3 + db].append(((lambda db=db: read_vt(p, nxt, 0, db, seq + 1)), 2))

    valu_e = valu_exp(1 - par, 1 - par) if do_valu else []
    vi = [0]
    left = 0

    def side_units(k):                                   # what stands beside the softmax behind MFMA slot k
        return sum(n for _, n in reads[k]) + (2 if side and k in side else 0)

    if head is not None:
        head()
    for fn, _ in reads[-1]:
        fn()
    for k, sl in enumerate(slots):
        if sl is not None and sl[0] == "B":
            _, m, db, qb = sl
            tag = f"t{seq}_{m}_{db}"
            e.need(tag)
            acc = ar(ACC(db, qb), 16)
            e.mfma(acc, vr(p.use(tag), 4), vr(P16(par, qb, m), 4), acc)
        elif sl is not None:
            _, ks, qb = sl
            tag = f"k{seq}_{ks}"
            e.need(tag)
            d = vr(SBUF(par, qb), 16)
            e.mfma(d, vr(p.use(tag), 4), ar(QF(qb, ks), 4), vr(NL(qb), 16) if ks == 0 else d)
        units = side_units(k)
        for fn, _ in reads[k]:
            fn()
        if side and k in side:                           # tile request / stream bookkeeping spread under the MFMAs
            for ln in side[k]:
                e.raw(ln)
        if do_valu and masked and k == 3:
            mask_test(e, S_NM1 if par else S_NM, 1 - par)
        if do_valu:
            # S(i+1) was written by the last group of the block before: first reader three MFMA issues later
            budget = BUDGET or -(-(sum(x[2] for x in valu_e[vi[0]:]) + sum(side_units(j) for j in range(k, BRANCH_SLOT))) // max(BRANCH_SLOT - k, 1))
            while 3 <= k < BRANCH_SLOT and vi[0] < len(valu_e) and units + valu_e[vi[0]][2] <= budget:
                e.valu(valu_e[vi[0]][0], valu_e[vi[0]][1])
                units += valu_e[vi[0]][2]
                vi[0] += 1
            if k == BRANCH_SLOT:
                left = len(valu_e) - vi[0]
                for text, writes, _ in valu_e[vi[0]:]:       # what did not fit under the MFMAs (the pipeline stalls on it)
                    e.valu(text, writes)
                # the common path falls through; the call sits out of line behind the loop (a taken branch costs a refetch)
                l_call, l_back = e.label("call"), e.label("back")
                e.raw(f"v_max_f32 {vr(SMAX)}, {vr(BSUM(0, 0))}, {vr(BSUM(1, 0))}")
                e.raw(f"v_cmp_gt_f32 vcc, {vr(SMAX)}, {vr(LIMR)}")
                e.raw("s_cmp_lg_u64 vcc, 0")
                e.raw(f"s_cbranch_scc1 {l_call}")
                e.raw(l_back + ":")
                STUBS.append((l_call, l_back, par))
                for ln in valu_take():
                    e.raw(ln)
    return left if do_a else 0


def mask_test(e, limit, buf):
    """Call the mask routine of score buffer `buf` if its block lies in one of the last S_NM tiles (the tile in hand is
    the T_REM-th from the end; limit = S_NM for a block of that tile, S_NM + 1 for one of the next)."""
    l_call, l_back = e.label("mcall"), e.label("mback")
    e.raw(f"s_cmp_le_u32 {sr(T_REM)}, {sr(limit)}")
    e.raw(f"s_cbranch_scc1 {l_call}")
    e.raw(l_back + ":")
    MASK_STUBS.append((l_call, l_back, buf))


def gen_mask_routine(e, kb):
    """Score buffer kb holds the exponents of key block kb of a masked tile: -inf wherever the key is not the row's.
    Key t of the tile (0 .. 63) is visible to a row iff t >= M_LO and M_REL + t <= the row's position, both relative to
    the position of the workgroup's first row.  Block 0 moves on to the next tile of the masked walk first."""
    n4, ninf, lim, lo = RT, RT + 1, RT + 2, RT + 4
    if kb == 0:
        l_step, l_go = e.label("mstep"), e.label("mgo")
        e.raw(f"s_cmp_lg_u32 {sr(M_LEFT)}, 0")
        e.raw(f"s_cbranch_scc1 {l_step}")
        e.raw(f"v_mov_b32 {vr(RT)}, {sr(S_MTBL)}")
        e.raw(f"ds_read_b128 {vr(RT + 4, 4)}, {vr(RT)} offset:16")
        e.raw("s_waitcnt lgkmcnt(0)")
        for i, dst in enumerate((M_LEFT, M_REL, M_LO)):
            e.raw(f"v_readfirstlane_b32 {sr(dst)}, {vr(RT + 4 + i)}")
        e.raw(f"s_add_u32 {sr(S_MTBL)}, {sr(S_MTBL)}, 32")
        e.raw(f"s_branch {l_go}")
        e.raw(l_step + ":")
        e.raw(f"s_add_i32 {sr(M_REL)}, {sr(M_REL)}, 64")
        e.raw(l_go + ":")
        e.raw(f"s_sub_u32 {sr(M_LEFT)}, {sr(M_LEFT)}, 1")
    e.raw(f"v_mbcnt_lo_u32_b32 {vr(n4)}, -1, 0")
    e.raw(f"v_mbcnt_hi_u32_b32 {vr(n4)}, -1, {vr(n4)}")
    e.raw(f"v_lshrrev_b32 {vr(n4)}, 5, {vr(n4)}")
    e.raw(f"v_lshlrev_b32 {vr(n4)}, 2, {vr(n4)}")
    e.raw(f"v_mov_b32 {vr(ninf)}, 0xff800000")
    for qb in range(QB):
        e.raw(f"v_subrev_u32 {vr(lim + qb)}, {sr(M_REL)}, {vr(QREL(qb))}")
        if kb:
            e.raw(f"v_subrev_u32 {vr(lim + qb)}, 32, {vr(lim + qb)}")

    def each(cmp, bound):
        for qb in range(QB):
            for v0 in range(0, 16, 4):              # four compares ahead of the four selects that read them
                for i in range(4):
                    e.raw(f"{cmp} {sr(T_CMP + 2 * i, 2)}, {vr(bound(qb))}, {8 * (v0 // 4) + i}")
                for i in range(4):
                    x = vr(SBUF(kb, qb) + v0 + i)
                    e.raw(f"v_cndmask_b32_e64 {x}, {vr(ninf)}, {x}, {sr(T_CMP + 2 * i, 2)}")
    each("v_cmp_ge_i32_e64", lambda qb: lim + qb)
    l_nolo = e.label("mnolo")
    e.raw(f"s_cmp_eq_u32 {sr(M_LO)}, 0")
    e.raw(f"s_cbranch_scc1 {l_nolo}")
    e.raw(f"v_sub_u32 {vr(lo)}, {sr(M_LO)}, {vr(n4)}")
    if kb:
        e.raw(f"v_subrev_u32 {vr(lo)}, 32, {vr(lo)}")
    each("v_cmp_le_i32_e64", lambda qb: lo)
    e.raw(l_nolo + ":")
    l_ret = e.label("mret")
    e.raw(f"s_cmp_eq_u32 {sr(S_FRESH)}, 0")
    e.raw(f"s_cbranch_scc1 {l_ret}")
    mx, t, k = RT + 8, RT + 10, RT + 12
    for qb in range(QB):
        x = SBUF(kb, qb)
        e.raw(f"v_max3_f32 {vr(mx + qb)}, {vr(x)}, {vr(x + 1)}, {vr(x + 2)}")
        for v in range(3, 15, 2):
            e.raw(f"v_max3_f32 {vr(mx + qb)}, {vr(mx + qb)}, {vr(x + v)}, {vr(x + v + 1)}")
        e.raw(f"v_max_f32 {vr(mx + qb)}, {vr(mx + qb)}, {vr(x + 15)}")
        e.raw(f"v_mov_b32 {vr(t + qb)}, {vr(mx + qb)}")
    e.raw("s_nop 1")
    for qb in range(QB):
        e.raw(f"v_permlane32_swap_b32 {vr(t + qb)}, {vr(mx + qb)}")
    e.raw("s_nop 1")
    for qb in range(QB):
        e.raw(f"v_max_f32 {vr(mx + qb)}, {vr(mx + qb)}, {vr(t + qb)}")
        e.raw(f"v_cmp_neq_f32_e64 {sr(T_CMP, 2)}, {vr(ninf)}, {vr(mx + qb)}")
        e.raw(f"v_cmp_eq_u32_e64 {sr(T_CMP + 2, 2)}, 0, {vr(SEEN(qb))}")
        e.raw("s_nop 1")
        e.raw(f"s_and_b64 {sr(T_CMP, 2)}, {sr(T_CMP, 2)}, {sr(T_CMP + 2, 2)}")
        e.raw("s_nop 1")
        e.raw(f"v_cndmask_b32_e64 {vr(k + qb)}, 0, {vr(mx + qb)}, {sr(T_CMP, 2)}")
        e.raw(f"v_cndmask_b32_e64 {vr(SEEN(qb))}, {vr(SEEN(qb))}, 1, {sr(T_CMP, 2)}")
        for v in range(16):
            e.raw(f"v_sub_f32 {vr(NL(qb) + v)}, {vr(NL(qb) + v)}, {vr(k + qb)}")
        for v in range(16):
            e.raw(f"v_sub_f32 {vr(SBUF(kb, qb) + v)}, {vr(SBUF(kb, qb) + v)}, {vr(k + qb)}")
    e.raw(l_ret + ":")
    e.raw("s_nop 1")
    e.raw(f"s_setpc_b64 {sr(T_MRET, 2)}")


def gen_rescale_routine(e, par):
    """Called when some row's sum over the block whose softmax has just been done exceeds the limit 2^(GAP + 4): its
    largest exponent exceeds GAP then (a lane's sum has 16 terms), or was too large for exp2.  Nothing of that block has
    been used: its exponents still sit in score buffer 1 - par, its P in P buffer 1 - par and its sums apart.  Moves the
    reference of these rows up by k = ceil(maximum) log2 units: accumulators and running sums are multiplied by 2^-k
    (exact), k is taken off the exponents of this block, off those of the next one (score buffer par; an MFMA or two that
    add to them are still to come) and off the start values of the S^T accumulators; then the softmax is done again."""
    e.raw("s_nop 7")
    e.raw("s_nop 7")
    e.raw("s_nop 7")
    for qb in range(QB):
        x = SBUF(1 - par, qb)
        e.raw(f"v_max3_f32 {vr(MX(qb))}, {vr(x)}, {vr(x + 1)}, {vr(x + 2)}")
        for v in range(3, 15, 2):
            e.raw(f"v_max3_f32 {vr(MX(qb))}, {vr(MX(qb))}, {vr(x + v)}, {vr(x + v + 1)}")
        e.raw(f"v_max_f32 {vr(MX(qb))}, {vr(MX(qb))}, {vr(x + 15)}")
    for ln in valu_exchange():          # both halves of a query column must move their reference by the same amount
        e.raw(ln)
    for ln in valu_exchange(lambda qb: BSUM(qb, 0)):
        e.raw(ln)
    alpha = [RT, RT + 1]
    for qb in range(QB):
        k, ki = RT + 2 + qb, RT + 4 + qb
        e.raw(f"v_ceil_f32 {vr(k)}, {vr(MX(qb))}")
        e.raw(f"v_cmp_gt_f32 vcc, {vr(BSUM(qb, 0))}, {vr(LIMR)}")
        e.raw("s_nop 1")
        e.raw(f"v_cndmask_b32 {vr(k)}, 0, {vr(k)}, vcc")
        for reg in (NL(qb), SBUF(0, qb), SBUF(1, qb)):
            for v in range(16):
                e.raw(f"v_sub_f32 {vr(reg + v)}, {vr(reg + v)}, {vr(k)}")
        e.raw(f"v_cvt_i32_f32 {vr(ki)}, {vr(k)}")
        e.raw(f"v_sub_u32 {vr(ki)}, 0, {vr(ki)}")
        e.raw(f"v_ldexp_f32 {vr(alpha[qb])}, 1.0, {vr(ki)}")
        e.raw(f"v_mul_f32 {vr(LSUM(qb))}, {vr(alpha[qb])}, {vr(LSUM(qb))}")
    t = RT + 8
    for qb in range(QB):
        for db in range(DB):
            for v0 in range(0, 16, 8):
                for i in range(8):
                    e.raw(f"v_accvgpr_read_b32 {vr(t + i)}, {ar(ACC(db, qb) + v0 + i)}")
                for i in range(8):
                    e.raw(f"v_mul_f32 {vr(t + i)}, {vr(alpha[qb])}, {vr(t + i)}")
                for i in range(8):
                    e.raw(f"v_accvgpr_write_b32 {ar(ACC(db, qb) + v0 + i)}, {vr(t + i)}")
    for text, _, _ in valu_exp(1 - par, 1 - par):
        e.raw(text)
    e.raw("s_nop 3")
    e.raw(f"s_setpc_b64 {sr(T_RET, 2)}")


def dma_groups(stage):
    """The direct-to-LDS loads of one K / V tile into LDS stage `stage`: one [M0 setup, gap, load] group per load."""
    g = []
    for j in range(NDMA):
        g.append([f"s_add_u32 m0, {sr(T_M0)}, {KT(stage) + 4096 * j}", "s_nop 0",
                  f"global_load_lds_dwordx4 {vr(KOFF + j)}, {sr(D_KPTR, 2)}"])
        g.append([f"s_add_u32 m0, {sr(T_M0)}, {VT(stage) + 4096 * j}", "s_nop 0",
                  f"global_load_lds_dwordx4 {vr(VOFF + j)}, {sr(D_VPTR, 2)}"])
    return g


def advance_lines(e):
    """Move the K / V stream to the next tile of the walk (it stays on the last tile once all S_NT tiles have been
    requested).  The common path falls through; the switch to the next chunk of the table sits out of line."""
    l_skip, l_next = e.label("skip"), e.label("nextchunk")
    NEXT_STUBS.append((l_next, l_skip))
    return [f"s_add_u32 {sr(T_X)}, {sr(D_IDX)}, 1",
            f"s_cmp_ge_u32 {sr(T_X)}, {sr(S_NT)}",
            f"s_cbranch_scc1 {l_skip}",
            f"s_mov_b32 {sr(D_IDX)}, {sr(T_X)}",
            f"s_sub_u32 {sr(D_LEFT)}, {sr(D_LEFT)}, 1",
            f"s_cmp_eq_u32 {sr(D_LEFT)}, 0",
            f"s_cbranch_scc1 {l_next}",
            f"s_add_u32 {sr(D_KPTR)}, {sr(D_KPTR)}, {sr(S_KTILE)}",
            f"s_addc_u32 {sr(D_KPTR + 1)}, {sr(D_KPTR + 1)}, 0",
            f"s_add_u32 {sr(D_VPTR)}, {sr(D_VPTR)}, {sr(S_VTILE)}",
            f"s_addc_u32 {sr(D_VPTR + 1)}, {sr(D_VPTR + 1)}, 0",
            l_skip + ":"]


def gen_dma(e, stage):
    """Request a tile and advance the stream, in one piece (prologue)."""
    for grp in dma_groups(stage):
        for ln in grp:
            e.raw(ln)
    for ln in advance_lines(e):
        e.raw(ln)


def gen_table_entry(e):
    e.raw(f"v_mov_b32 {vr(TMP)}, {sr(D_TBL)}")
    e.raw(f"ds_read_b128 {vr(TMP + 2, 4)}, {vr(TMP)}")
    e.raw(f"ds_read_b32 {vr(TMP + 6)}, {vr(TMP)} offset:16")
    e.raw("s_waitcnt lgkmcnt(0)")
    for i, dst in enumerate((D_KPTR, D_KPTR + 1, D_VPTR, D_VPTR + 1, D_LEFT)):
        e.raw(f"v_readfirstlane_b32 {sr(dst)}, {vr(TMP + 2 + i)}")
    e.raw(f"s_add_u32 {sr(D_TBL)}, {sr(D_TBL)}, 32")


def generate():
    e = Emitter()
    p = Pipe(e)
    l_rare = [e.label("rescale0"), e.label("rescale1")]
    l_mask = [e.label("mask0"), e.label("mask1")]
    e.comment("---- prologue")
    e.raw(f"s_lshl_b32 {sr(T_M0)}, {sr(S_WAVE)}, 10")
    e.raw(f"s_add_u32 {sr(T_M0)}, {sr(T_M0)}, {sr(S_LDS)}")
    e.raw(f"s_mov_b32 {sr(T_REM)}, {sr(S_NT)}")
    e.raw(f"s_mov_b32 {sr(D_IDX)}, 0")
    e.raw(f"s_mov_b32 {sr(D_TBL)}, {sr(S_TBL)}")
    for dst, target in [(T_RARE + 2 * b, l_rare[b]) for b in range(2)] + [(T_MASK + 2 * b, l_mask[b]) for b in range(2)]:
        l_here = e.label("here")
        e.raw(f"s_getpc_b64 {sr(dst, 2)}")
        e.raw(l_here + ":")
        e.raw(f"s_add_u32 {sr(dst)}, {sr(dst)}, {target}-{l_here}")
        e.raw(f"s_addc_u32 {sr(dst + 1)}, {sr(dst + 1)}, 0")
    e.raw(f"v_mov_b32 {vr(TMP)}, {sr(S_TBL)}")
    e.raw(f"ds_read_b128 {vr(TMP + 4, 4)}, {vr(TMP)} offset:{PARAMS}")
    e.raw(f"ds_read_b32 {vr(TMP + 8)}, {vr(TMP)} offset:{PARAMS + 16}")
    e.raw("s_waitcnt lgkmcnt(0)")
    for i, dst in enumerate((S_NM, S_MTBL, S_FRESH, S_OLOW, S_OLOW + 1)):
        e.raw(f"v_readfirstlane_b32 {sr(dst)}, {vr(TMP + 4 + i)}")
    e.raw(f"s_add_u32 {sr(S_NM1)}, {sr(S_NM)}, 1")
    e.raw(f"s_mov_b32 {sr(M_LEFT)}, 0")
    for qb in range(QB):
        e.raw(f"v_mov_b32 {vr(QREL(qb))}, {vr(I_QREL + qb)}")
        e.raw(f"v_mov_b32 {vr(SEEN(qb))}, 1")
        e.raw(f"v_and_b32 {vr(TMP)}, {1 << qb}, {vr(I_LIVE)}")
        e.raw(f"v_cmp_ne_u32_e64 {sr(S_LIVE + 2 * qb, 2)}, 0, {vr(TMP)}")
    e.raw(f"v_mov_b32 {vr(TMP)}, 0x3fb8aa3b")
    e.raw(f"v_mul_f32 {vr(TMP)}, {sr(S_SCALE)}, {vr(TMP)}")
    e.raw("s_nop 0")
    e.raw(f"v_readfirstlane_b32 {sr(S_CEXP)}, {vr(TMP)}")
    e.raw(f"v_mov_b32 {vr(LIMR)}, {sr(S_LIMIT)}")
    e.raw(f"v_mov_b32 {vr(KOFF)}, {vr(I_KOFF0)}")
    e.raw(f"v_mov_b32 {vr(VOFF)}, {vr(I_VOFF0)}")
    e.raw(f"v_mov_b32 {vr(OOFF)}, {vr(I_OOFF)}")
    e.raw(f"v_mov_b32 {vr(LSEOFF)}, {vr(I_LSEOFF)}")
    for j in range(1, NDMA):
        e.raw(f"v_add_u32 {vr(KOFF + j)}, {sr(S_KRS16)}, {vr(KOFF + j - 1)}")
        e.raw(f"v_add_u32 {vr(VOFF + j)}, {sr(S_VRS16)}, {vr(VOFF + j - 1)}")
    gen_table_entry(e)
    for st in range(3):
        gen_dma(e, st)
    e.comment("Q fragments (B operands) -> AGPRs; lane = query column, elements 16 ks + 8 (lane / 32) .. + 7")
    for qb, qrow in enumerate((I_QROW0, I_QROW1)):
        for ks in range(KS):
            e.raw(f"global_load_dwordx4 {vr(4 * (KS * qb + ks), 4)}, {vr(qrow, 2)}, off offset:{32 * ks}")
    for ks in range(KS):
        e.raw(f"v_xor_b32 {vr(TMP)}, {32 * ks}, {vr(I_GF16)}")
        e.raw(f"v_add_u32 {vr(XL + ks)}, {vr(I_XBASE)}, {vr(TMP)}")
        if SPLIT:
            e.raw(f"v_add_u32 {vr(XH + ks)}, 0x10000, {vr(XL + ks)}")
    for db in range(DB):
        e.raw(f"v_xor_b32 {vr(TMP)}, {64 * db}, {vr(I_LF16)}")
        e.raw(f"v_add_u32 {vr(TRLO_L + db)}, {vr(I_TRBASE)}, {vr(TMP)}")
        e.raw(f"v_xor_b32 {vr(TMP)}, {(64 * db) ^ 32}, {vr(I_LF16)}")
        e.raw(f"v_add_u32 {vr(TRHI_L + db)}, {vr(I_TRBASE)}, {vr(TMP)}")
        e.raw(f"v_add_u32 {vr(TRHI_L + db)}, {8 * ROW}, {vr(TRHI_L + db)}")
        if SPLIT:
            e.raw(f"v_add_u32 {vr(TRLO_H + db)}, 0x10000, {vr(TRLO_L + db)}")
            e.raw(f"v_add_u32 {vr(TRHI_H + db)}, 0x10000, {vr(TRHI_L + db)}")
    for i in range(32 * DB):
        e.raw(f"v_accvgpr_write_b32 {ar(i)}, 0")
    for qb in range(QB):
        e.raw(f"v_mov_b32 {vr(LSUM(qb))}, 0")
    e.raw("s_waitcnt vmcnt(0)")
    e.comment("Q <- bf16(Q * scale * log2(e)): the MFMAs then deliver exponents in log2 units")
    for i in range(0, 8 * KS, 4):
        for j in range(4):
            e.raw(f"v_lshlrev_b32 {vr(64 + 2 * j)}, 16, {vr(i + j)}")
            e.raw(f"v_and_b32 {vr(65 + 2 * j)}, 0xffff0000, {vr(i + j)}")
        for j in range(8):
            e.raw(f"v_mul_f32 {vr(64 + j)}, {sr(S_CEXP)}, {vr(64 + j)}")
        for j in range(4):
            e.raw(f"v_cvt_pk_bf16_f32 {vr(i + j)}, {vr(64 + 2 * j)}, {vr(65 + 2 * j)}")
    for i in range(8 * KS):
        e.raw(f"v_accvgpr_write_b32 {ar(128 + i)}, {vr(i)}")
    e.raw("s_barrier")

    e.comment("---- pipeline fill: exponents of tile 0 from zero, reference; P and row sums of its first block")

    def fill_s(blk, buf, seq, c_init):
        for ks in range(KS):
            read_k(p, blk, ks, seq)
            if ks % 4 == 3:
                for k2 in range(ks - 3, ks + 1):
                    e.need(f"k{seq}_{k2}")
                    for qb in range(QB):
                        d = vr(SBUF(buf, qb), 16)
                        e.mfma(d, vr(p.use(f"k{seq}_{k2}"), 4), ar(QF(qb, k2), 4), c_init(qb) if k2 == 0 else d)

    for kb in range(2):
        fill_s((0, kb), kb, kb - 2, lambda qb: "0")
    e.raw("s_nop 7")
    e.raw("s_nop 7")
    for kb in range(2):
        mask_test(e, S_NM, kb)
    for qb in range(QB):                        # with r = 0: d = row maximum of S c
        x = [SBUF(kb, qb) + v for kb in range(2) for v in range(16)]
        e.raw(f"v_max_f32 {vr(MX(qb))}, {vr(x[0])}, {vr(x[1])}")
        for v in range(2, 32, 2):
            e.raw(f"v_max3_f32 {vr(MX(qb))}, {vr(MX(qb))}, {vr(x[v])}, {vr(x[v + 1])}")
    for ln in valu_exchange():
        e.raw(ln)
    for qb in range(QB):                        # reference = the maximum (its P is 1, exactly); shift the tile by hand
        e.raw(f"v_mov_b32 {vr(TMP)}, 0xff800000")
        e.raw(f"v_cmp_neq_f32 vcc, {vr(TMP)}, {vr(MX(qb))}")
        e.raw("s_nop 1")
        e.raw(f"v_cndmask_b32 {vr(MX(qb))}, 0, {vr(MX(qb))}, vcc")      # a row that sees no key of this tile: zero
        e.raw(f"v_cndmask_b32_e64 {vr(SEEN(qb))}, 0, 1, vcc")
        for v in range(16):
            e.raw(f"v_sub_f32 {vr(NL(qb) + v)}, 0, {vr(MX(qb))}")
        for kb in range(2):
            for v in range(16):
                e.raw(f"v_sub_f32 {vr(SBUF(kb, qb) + v)}, {vr(SBUF(kb, qb) + v)}, {vr(MX(qb))}")
    for text, writes, _ in valu_exp(0, 0):
        e.valu(text, writes)
    for ln in valu_take():
        e.raw(ln)
    for db in range(2):
        read_vt(p, (0, 0), 0, db, 0)

    l_done = e.label("done")
    l_loop = e.label("loop")
    l_masked = [e.label(f"masked{u}") for u in range(NS)]
    strip = lambda tags: [t.split("_", 1)[1] for t in tags]
    leftover = 0

    def tile(u, seq, masked):
        nonlocal leftover
        un = (u + 1) % NS

        def head():
            # tile T + 1 has landed everywhere and nobody reads tile T - 1 any more: tile T + 3 may be requested
            e.raw(f"s_waitcnt vmcnt({2 * NDMA})")
            e.raw("s_barrier")
        side = {k: grp for k, grp in enumerate(dma_groups((u + 3) % NS))}
        side[2 * NDMA] = advance_lines(e)
        leftover += gen_iter(p, (u, 0), (u, 1), (un, 0), 0, seq, head=head, side=side, masked=masked)
        leftover += gen_iter(p, (u, 1), (un, 0), (un, 1), 1, seq + 1, masked=masked)
        e.raw(f"s_sub_u32 {sr(T_REM)}, {sr(T_REM)}, 1")

    e.comment("---- tiles T with T and T + 1 whole")
    if D == 64:
        # Where the loop lies among the 64-byte lines of the instruction cache was 1 to 3 % at this head size when the loop still
        # kept a row maximum (24 heads x 16384 rows x 131072 keys 12.3 ms from byte 4 of a line, 12.4 from 16, 32 or 48, 12.5
        # to 12.6 from 0 or 8; 11.1 today from byte 4, the others not measured again).  At 128 it is nothing.
        e.raw(".p2align 6")
        e.raw("s_nop 0")
    e.raw(l_loop + ":")
    start = p.snapshot()
    at = []
    for u in range(NS):
        e.raw(f"s_cmp_le_u32 {sr(T_REM)}, {sr(S_NM1)}")
        e.raw(f"s_cbranch_scc1 {l_masked[u]}")
        at.append(strip(e.ds))
        tile(u, 2 * u, False)
    assert strip(e.ds) == at[0], (e.ds, at[0])
    e.raw(f"s_branch {l_loop}")
    e.comment("---- the last ones")
    p.restore(start)
    drains = []
    for u in range(NS):
        e.raw(l_masked[u] + ":")
        assert strip(e.ds) == at[u], (e.ds, at[u])
        l_drain = e.label("drain")
        e.raw(f"s_cmp_eq_u32 {sr(T_REM)}, 1")
        e.raw(f"s_cbranch_scc1 {l_drain}")
        drains.append((l_drain, u, p.snapshot(), 2 * u))
        tile(u, 2 * u, True)
    assert strip(e.ds) == at[0], (e.ds, at[0])
    e.raw(f"s_branch {l_masked[0]}")
    for l_drain, u, snap, sq in drains:
        e.raw(l_drain + ":")
        p.restore(snap)
        # the last tile: its second block still needs its softmax, nothing beyond it exists
        gen_iter(p, (u, 0), (u, 1), None, 0, sq, do_a=False, masked=True)
        e.raw("s_nop 7")                 # the exponentials above were not hidden under a second MFMA group
        gen_iter(p, (u, 1), None, None, 1, sq + 1, do_a=False, do_valu=False, prefetch=False)
        e.raw(f"s_branch {l_done}")
    for l_next, l_skip in NEXT_STUBS:
        e.raw(l_next + ":")
        gen_table_entry(e)
        e.raw(f"s_branch {l_skip}")
    for l_call, l_back, par in STUBS:
        e.raw(l_call + ":")
        e.raw(f"s_swappc_b64 {sr(T_RET, 2)}, {sr(T_RARE + 2 * par, 2)}")
        e.raw(f"s_branch {l_back}")
    for l_call, l_back, buf in MASK_STUBS:
        e.raw(l_call + ":")
        e.raw(f"s_swappc_b64 {sr(T_MRET, 2)}, {sr(T_MASK + 2 * buf, 2)}")
        e.raw(f"s_branch {l_back}")
    for b in range(2):
        e.raw(l_rare[b] + ":")
        gen_rescale_routine(e, b)
        e.raw(l_mask[b] + ":")
        gen_mask_routine(e, b)
    e.raw(l_done + ":")
    e.raw("s_waitcnt vmcnt(0) lgkmcnt(0)")

    e.comment("---- epilogue: O = acc / l, lse = (log2(l) + r) ln 2; lane = query row, 4 consecutive d per 16-byte store")
    e.raw("s_nop 7")
    e.raw("s_nop 7")
    for qb in range(QB):
        l, t = TMP, TMP + 1
        e.raw(f"v_mov_b32 {vr(l)}, {vr(LSUM(qb))}")
        e.raw(f"v_mov_b32 {vr(t)}, {vr(LSUM(qb))}")
        e.raw("s_nop 1")
        e.raw(f"v_permlane32_swap_b32 {vr(t)}, {vr(l)}")
        e.raw("s_nop 1")
        e.raw(f"v_add_f32 {vr(l)}, {vr(l)}, {vr(t)}")
        e.raw(f"v_rcp_f32 {vr(TMP + 2)}, {vr(l)}")
        e.raw(f"v_log_f32 {vr(TMP + 3)}, {vr(l)}")
        e.raw(f"v_cmp_lt_f32 vcc, 0, {vr(l)}")                     # a row without a visible key: O = 0, lse = -inf
        e.raw("s_nop 1")
        e.raw(f"v_cndmask_b32 {vr(TMP + 2)}, 0, {vr(TMP + 2)}, vcc")
        e.raw(f"v_sub_f32 {vr(TMP + 3)}, {vr(TMP + 3)}, {vr(NL(qb))}")
        e.raw(f"v_mul_f32 {vr(TMP + 3)}, 0x3f317218, {vr(TMP + 3)}")
        if qb == 1:
            e.raw(f"v_add_u32 {vr(OOFF)}, {sr(S_OQB)}, {vr(OOFF)}")
            e.raw(f"v_add_u32 {vr(LSEOFF)}, 128, {vr(LSEOFF)}")
        e.raw(f"s_mov_b64 exec, {sr(S_LIVE + 2 * qb, 2)}")
        for db in range(DB):
            for j in range(4):
                t0 = 4 * (4 * db + j)
                for i in range(4):
                    e.raw(f"v_accvgpr_read_b32 {vr(t0 + i)}, {ar(ACC(db, qb) + 4 * j + i)}")
                e.raw("s_nop 0")
                for i in range(4):
                    e.raw(f"v_mul_f32 {vr(t0 + i)}, {vr(TMP + 2)}, {vr(t0 + i)}")
                e.raw(f"global_store_dwordx4 {vr(OOFF)}, {vr(t0, 4)}, {sr(S_OPTR, 2)} offset:{128 * db + 32 * j}")
        l_nolow = e.label("nolow")
        e.raw(f"s_cmp_eq_u64 {sr(S_OLOW, 2)}, 0")
        e.raw(f"s_cbranch_scc1 {l_nolow}")
        e.raw(f"v_lshrrev_b32 {vr(TMP + 4)}, 1, {vr(OOFF)}")
        for db in range(DB):
            for j in range(4):
                t0, d = 4 * (4 * db + j), 64 + 2 * (4 * db + j)
                e.raw(f"v_cvt_pk_bf16_f32 {vr(d)}, {vr(t0)}, {vr(t0 + 1)}")
                e.raw(f"v_cvt_pk_bf16_f32 {vr(d + 1)}, {vr(t0 + 2)}, {vr(t0 + 3)}")
                e.raw(f"global_store_dwordx2 {vr(TMP + 4)}, {vr(d, 2)}, {sr(S_OLOW, 2)} offset:{64 * db + 16 * j}")
        e.raw(l_nolow + ":")
        # lse: one lane per row (the lower half of the wavefront)
        e.raw("s_mov_b32 exec_hi, 0")
        e.raw(f"global_store_dword {vr(LSEOFF)}, {vr(TMP + 3)}, {sr(S_LSEPTR, 2)}")
        e.raw("s_mov_b64 exec, -1")
        e.raw("s_waitcnt vmcnt(0)")
    return e, leftover


def main():
    e, leftover = generate()
    if leftover:
        sys.stderr.write(f"gen_fwd_asm: {leftover} VALU instructions did not fit under the MFMAs\n")
    clob = [f"v{i}" for i in range(256) if not 224 <= i < 240] + [f"a{i}" for i in range(256)]
    clob += [f"s{i}" for i in range(S_CEXP, 94)]
    write_inc(sys.stdout, "gen_fwd_asm.py" + (" 64" if D == 64 else ""), "ST_FWD_FAST" + ("64" if D == 64 else ""), e,
              LDS_BYTES, clob)


if __name__ == "__main__":
    main()
