#!/usr/bin/env python3
"""Generates the gfx950 assembly of the loop that makes dK, dV and dQ in one walk (head_dim 128, or 64) as a C string literal.

    python gen_bwd_one_asm.py > st_bwd_one_asm.inc          (build.py does this before compiling)
    python gen_bwd_one_asm.py 64 > st_bwd_one64_asm.inc     (head_dim 64)

The walk, the masks, the statistics and the epilogue are those of gen_bwd_dkv_asm.py; what is said there holds here.  Five contractions
a pair in place of the seven that the loop there and the one of gen_bwd_dq_asm.py execute: S and dP are not made again for dQ.

  * Head size 128: the packed dS of a block goes to LDS as [key][row] (two buffers; rows padded to 72 bytes, so that the 8-byte writes
    and the transposing reads meet few bank conflicts).  From the barrier of the next block on, wavefront w contracts all 256 keys of it with
    columns 32 w .. 32 w + 31 of K: dQ^T[32 x 32] += K^T dS^T, sixteen MFMAs spread to the barrier after that.  K lies in LDS for
    this, as the tile that S reads; V is resident instead.
  * dQ of a (head, block) pair, 16 KiB, travels from key tile to key tile of its KV head through a workspace in the order of the walk
    (and of the accumulator registers: 1 KiB an access; read and written where dQ lies, in rows of 16 KiB, the exchange cost more than
    the two contractions).  A wavefront reads what the tile before has left, adds its own and stores it; key tile i may read a pair
    when wavefront w of tile i - 1 has counted it done.  All of them run on one XCD, whose L2 the loads (sc1: past
    the L1) and stores meet in.  The first tile reads zeros.  Every sum has a fixed order; a pass behind the launch multiplies them by
    the softmax scale and adds them to dQ.
  * Under way two pairs behind the block in hand: pair x is contracted behind the barrier of block x + 1, read in block x + 2
    (into the registers that the exponents' start values have just left), added and stored before its barrier, and counted
    when the stores are acknowledged.  Pairs -2 and -1 do not exist; the workspace has room for them.
  * LDS rows of Q', dO and K tiles: groups of four rows (1 KiB, what one direct-to-LDS load fills), 16 bytes between groups; the
    16-byte chunk c of row r lies at c ^ 4 (r % 4).  Conflict-free like the swizzle of the other loops, and all but two bits of an
    offset are immediates, which leaves the sixteen registers that dQ's accumulator takes.
  * Three stages of tiles, two blocks ahead; with the two buffers of dS six copies of the block make the loop.

What bounds it: the matrix cores at the chip's power limit, as with the two loops it replaces.  Its instruction mix without dependences and
global memory operations (gen_probe_asm.py, "one": 80 MFMAs, 40 16-byte and 96 transposing LDS reads, 8 writes, 112 VALU instructions per block
and wavefront) reaches 1451 TFLOP/s on normal values, the walk of 32/8 heads x 4096 rows x 32 chunks 1294 on that card, and the two
passes, each within 1 % of its mix, execute 14/10 of the work at 1495 and 1569.  The rest is the exchange of sums, waits of the chain and, of the 150 us of a
tile of 64 blocks, 25 before and behind the loop.  Backward of that share 20.0 -> 16.8 ms, 32 heads x 2048 rows x 16 chunks 2.75 -> 2.39.
Where the MFMAs of a pair lie in the block, how far ahead their operands are read and how much side work a slot gets moved that by less than
1 % each; half of them under the first phase, whose reads are the densest, cost 3 %.

Head size 64 differs where half as many MFMAs leave less time to hide the rest in, and half as many registers are taken:
  * K is resident too, as the fragments of S and, in accumulator registers, as those of K^T; so are the fragments of dS^T.  Four stages
    of tiles, three blocks ahead.
  * A wavefront makes 16 columns of dQ from all keys (MFMAs of 16 x 16 x 32), so that a pair is 8 KiB.  With 32 columns from half the
    keys it reads half as much of dS, but the exchange is of two halves: 30.6 instead of 33.3 ms below; without any exchange 27.5.
  * What the tile before left is loaded into the accumulators themselves, a block ahead, and nothing is added up.  Two sets of sums.
  * All MFMAs of a pair behind the barrier, two a slot, every second slot (three slots apart 30.9 ms, in one block of eight slots 29.9);
    eleven units of side work a slot (nine and ten 2 to 3 % slower).
Backward of 24 heads x 16384 rows x 8 chunks, no mask: 34.6 -> 29.6 ms.
"""
import os
import sys

import gen_bwd_dkv_asm as kv
from gen_bwd_dkv_asm import (ACC_K, ACC_V, DB, DP0, KS, ND, NDQ, NINF, NKB, NL, NSLOT, P16, P2, P3, P4, POOL0, S0, ST, TMP,
                             S_CI, S_CI0, S_DIAG, S_EVT, S_FLAGS, S_GREC, S_LDS, S_NIN, S_NRAG, S_NSTEPS, S_QOUT, S_ROWS, S_SQ, S_VRS, S_WAVE, T_CMP,
                             T_DBLK, T_DLHEAD, T_INC, T_DLPTR, T_DOHEAD, T_DOPTR, T_DSTEP, T_HIMASK, T_LSEHEAD, T_LSEPTR, T_M0, T_MASK, T_MRET, T_MT,
                             T_OHI, T_QHEAD, T_QPTR, T_REM, T_VPTR, T_X)
from st_asmgen import Emitter, ar, sr, vr, write_inc

D = kv.D
NS, PF, COPIES = (3, 2, 6) if D == 128 else (4, 3, 4)
GRP = 1024 + 16                                      # bytes from one group of rows (four, or eight of head size 64) to the next
def rows(n): return n * 2 * D // 1024 * GRP          # bytes of n rows, whole groups
TQ = rows(32)
def QT(s): return 1024 + 2 * TQ * s
def DOT(s): return 1024 + 2 * TQ * s + TQ
TILES = 1024 + 2 * TQ * NS
DSR_ROW = 72                                         # bytes of a key's 32 dS
DS_BYTES = 256 * DSR_ROW
KT = TILES                                           # K tile; head size 64 has it in fragments, and only at the start in the place of dS
DS0 = KT + (rows(256) if D == 128 else 0)
assert D == 128 or rows(256) <= 2 * DS_BYTES
PBLK = DS0 + 2 * DS_BYTES                            # as in gen_bwd_dkv_asm.py; it stays, the mask routine reads it
NUNI = 20                                            # words of the uniform block behind it
LDS_BYTES = PBLK + 256 * 32 + 4 * NUNI
assert LDS_BYTES <= 163840 and PBLK >= 4 * 2 * 32 * (4 * D + 16)
# words of the uniform block behind the six of gen_bwd_dkv_asm.py: what only the epilogue needs
U_DKPTR, U_DVPTR, U_RS32, U_SCALE, U_FLAGS, U_DKLP, U_DVLP = 8, 10, 12, 13, 14, 16, 18
U_PLENTY = 6                                         # address of the count that is never too low, which a wait that gives up goes over to
GAVE_UP = 64                                         # from there to the word that says so (OneRoom::gave_up)
NP = D // 32                                         # accesses of 1 KiB that a wavefront's part of a pair takes
SLICE = 1024 * NP                                    # the part in the workspace
PAIR = 4 * SLICE

# registers
VF = kv.KF                                           # resident V fragments
def KR(nb, ks): return 32 + VF(nb, ks)               # head size 64: resident K fragments of S
def KTF(t): return 64 + 4 * t                        # and of K^T, in accumulator registers that dK and dV leave
def DSF(t): return 192 + 4 * (t % 8)                 # of dS^T
def ACC64(x): return 96 + 4 * NP * (x % 2)           # as the sums of a pair are
X, XK, TR, KTR, DSW, DSR, DQO, FLG = 216, 220, 224, 228, 229, 230, 231, 232
QOFF, DOOFF, STAT_G, STAT_L, G16, ACC_Q = 233, 235, 237, 238, 239, 240
OLD = NL                                             # what the tile before left, from slot 3 to the stores
MASK_HIGH = FLG if D == 128 else XK                  # a register that is free when the masks are made
# scalars in the places of the epilogue's inputs
S_DQL, S_DQW, S_DQINC, S_POLLS, S_CNT, S_PRED, S_OWN = 52, 54, 57, 58, 59, 60, 62

LAT = int(os.environ.get("ST_GEN_ONE_LAT", 3))
LATQ = 3                                             # the same for the operands of a pair
BUDGET = int(os.environ.get("ST_GEN_ONE_BUDGET", 6 if D == 128 else 11))
BUDGET_Q = 4                                         # issue units behind an MFMA of a pair
EARLY = 12
SYNC_SLOT, PUBLISH_SLOT = P3 - 1, P3 - 6
# slots behind which the MFMAs of a pair are issued, from the barrier of one block (slot 32 on) to that of the next (64 + 26)
DQ_AT = [35, 37, 39, 41, 43, 45, 47, 49, 52, 55, 58, 61, 80, 82, 84, 86] if D == 128 else [19 + 2 * (t // 2) for t in range(16)]
N_DQ = 16                                            # head size 64: of 16 columns, 32 keys and 16 rows
assert len(DQ_AT) == N_DQ and DQ_AT == sorted(DQ_AT) and DQ_AT[0] - LATQ > SYNC_SLOT and DQ_AT[-1] <= NSLOT + P3 - (6 if D == 128 else 8)
N_A = sum(1 for p in DQ_AT if p < NSLOT)             # of them in the block behind the pair's own
SUM_SLOT = P3 - 3                                    # the sums behind this slot, the stores behind the next
NREQ = 2 + 2 * NDQ


class Pool(kv.Pool):
    """Head size 64 has the fragments of dS^T in accumulator registers, and eight here, which divides the sixteen a block has left."""
    size = kv.Pool.size if D == 128 else 8

    def __init__(self):
        super().__init__()
        self.ds = {}

    def alloc_ds(self, tag, t):
        assert t % 8 not in self.ds, f"fragment {self.ds[t % 8]} overwritten by {tag} before its use"
        self.ds[t % 8] = tag
        return DSF(t)

    def use_ds(self, tag, t):
        assert self.ds.pop(t % 8) == tag
        return DSF(t)

    def state(self):
        return self.next, dict(self.owner), dict(self.uses_left), dict(self.reg), dict(self.ds)

    def restore(self, state):
        self.next, self.owner, self.uses_left, self.reg, self.ds = state[0], *(dict(x) for x in state[1:])


class OneEmitter(Emitter):
    def __init__(self):
        super().__init__()
        self.waits = []                                 # (label, where it goes back to, the count's scalar) of the polls

    def ds_read(self, text, tag):
        if len(self.ds) >= 15:                          # the counter has four bits
            self.need(self.ds[2])
        super().ds_read(text, tag)


def request_code(stage, st_set):
    c = [[f"global_load_dword {vr(ST + 2 * st_set)}, {vr(STAT_G)}, {sr(T_LSEPTR, 2)}",
          f"global_load_dword {vr(ST + 2 * st_set + 1)}, {vr(STAT_G)}, {sr(T_DLPTR, 2)}"]]
    for ptr, off, tbase in ((T_QPTR, QOFF, QT(stage)), (T_DOPTR, DOOFF, DOT(stage))):
        for j in range(NDQ):
            c.append([f"s_add_u32 m0, {sr(T_M0)}, {tbase + 4 * GRP * j}", "s_nop 0",
                      f"global_load_lds_dwordx4 {vr(off + j)}, {sr(ptr, 2)}"])
    return c


def flag_load(e):
    e.raw(f"v_mov_b32 {vr(TMP + 2)}, 0")
    e.raw(f"global_load_dword {vr(FLG)}, {vr(TMP + 2)}, {sr(S_PRED, 2)} sc1")


def flag_wait(e, newer, ahead=0):
    """Until the tile before has counted the pair (`ahead` pairs behind this tile's own count); `newer` memory operations were issued
    behind the load of its count (None: ask again).  What is not there yet is waited for out of line (gen_polls)."""
    l_polls, l_ok = e.label("polls"), e.label("counted")
    need = S_CNT
    if ahead:
        need = T_INC
        e.raw(f"s_add_u32 {sr(T_INC)}, {sr(S_CNT)}, {ahead}")
    if newer is not None:
        e.raw(f"s_waitcnt vmcnt({newer})")
        e.raw(f"v_readfirstlane_b32 {sr(T_MT)}, {vr(FLG)}")
        e.raw(f"s_cmp_ge_i32 {sr(T_MT)}, {sr(need)}")
        e.raw(f"s_cbranch_scc0 {l_polls}")
    else:
        e.raw(f"s_branch {l_polls}")
    e.raw(l_ok + ":")
    e.waits.append((l_polls, l_ok, need))


def gen_polls(e, label, l_back, need):
    """At most S_POLLS polls (seconds): a tile waits for running workgroups only and never needs so many, but a launch has to end
    whatever happens, and not with wrong sums unnoticed.  A wavefront that has used them up takes every pair from here on for counted, so
    that a launch waits that long once a wavefront and not once a pair, and marks the launch as one without gradients (add_pairs_kernel
    writes NaN).  Leaves no memory operation under way; the waits behind it count later ones only."""
    l_spin = e.label("spin")
    e.raw(label + ":")
    e.raw(f"s_mov_b32 {sr(T_X)}, {sr(S_POLLS)}")
    e.raw(l_spin + ":")
    flag_load(e)
    e.raw("s_waitcnt vmcnt(0)")
    e.raw(f"v_readfirstlane_b32 {sr(T_MT)}, {vr(FLG)}")
    e.raw(f"s_cmp_ge_i32 {sr(T_MT)}, {sr(need)}")
    e.raw(f"s_cbranch_scc1 {l_back}")
    e.raw("s_sleep 1")
    e.raw(f"s_sub_u32 {sr(T_X)}, {sr(T_X)}, 1")
    e.raw(f"s_cmp_lg_u32 {sr(T_X)}, 0")
    e.raw(f"s_cbranch_scc1 {l_spin}")
    e.raw(f"s_add_u32 {sr(T_X)}, {sr(S_LDS)}, {PBLK + 256 * 32}")
    e.raw(f"v_mov_b32 {vr(TMP)}, {sr(T_X)}")
    e.raw(f"ds_read_b64 {vr(TMP, 2)}, {vr(TMP)} offset:{4 * U_PLENTY}")
    e.raw("s_waitcnt lgkmcnt(0)")
    for i in range(2):
        e.raw(f"v_readfirstlane_b32 {sr(S_PRED + i)}, {vr(TMP + i)}")
    e.raw(f"v_mov_b32 {vr(TMP + 1)}, 1")
    e.raw(f"v_mov_b32 {vr(TMP + 2)}, 0")
    e.raw("s_nop 4")                                   # a scalar written by a vector instruction, as the address of a store
    e.raw("s_mov_b64 exec, 1")
    e.raw(f"global_store_dword {vr(TMP + 2)}, {vr(TMP + 1)}, {sr(S_PRED, 2)} offset:{GAVE_UP}")
    e.raw("s_mov_b64 exec, -1")
    e.raw("s_waitcnt vmcnt(0)")
    e.raw(f"s_branch {l_back}")


def flag_store(e):
    e.raw(f"v_mov_b32 {vr(TMP + 2)}, 0")
    e.raw(f"v_mov_b32 {vr(TMP + 1)}, {sr(S_CNT)}")
    e.raw("s_mov_b64 exec, 1")
    e.raw(f"global_store_dword {vr(TMP + 2)}, {vr(TMP + 1)}, {sr(S_OWN, 2)}")
    e.raw("s_mov_b64 exec, -1")


def old_load(e, j, x=0):
    to = vr(OLD + 4 * j, 4) if D == 128 else ar(ACC64(x) + 4 * j, 4)
    e.raw(f"global_load_dwordx4 {to}, {vr(DQO)}, {sr(S_DQL, 2)} offset:{1024 * j} sc1")


def sum_store(e, j, x=0):
    what = vr(OLD + 4 * j, 4) if D == 128 else ar(ACC64(x) + 4 * j, 4)
    e.raw(f"global_store_dwordx4 {vr(DQO)}, {what}, {sr(S_DQW, 2)} offset:{1024 * j}")


def next_old():
    return [f"s_add_u32 {sr(S_DQL)}, {sr(S_DQL)}, {sr(S_DQINC)}", f"s_addc_u32 {sr(S_DQL + 1)}, {sr(S_DQL + 1)}, 0"]


def next_sum():
    return [f"s_add_u32 {sr(S_DQW)}, {sr(S_DQW)}, {PAIR}", f"s_addc_u32 {sr(S_DQW + 1)}, {sr(S_DQW + 1)}, 0"]


def rd_dq(e, pool, tag, t, buf):
    """The two operands of MFMA t of a pair: 16 keys of K^T and of dS^T.  Head size 64: 32 keys, rows 16 (t % 2) .. + 15 of dS^T."""
    if D == 128:
        r = pool.alloc(tag + "k", 1)
        e.ds_read(f"ds_read_b64_tr_b16 {vr(r, 2)}, {vr(KTR)} offset:{rows(16) * t}", tag + "klo")
        e.ds_read(f"ds_read_b64_tr_b16 {vr(r + 2, 2)}, {vr(KTR)} offset:{rows(16) * t + rows(8)}", tag + "k")
    r = pool.alloc(tag + "s", 1) if D == 128 else pool.alloc_ds(tag, t)
    reg = vr if D == 128 else ar
    at, half = (16 * DSR_ROW * t, 8 * DSR_ROW) if D == 128 else (32 * DSR_ROW * (t // 2) + 32 * (t % 2), 16 * DSR_ROW)
    e.ds_read(f"ds_read_b64_tr_b16 {reg(r, 2)}, {vr(DSR)} offset:{DS_BYTES * buf + at}", tag + "slo")
    e.ds_read(f"ds_read_b64_tr_b16 {reg(r + 2, 2)}, {vr(DSR)} offset:{DS_BYTES * buf + at + half}", tag + "s")


def mfma_dq(e, pool, tag, t, buf):
    """(the pairs' sums alternate between two sets of registers as their dS do between buffers)"""
    if D == 64:
        e.need(tag + "s")
        acc = ar(ACC64(buf) + 4 * (t % 2), 4)
        e.mfma(acc, ar(KTF(t // 2), 4), ar(pool.use_ds(tag, t), 4), acc, shape="16x16x32")
        return
    e.need(tag + "k")
    e.need(tag + "s")
    a, b = pool.use(tag + "k"), pool.use(tag + "s")
    e.mfma(vr(ACC_Q, 16), vr(a, 4), vr(b, 4), "0" if t == 0 else vr(ACC_Q, 16))


def plan_dq(e, pool, buf, seq):
    """Reads and MFMAs of a pair by slot: in the block behind its own, and in the one after that (negative slots: the tail of the first)."""
    parts = [({k: [] for k in range(NSLOT)}, {k: [] for k in range(NSLOT)}), ({k: [] for k in range(-EARLY, NSLOT)}, {k: [] for k in range(NSLOT)})]
    for t, p in enumerate(DQ_AT):
        tag = f"{seq}dq{t}_"
        def rd(tag=tag, t=t): rd_dq(e, pool, tag, t, buf)
        def mm(tag=tag, t=t): mfma_dq(e, pool, tag, t, buf)
        second = p >= NSLOT
        parts[second][0][p - LATQ - NSLOT * second].append(rd)
        parts[second][1][p - NSLOT * second].append(mm)
    return parts


def plan_reads(e, pool, stage, seq):
    qt, dot_, stats = QT(stage), DOT(stage), 256 * stage
    reads = {k: [] for k in range(-EARLY, NSLOT)}

    def plan(first_use, fn):
        reads[first_use - LAT].append(fn)

    def rd_nat(tag, imm, ks, xbase, uses):
        def f():
            r = pool.alloc(tag, uses)
            x, off = (xbase + ks // 2, 32 * (ks % 2)) if D == 128 else (xbase + ks, 0)
            e.ds_read(f"ds_read_b128 {vr(r, 4)}, {vr(x)} offset:{imm + off}", tag)
        return f

    def rd_tr(tag, imm, m, db):
        def f():
            r = pool.alloc(tag, NKB)
            e.ds_read(f"ds_read_b64_tr_b16 {vr(r, 2)}, {vr(TR + db)} offset:{imm + rows(16) * m}", tag + "lo")
            e.ds_read(f"ds_read_b64_tr_b16 {vr(r + 2, 2)}, {vr(TR + db)} offset:{imm + rows(16) * m + rows(8)}", tag)
        return f

    def rd_stat(tag, base_reg, imm, js):
        def f():
            for j in js:
                e.ds_read(f"ds_read_b128 {vr(base_reg + 4 * j, 4)}, {vr(G16)} offset:{imm + 32 * j}", f"{tag}{j}")
        return f

    for ks in range(KS):
        plan(2 * ks, rd_nat(f"{seq}q{ks}", qt, ks, X, NKB))
        for nb in range(NKB if D == 128 else 0):
            plan(2 * ks + nb, rd_nat(f"{seq}K{nb}_{ks}", rows(32) * nb, ks, XK, 1))
        if ks == 0:
            reads[-EARLY].append(rd_stat(f"{seq}nl", NL, stats, (0, 1)))
            reads[-EARLY + 1].append(rd_stat(f"{seq}nl", NL, stats, (2, 3)))
            reads[-EARLY + 4].append(rd_stat(f"{seq}nd", ND, stats + 128, (0, 1)))
            reads[-EARLY + 5].append(rd_stat(f"{seq}nd", ND, stats + 128, (2, 3)))
    for ks in range(KS):
        plan(P2 + 2 * ks, rd_nat(f"{seq}do{ks}", dot_, ks, X, NKB))
    for ph, tile in (("dV", dot_), ("dK", qt)):
        for m in range(2):
            for db in range(DB):
                plan((P3 if ph == "dV" else P4) + 2 * (DB * m + db), rd_tr(f"{seq}{ph}t{m}_{db}", tile, m, db))
    return reads


def gen_step(e, pool, u, seq, reads, next_reads, dq_behind, dq_next, dq_start, masked):
    """Block u of the copies.  dq_behind: the pair two blocks back, finished here; dq_start: the pair of the block before, begun here;
    dq_next: the same pair's second part, whose first reads are at the tail of this block."""
    stage, buf = u % NS, u % 2
    e.comment(f"================ block {u}")
    slots = [("S", ks, nb) for ks in range(KS) for nb in range(NKB)] + [("dP", ks, nb) for ks in range(KS) for nb in range(NKB)]
    slots += [(ph, m, db, nb) for ph in ("dV", "dK") for m in range(2) for db in range(DB) for nb in range(NKB)]

    def S(nb, v): return S0 + 16 * nb + v
    def DP(nb, v): return DP0 + 16 * nb + v
    valu = []                                          # (earliest slot, text, registers written, issue units, LDS write behind it)
    for m in range(2):
        for nb in range(NKB):
            early = P2 + 1 + nb
            for grp in range(2):
                for v in [8 * m + 4 * grp + i for i in range(4)]:
                    valu.append((early, f"v_exp_f32 {vr(S(nb, v))}, {vr(S(nb, v))}", (), 2, None))
                if grp == 1:
                    for i in range(4):
                        d, a = P16 + 8 * nb + 4 * m + i, S(nb, 8 * m + 2 * i)
                        valu.append((max(early, P2 + 4), f"v_cvt_pk_bf16_f32 {vr(d)}, {vr(a)}, {vr(a + 1)}", (d,), 1, None))
    for m in range(2):
        for nb in range(NKB):
            early = P3 + 1 + nb
            for v in range(8 * m, 8 * m + 8):
                valu.append((early, f"v_mul_f32 {vr(DP(nb, v))}, {vr(S(nb, v))}, {vr(DP(nb, v))}", (), 1, None))
            for i in range(4):
                d, a = DP(nb, 4 * m + i), DP(nb, 8 * m + 2 * i)
                valu.append((early, f"v_cvt_pk_bf16_f32 {vr(d)}, {vr(a)}, {vr(a + 1)}", (d,), 1, None))
                if i % 2:                              # rows 16 m + 8 (i / 2) + 4 g .. + 3 of the lane's key
                    off = DS_BYTES * buf + 32 * DSR_ROW * nb + 16 * (2 * m + i // 2)
                    valu.append((early, f"ds_write_b64 {vr(DSW)}, {vr(d - 1, 2)} offset:{off}", (), 2, f"{seq}ds{m}{nb}{i}"))
    vi, produced = [0], {}

    def emit_valu(item):
        _, text, writes, units, tag = item
        if tag:
            e.ds_read(text, tag)
        else:
            e.valu(text, writes)
        for r in writes:
            produced[r] = True
        return units

    def flush_until(regs):
        while not all(produced.get(r) for r in regs):
            assert vi[0] < len(valu), "packed operand never produced"
            emit_valu(valu[vi[0]])
            vi[0] += 1

    side = {k: [] for k in range(NSLOT)}               # scalar and memory work behind fixed slots: text, or a function
    req = request_code((u + PF) % NS, (u + PF) % 2)

    def counted(newer):
        e.raw(f"s_waitcnt vmcnt({newer})")             # operations behind the stores
        flag_store(e)
        e.raw(f"s_add_u32 {sr(S_CNT)}, {sr(S_CNT)}, 1")
    if D == 128:
        # pair s - 2 of block s: what the tile before left is read, added to and stored in this block
        side[2].append(lambda: flag_wait(e, NREQ + 1))             # behind the count's load: the request, a count's store
        for j in range(4):
            side[3 + j].append(lambda j=j: old_load(e, j))
            side[SUM_SLOT + 1 + j].append(lambda j=j: sum_store(e, j))
        side[SUM_SLOT + 5] += next_old() + next_sum()
        side[SUM_SLOT + 5].append(lambda: flag_load(e))
        for i, grp in enumerate(req):
            side[SUM_SLOT + 6 + i] += grp
        assert SUM_SLOT + 5 > SYNC_SLOT and SUM_SLOT < DQ_AT[0] and SUM_SLOT + 6 + len(req) <= P4
        side[NSLOT - 2].append(lambda: counted(NREQ + 1))          # behind the stores: the count's load, the request
    else:
        # pair s - 3 is counted, pair s - 2 stored, pair s read into the registers that leaves.  (Read behind the barrier instead,
        # ahead of the request, and the tile waits for less: 3 % slower, the next tile runs further behind)
        side[0].append(lambda: counted(NREQ + NP))                 # behind the stores: the request, what the tile before left
        side[2].append(lambda: flag_load(e))
        for j in range(NP):
            side[SYNC_SLOT - 3 + j].append(lambda j=j: sum_store(e, j, u))
        side[SYNC_SLOT + 1] += next_sum()
        side[SYNC_SLOT + 1].append(f"s_waitcnt vmcnt({2 + NP})")         # pair s - 1 is there; behind it: a count's store, a count, the stores
        for i, grp in enumerate(req):
            side[SYNC_SLOT + 2 + i] += grp
        side[NSLOT - 2].append(lambda: flag_wait(e, NREQ + NP, 2))
        for j in range(NP):
            side[NSLOT - 2].append(lambda j=j: old_load(e, j, u))
        side[NSLOT - 1] += next_old()
    adv = kv.advance_code()
    per = 4 if D == 128 else 8
    for i in range(0, len(adv), per):
        side[P4 + i // per] += adv[i:i + per]
    assert P4 + (len(adv) - 1) // per < NSLOT - 3      # a wait that looks ahead uses the same scalar
    stw = f"{seq}stw"

    def fill(units, budget, k):
        while vi[0] < len(valu) and valu[vi[0]][0] <= k and units + valu[vi[0]][3] <= budget:
            units += emit_valu(valu[vi[0]])
            vi[0] += 1

    for k, sl in enumerate(slots):
        ph = sl[0]
        if ph == "S":
            _, ks, nb = sl
            tag = f"{seq}q{ks}"
            e.need(tag)
            if D == 128:
                e.need(f"{seq}K{nb}_{ks}")
            if ks == 0:
                e.need(f"{seq}nl3")
            c = vr(NL, 16) if ks == 0 else vr(S0 + 16 * nb, 16)
            a_reg = pool.use(tag)
            e.mfma(vr(S0 + 16 * nb, 16), vr(a_reg, 4), vr(pool.use(f"{seq}K{nb}_{ks}") if D == 128 else KR(nb, ks), 4), c)
        elif ph == "dP":
            _, ks, nb = sl
            e.need(f"{seq}do{ks}")
            if ks == 0:
                e.need(f"{seq}nd3")
            c = vr(ND, 16) if ks == 0 else vr(DP0 + 16 * nb, 16)
            e.mfma(vr(DP0 + 16 * nb, 16), vr(pool.use(f"{seq}do{ks}"), 4), vr(VF(nb, ks), 4), c)
        else:
            _, m, db, nb = sl
            tag = f"{seq}{ph}t{m}_{db}"
            e.need(tag)
            b0, acc = (P16 + 8 * nb + 4 * m, ACC_V(db, nb)) if ph == "dV" else (DP0 + 16 * nb + 4 * m, ACC_K(db, nb))
            flush_until([b0 + i for i in range(4)])
            e.mfma(ar(acc, 16), vr(pool.use(tag), 4), vr(b0, 4), ar(acc, 16), breads=[b0 + i for i in range(4)])
        # ---- side work of this slot
        n0 = len(e.lines)
        for fn in reads[k] + next_reads.get(k - NSLOT, []) + dq_start[0].get(k, []) + dq_behind[0].get(k, []) + dq_next[0].get(k - NSLOT, []):
            fn()
        for x in side[k]:
            if callable(x):
                x()
            else:
                e.raw(x)
        units = len(e.lines) - n0
        if masked and k == P2 + 1:
            e.raw(f"s_swappc_b64 {sr(T_MRET, 2)}, {sr(T_MASK, 2)}")
        if k == PUBLISH_SLOT:
            # behind the request of the next block: a count's store, what the tile before left; head size 64: all of a block's and a
            # count's store
            e.raw(f"s_waitcnt vmcnt({5 if D == 128 else NREQ + 2})")
            kv.stat_publish_to(e, STAT_L, (u + 1) % 2, (u + 1) % NS, stw)
            units += 8
        if D == 128 and k == SUM_SLOT:
            e.raw("s_waitcnt vmcnt(0)")
            for v in range(16):
                e.raw(f"v_add_f32 {vr(OLD + v)}, {vr(OLD + v)}, {vr(ACC_Q + v)}")
            units += 16
        fill(units, BUDGET, k)
        for fn in dq_start[1].get(k, []) + dq_behind[1].get(k, []):
            fn()
            fill(0, BUDGET_Q, k)
        if k == SYNC_SLOT:
            e.need(stw)                                # and with it everything older: dS of the block before
            e.raw("s_barrier")
    assert vi[0] == len(valu), f"VALU work left over: {len(valu) - vi[0]}"


def pblk_address(e, reg, tmp):
    """reg = LDS address of this thread's parameters"""
    e.raw(f"v_mbcnt_lo_u32_b32 {vr(reg)}, -1, 0")
    e.raw(f"v_mbcnt_hi_u32_b32 {vr(reg)}, -1, {vr(reg)}")
    e.raw(f"v_lshlrev_b32 {vr(reg)}, 5, {vr(reg)}")
    e.raw(f"s_lshl_b32 {sr(tmp)}, {sr(S_WAVE)}, 11")
    e.raw(f"s_add_u32 {sr(tmp)}, {sr(tmp)}, {sr(S_LDS)}")
    e.raw(f"s_add_u32 {sr(tmp)}, {sr(tmp)}, {PBLK}")
    e.raw(f"v_add_u32 {vr(reg)}, {sr(tmp)}, {vr(reg)}")


def gen_whole_offsets(e, reg, tmp):
    pblk_address(e, reg, tmp)
    for i, dst in enumerate((QOFF, QOFF + 1, DOOFF, DOOFF + 1, STAT_G)):
        e.raw(f"ds_read_b32 {vr(dst)}, {vr(reg)} offset:{8 + 4 * i}")
    e.raw("s_waitcnt lgkmcnt(0)")


def gen_mask_routine(e):
    """As in gen_bwd_dkv_asm.py, with the parameters of a thread read from LDS."""
    n4, low, high = TMP, TMP + 1, MASK_HIGH
    l_one, l_still = e.label("onehead"), e.label("still")
    for _ in range(3):
        e.raw("s_nop 7")
    e.raw(f"s_sub_u32 {sr(T_MT)}, {sr(S_NSTEPS)}, {sr(T_REM)}")
    e.raw(f"s_cmp_eq_u32 {sr(S_NIN)}, 1")
    e.raw(f"s_cbranch_scc1 {l_one}")
    e.raw(f"s_mul_hi_u32 {sr(T_MT)}, {sr(T_MT)}, {sr(S_GREC)}")
    e.raw(l_one + ":")
    e.raw(f"s_lshl_b32 {sr(T_MT)}, {sr(T_MT)}, 5")
    e.raw(f"s_sub_u32 {sr(S_CI)}, {sr(S_CI0)}, {sr(T_MT)}")
    e.raw(f"s_sub_u32 {sr(T_MT)}, {sr(S_NSTEPS)}, {sr(S_NRAG)}")
    e.raw(f"s_add_u32 {sr(T_MT)}, {sr(T_MT)}, 1")
    e.raw(f"s_cmp_gt_u32 {sr(T_REM)}, {sr(T_MT)}")
    e.raw(f"s_cselect_b32 {sr(S_EVT)}, -1, {sr(S_DIAG)}")
    e.raw(f"s_cmp_lt_u32 {sr(T_DSTEP)}, {sr(S_NRAG)}")
    e.raw(f"s_cbranch_scc1 {l_still}")
    gen_whole_offsets(e, n4, T_MT)
    e.raw(l_still + ":")
    pblk_address(e, n4, T_MT)
    for nb in range(NKB):
        e.raw(f"ds_read_b32 {vr(low + nb)}, {vr(n4)} offset:{4 * nb}")
    e.raw("s_waitcnt lgkmcnt(0)")
    e.raw(f"v_mbcnt_lo_u32_b32 {vr(n4)}, -1, 0")
    e.raw(f"v_mbcnt_hi_u32_b32 {vr(n4)}, -1, {vr(n4)}")
    e.raw(f"v_lshrrev_b32 {vr(n4)}, 5, {vr(n4)}")
    e.raw(f"v_lshlrev_b32 {vr(n4)}, 2, {vr(n4)}")
    for nb in range(NKB):
        e.raw(f"v_subrev_u32 {vr(low + nb)}, {sr(S_CI)}, {vr(low + nb)}")
        e.raw(f"v_sub_u32 {vr(low + nb)}, {vr(low + nb)}, {vr(n4)}")

    def each(cmp, bound):
        for nb in range(NKB):
            for v0 in range(0, 16, 3):
                vs = range(v0, min(v0 + 3, 16))
                for v in vs:
                    e.raw(f"{cmp} {sr(T_CMP[v - v0], 2)}, {vr(bound(nb))}, {8 * (v // 4) + v % 4}")
                if len(vs) < 3:
                    e.raw("s_nop 1")
                for v in vs:
                    x = vr(S0 + 16 * nb + v)
                    e.raw(f"v_cndmask_b32_e64 {x}, {vr(NINF)}, {x}, {sr(T_CMP[v - v0], 2)}")
    each("v_cmp_le_i32_e64", lambda nb: low + nb)
    l_ret = e.label("mret")
    e.raw(f"s_add_u32 {sr(T_MT)}, {sr(S_CI)}, 32")
    e.raw(f"s_cmp_le_u32 {sr(T_MT)}, {sr(S_SQ)}")
    e.raw(f"s_cbranch_scc1 {l_ret}")
    e.raw(f"s_sub_u32 {sr(T_MT)}, {sr(S_SQ)}, {sr(S_CI)}")
    e.raw(f"v_sub_u32 {vr(high)}, {sr(T_MT)}, {vr(n4)}")
    each("v_cmp_gt_i32_e64", lambda nb: high)
    e.raw(l_ret + ":")
    e.raw("s_nop 1")
    e.raw(f"s_setpc_b64 {sr(T_MRET, 2)}")


def gen_tail(e, buf):
    """Behind the last block: the rest of the pair before the last one (dS in buffer `buf`), then the last one."""
    pool = Pool()

    def mfmas(ts, b, name):
        ahead = 3
        for i in range(min(ahead, len(ts))):
            rd_dq(e, pool, f"{name}{ts[i]}_", ts[i], b)
        for i, t in enumerate(ts):
            if i + ahead < len(ts):
                rd_dq(e, pool, f"{name}{ts[i + ahead]}_", ts[i + ahead], b)
            mfma_dq(e, pool, f"{name}{t}_", t, b)

    def finish():
        for _ in range(4):
            e.raw("s_nop 7")
        e.raw("s_waitcnt vmcnt(0)")
        for v in range(16):
            e.raw(f"v_add_f32 {vr(OLD + v)}, {vr(OLD + v)}, {vr(ACC_Q + v)}")
        for j in range(4):
            sum_store(e, j)
        for ln in next_old() + next_sum():
            e.raw(ln)

    if D == 64:                                        # both pairs have been read
        e.raw("s_waitcnt vmcnt(0) lgkmcnt(0)")
        e.ds = []
        e.raw("s_barrier")
        mfmas(list(range(N_A, N_DQ)), buf, "a")
        mfmas(list(range(N_DQ)), 1 - buf, "b")
        for _ in range(4):
            e.raw("s_nop 7")
        for x in (buf, 1 - buf):
            for j in range(NP):
                sum_store(e, j, x)
            for ln in next_sum():
                e.raw(ln)
        e.raw(f"s_add_u32 {sr(S_CNT)}, {sr(S_CNT)}, 2")
        e.raw("s_waitcnt vmcnt(0)")
        flag_store(e)
        e.raw("s_waitcnt vmcnt(0) lgkmcnt(0)")
        return
    e.raw("s_waitcnt vmcnt(0) lgkmcnt(0)")             # every wavefront has written its dS of the last block
    e.ds = []
    flag_wait(e, 0)
    for j in range(4):
        old_load(e, j)
    e.raw("s_barrier")
    mfmas(list(range(N_A, 16)), buf, "a")
    finish()
    e.raw(f"s_add_u32 {sr(S_CNT)}, {sr(S_CNT)}, 1")
    mfmas(list(range(16)), 1 - buf, "b")
    flag_wait(e, None)
    for j in range(4):
        old_load(e, j)
    finish()
    e.raw("s_waitcnt vmcnt(0)")
    flag_store(e)
    e.raw("s_waitcnt vmcnt(0) lgkmcnt(0)")


def generate():
    e = OneEmitter()
    pool = Pool()
    l_mask = e.label("mask")
    e.comment("---- prologue: stream state")
    for t, s_ in ((T_QPTR, kv.S_QPTR), (T_QHEAD, kv.S_QPTR), (T_DOPTR, kv.S_DOPTR), (T_DOHEAD, kv.S_DOPTR),
                  (T_LSEPTR, kv.S_LSEPTR), (T_LSEHEAD, kv.S_LSEPTR), (T_DLPTR, kv.S_DLPTR), (T_DLHEAD, kv.S_DLPTR),
                  (T_VPTR, kv.S_VPTR)):
        e.raw(f"s_mov_b64 {sr(t, 2)}, {sr(s_, 2)}")
    for t in (T_DBLK, T_DSTEP):
        e.raw(f"s_mov_b32 {sr(t)}, 0")
    e.raw(f"s_mov_b32 {sr(T_REM)}, {sr(S_NSTEPS)}")
    e.raw(f"s_mov_b32 {sr(S_CNT)}, {-1 if D == 128 else -2}")
    e.raw(f"s_ashr_i32 {sr(T_OHI)}, {sr(S_QOUT)}, 31")
    e.raw(f"s_mul_i32 {sr(T_M0)}, {sr(S_WAVE)}, {GRP}")
    e.raw(f"s_add_u32 {sr(T_M0)}, {sr(T_M0)}, {sr(S_LDS)}")
    e.raw(f"s_mov_b32 {sr(T_HIMASK)}, 0")
    e.raw(f"s_mov_b32 {sr(T_HIMASK + 1)}, -1")
    e.comment("---- resident V fragments (B operands): key row = lane % 32, elements 16 ks + 8 (lane / 32) .. + 7")
    for nb, row in ((0, kv.I_KROW0), (1, kv.I_KROW1)):
        for ks in range(KS):
            e.raw(f"global_load_dwordx4 {vr(VF(nb, ks), 4)}, {vr(row, 2)}, off offset:{32 * ks}")
    e.comment("---- parameters")
    e.raw(f"s_add_u32 {sr(T_X)}, {sr(S_LDS)}, {PBLK + 256 * 32}")
    e.raw(f"v_mov_b32 {vr(TMP)}, {sr(T_X)}")
    e.raw(f"ds_read_b128 {vr(ST, 4)}, {vr(TMP)}")
    e.raw(f"ds_read_b64 {vr(TMP, 2)}, {vr(TMP)} offset:16")
    e.raw("s_waitcnt lgkmcnt(0)")
    for src, dst in ((ST, S_NRAG), (ST + 1, S_DIAG), (ST + 2, S_GREC), (ST + 3, S_CI0), (TMP, S_SQ), (TMP + 1, S_ROWS)):
        e.raw(f"v_readfirstlane_b32 {sr(dst)}, {vr(src)}")
    e.raw(f"s_cmp_lg_u32 {sr(S_NRAG)}, -1")
    e.raw(f"s_cselect_b32 {sr(S_EVT)}, -1, {sr(S_DIAG)}")
    # (keys that no row sees are copies of the last one that some row does, here and in V: P is 0 there, but 0 times what lies in memory
    # that nobody has to have written need not be)
    e.comment("---- K tile of the workgroup (256 rows) to LDS: instruction 4 j + wave fills group 4 j + wave")
    per_load = 4 * 1024 // (2 * D)                     # rows
    e.raw(f"s_sub_u32 {sr(T_X)}, {sr(S_ROWS)}, 1")
    for j in range(256 // per_load):
        e.raw(f"v_min_u32 {vr(TMP)}, {sr(T_X)}, {vr(kv.I_SROW)}")
        e.raw(f"v_mul_lo_u32 {vr(TMP)}, {vr(TMP)}, {sr(S_VRS)}")
        e.raw(f"v_add_u32 {vr(TMP)}, {vr(TMP)}, {vr(kv.I_VCOL)}")
        e.raw(f"s_add_u32 m0, {sr(T_M0)}, {KT + 4 * GRP * j}")
        e.raw("s_nop 0")
        e.raw(f"global_load_lds_dwordx4 {vr(TMP)}, {sr(T_VPTR, 2)}")
        e.raw(f"v_add_u32 {vr(kv.I_SROW)}, {per_load}, {vr(kv.I_SROW)}")
    if D == 64:
        e.comment("---- resident K fragments likewise, from the tile's first row on")
        e.raw(f"v_mbcnt_lo_u32_b32 {vr(TMP)}, -1, 0")
        e.raw(f"v_mbcnt_hi_u32_b32 {vr(TMP)}, -1, {vr(TMP)}")
        e.raw(f"v_and_b32 {vr(TMP + 1)}, 31, {vr(TMP)}")
        e.raw(f"v_lshrrev_b32 {vr(TMP)}, 5, {vr(TMP)}")
        e.raw(f"v_lshlrev_b32 {vr(TMP)}, 4, {vr(TMP)}")
        e.raw(f"s_lshl_b32 {sr(T_X)}, {sr(S_WAVE)}, 6")
        e.raw(f"v_add_u32 {vr(TMP + 1)}, {sr(T_X)}, {vr(TMP + 1)}")
        e.raw(f"s_sub_u32 {sr(T_X)}, {sr(S_ROWS)}, 1")
        for nb in range(NKB):
            e.raw(f"v_min_u32 {vr(TMP + 2)}, {sr(T_X)}, {vr(TMP + 1)}")
            e.raw(f"v_mul_lo_u32 {vr(TMP + 2)}, {vr(TMP + 2)}, {sr(S_VRS)}")
            e.raw(f"v_add_u32 {vr(TMP + 2)}, {vr(TMP + 2)}, {vr(TMP)}")
            for ks in range(KS):
                e.raw(f"global_load_dwordx4 {vr(KR(nb, ks), 4)}, {vr(TMP + 2)}, {sr(T_VPTR, 2)} offset:{32 * ks}")
            e.raw(f"v_add_u32 {vr(TMP + 1)}, 32, {vr(TMP + 1)}")
    l_here = e.label("here")
    e.raw(f"s_getpc_b64 {sr(T_MASK, 2)}")
    e.raw(l_here + ":")
    e.raw(f"s_add_u32 {sr(T_MASK)}, {sr(T_MASK)}, {l_mask}-{l_here}")
    e.raw(f"s_addc_u32 {sr(T_MASK + 1)}, {sr(T_MASK + 1)}, 0")
    e.comment("---- per-lane address registers")
    for dst, src in ((QOFF, kv.I_QOFF0), (QOFF + 1, kv.I_QOFF1), (DOOFF, kv.I_DOOFF0), (DOOFF + 1, kv.I_DOOFF1), (STAT_G, kv.I_STAT_G),
                     (STAT_L, kv.I_STAT_L)):
        e.raw(f"v_mov_b32 {vr(dst)}, {vr(src)}")
    e.raw(f"v_mov_b32 {vr(NINF)}, 0xff800000")
    L4, LANE, R, G = FLG, TMP, TMP + 1, TMP + 2
    e.raw(f"v_subrev_u32 {vr(L4)}, {sr(S_LDS)}, {vr(STAT_L)}")           # 4 * lane
    e.raw(f"v_lshrrev_b32 {vr(LANE)}, 2, {vr(L4)}")
    e.raw(f"v_lshrrev_b32 {vr(G)}, 5, {vr(LANE)}")                       # half of the wavefront
    e.raw(f"v_and_b32 {vr(R)}, 31, {vr(LANE)}")
    e.raw(f"v_lshlrev_b32 {vr(G16)}, 4, {vr(G)}")
    e.raw(f"v_add_u32 {vr(G16)}, {sr(S_LDS)}, {vr(G16)}")
    # dS, written: key 64 wave + lane % 32, 8 bytes per half
    e.raw(f"s_lshl_b32 {sr(T_X)}, {sr(S_WAVE)}, 6")
    e.raw(f"v_add_u32 {vr(DSW)}, {sr(T_X)}, {vr(R)}")
    e.raw(f"v_mul_u32_u24 {vr(DSW)}, {DSR_ROW}, {vr(DSW)}")
    e.raw(f"v_lshlrev_b32 {vr(DQO)}, 3, {vr(G)}")
    e.raw(f"v_add_u32 {vr(DSW)}, {vr(DSW)}, {vr(DQO)}")
    e.raw(f"s_add_u32 {sr(T_X)}, {sr(S_LDS)}, {DS0}")
    e.raw(f"v_add_u32 {vr(DSW)}, {sr(T_X)}, {vr(DSW)}")
    # dS, read transposed: key 4 g + (lane % 16) / 4, rows 16 ((lane / 16) % 2) + 4 (lane % 4) .. + 3; head size 64: key lane / 4, rows
    # 4 (lane % 4) .. + 3
    if D == 128:
        e.raw(f"v_and_b32 {vr(DSR)}, 15, {vr(LANE)}")
        e.raw(f"v_lshrrev_b32 {vr(DSR)}, 2, {vr(DSR)}")
        e.raw(f"v_lshlrev_b32 {vr(DQO)}, 2, {vr(G)}")
        e.raw(f"v_add_u32 {vr(DSR)}, {vr(DSR)}, {vr(DQO)}")
        e.raw(f"v_mul_u32_u24 {vr(DSR)}, {DSR_ROW}, {vr(DSR)}")
        e.raw(f"v_bfe_u32 {vr(DQO)}, {vr(LANE)}, 4, 1")
        e.raw(f"v_lshlrev_b32 {vr(DQO)}, 5, {vr(DQO)}")
        e.raw(f"v_add_u32 {vr(DSR)}, {vr(DSR)}, {vr(DQO)}")
    else:
        e.raw(f"v_lshrrev_b32 {vr(DSR)}, 2, {vr(LANE)}")
        e.raw(f"v_mul_u32_u24 {vr(DSR)}, {DSR_ROW}, {vr(DSR)}")
    e.raw(f"v_and_b32 {vr(DQO)}, 3, {vr(LANE)}")
    e.raw(f"v_lshlrev_b32 {vr(DQO)}, 3, {vr(DQO)}")
    e.raw(f"v_add_u32 {vr(DSR)}, {vr(DSR)}, {vr(DQO)}")
    e.raw(f"v_add_u32 {vr(DSR)}, {sr(T_X)}, {vr(DSR)}")
    if D == 64:
        # K^T, read transposed: key lane / 4 (groups of eight rows; chunk c of row r lies at c ^ (4 (r / 2 % 2) + 2 (r / 4 % 2))),
        # columns 16 wave + 4 (lane % 4) .. + 3
        e.raw(f"v_bfe_u32 {vr(KTR)}, {vr(LANE)}, 1, 1")                  # chunk 2 wave + (lane % 4) / 2, in 16 bytes
        e.raw(f"s_lshl_b32 {sr(T_X)}, {sr(S_WAVE)}, 1")
        e.raw(f"v_add_u32 {vr(KTR)}, {sr(T_X)}, {vr(KTR)}")
        e.raw(f"v_bfe_u32 {vr(DQO)}, {vr(LANE)}, 3, 1")                  # bit 1 of the row
        e.raw(f"v_lshlrev_b32 {vr(DQO)}, 2, {vr(DQO)}")
        e.raw(f"v_xor_b32 {vr(KTR)}, {vr(DQO)}, {vr(KTR)}")
        e.raw(f"v_bfe_u32 {vr(DQO)}, {vr(LANE)}, 4, 1")                  # bit 2
        e.raw(f"v_lshlrev_b32 {vr(DQO)}, 1, {vr(DQO)}")
        e.raw(f"v_xor_b32 {vr(KTR)}, {vr(DQO)}, {vr(KTR)}")
        e.raw(f"v_lshlrev_b32 {vr(KTR)}, 4, {vr(KTR)}")
        e.raw(f"v_and_b32 {vr(DQO)}, 1, {vr(LANE)}")
        e.raw(f"v_lshlrev_b32 {vr(DQO)}, 3, {vr(DQO)}")
        e.raw(f"v_add_u32 {vr(KTR)}, {vr(KTR)}, {vr(DQO)}")
        e.raw(f"v_bfe_u32 {vr(DQO)}, {vr(LANE)}, 2, 3")                  # row of its group
        e.raw(f"v_lshlrev_b32 {vr(DQO)}, 7, {vr(DQO)}")
        e.raw(f"v_add_u32 {vr(KTR)}, {vr(KTR)}, {vr(DQO)}")
        e.raw(f"v_mul_u32_u24 {vr(DQO)}, {GRP}, {vr(G)}")                # group lane / 32
        e.raw(f"v_add_u32 {vr(KTR)}, {vr(KTR)}, {vr(DQO)}")
        e.raw(f"s_add_u32 {sr(T_X)}, {sr(S_LDS)}, {KT}")
        e.raw(f"v_add_u32 {vr(KTR)}, {sr(T_X)}, {vr(KTR)}")
    # workspace: 16 lane + SLICE wave
    e.raw(f"s_mul_i32 {sr(T_X)}, {sr(S_WAVE)}, {SLICE}")
    e.raw(f"v_lshlrev_b32 {vr(DQO)}, 2, {vr(L4)}")
    e.raw(f"v_add_u32 {vr(DQO)}, {sr(T_X)}, {vr(DQO)}")
    # natural reads: x[a] = xbase + (gf16 ^ 64 a), steps 2 a and 2 a + 1; K: the wavefront's 64 rows.  Head size 64: x[ks] = xbase + (gf16 ^ 32 ks)
    if D == 128:
        e.raw(f"s_mul_i32 {sr(T_X)}, {sr(S_WAVE)}, {rows(64)}")
        e.raw(f"s_add_u32 {sr(T_X)}, {sr(T_X)}, {KT}")
    for a in range(4):
        e.raw(f"v_xor_b32 {vr(TMP)}, {(64 if D == 128 else 32) * a}, {vr(kv.I_GF16)}")
        e.raw(f"v_add_u32 {vr(X + a)}, {vr(kv.I_XBASE)}, {vr(TMP)}")
        if D == 128:
            e.raw(f"v_add_u32 {vr(XK + a)}, {sr(T_X)}, {vr(X + a)}")
    # transpose reads: tr[db] = trbase + (lf16 ^ 64 db); K^T: the wavefront's 32 columns
    for db in range(DB):
        e.raw(f"v_xor_b32 {vr(TMP)}, {64 * db}, {vr(kv.I_LF16)}")
        e.raw(f"v_add_u32 {vr(TR + db)}, {vr(kv.I_TRBASE)}, {vr(TMP)}")
    if D == 128:
        e.raw(f"s_lshl_b32 {sr(T_X)}, {sr(S_WAVE)}, 6")
        e.raw(f"v_xor_b32 {vr(TMP)}, {sr(T_X)}, {vr(kv.I_LF16)}")
        e.raw(f"v_add_u32 {vr(KTR)}, {vr(kv.I_TRBASE)}, {vr(TMP)}")
        e.raw(f"v_add_u32 {vr(KTR)}, {KT}, {vr(KTR)}")
    e.comment("---- the first blocks requested; accumulators to zero meanwhile")

    def request(blk):
        if blk:
            l_still = e.label("still")
            e.raw(f"s_cmp_lt_u32 {sr(T_DSTEP)}, {sr(S_NRAG)}")
            e.raw(f"s_cbranch_scc1 {l_still}")
            gen_whole_offsets(e, TMP, T_MT)
            e.raw(l_still + ":")
        for grp in request_code(blk % NS, blk % 2):
            for ln in grp:
                e.raw(ln)
        for ln in kv.advance_code():
            e.raw(ln)

    request(0)
    if D == 128:
        flag_load(e)
    request(1)
    if D == 128:
        flag_store(e)                                  # (as every block does: the waits count it)
    for i in range(256):
        e.raw(f"v_accvgpr_write_b32 {ar(i)}, 0")
    e.comment("statistics of block 0 to LDS stage 0")
    e.raw(f"s_waitcnt vmcnt({NREQ + (2 if D == 128 else 0)})")
    kv.stat_publish_to(e, STAT_L, 0, 0, "stw")
    e.raw("s_waitcnt lgkmcnt(0)")
    e.ds = []
    if D == 64:
        request(2)
        e.comment("K^T fragments")
        e.raw("s_barrier")
        for t in range(N_DQ // 2):
            for half in range(2):
                e.raw(f"ds_read_b64_tr_b16 {vr(POOL0 + 4 * t + 2 * half, 2)}, {vr(KTR)} offset:{rows(32) * t + rows(16) * half}")
        e.raw("s_waitcnt lgkmcnt(0)")
        for i in range(2 * N_DQ):
            e.raw(f"v_accvgpr_write_b32 {ar(KTF(0) + i)}, {vr(POOL0 + i)}")
    e.raw("s_barrier")

    plans = [plan_reads(e, pool, u % NS, u) for u in range(COPIES)] + [None]
    # pair of block u - 2 (u = 0, 1: none) begins in copy u - 1 and ends in copy u
    dq = [plan_dq(e, pool, u % 2, f"{u}x") for u in range(COPIES + 2)]          # dq[u]: the pair finished in copy u
    merged = [{k: plans[0][k] + dq[0][1][0][k] for k in range(-EARLY, 0)}]
    for k in range(-EARLY, 0):
        for fn in merged[0][k]:
            fn()
    e.need("0nd3")
    l_done = e.label("done")
    l_tail = [e.label("tail0"), e.label("tail1")]
    l_whole, l_masked = ([e.label(f"{x}{u}") for u in range(COPIES)] for x in ("whole", "masked"))
    strip = lambda tags: [t.lstrip("0123456789") for t in tags]
    entry, entry_pool = list(e.ds), pool.state()
    at = [(strip(entry), pool.next % pool.size)]
    e.raw(f"s_cmp_le_u32 {sr(T_REM)}, {sr(S_EVT)}")
    e.raw(f"s_cbranch_scc1 {l_masked[0]}")
    stubs = []
    for masked in (False, True):
        if masked:
            e.ds = list(entry)
            pool.restore(entry_pool)
        for u in range(COPIES):
            e.raw((l_masked if masked else l_whole)[u] + ":")
            assert (strip(e.ds), pool.next % pool.size) == at[u], (e.ds, at[u])
            if u == COPIES - 1:
                plans[COPIES] = plan_reads(e, pool, 0, COPIES)
            gen_step(e, pool, u, u, plans[u], plans[u + 1], dq[u][1], dq[u + 1][1], dq[u + 1][0], masked)
            e.raw(f"s_sub_u32 {sr(T_REM)}, {sr(T_REM)}, 1")
            # in this copy the pair of block u - 1 has begun, whose dS lies in buffer (u + 1) % 2
            if masked:
                e.raw(f"s_cmp_eq_u32 {sr(T_REM)}, 0")
                e.raw(f"s_cbranch_scc1 {l_tail[(u + 1) % 2]}")
                e.raw(f"s_cmp_gt_u32 {sr(T_REM)}, {sr(S_EVT)}")
                e.raw(f"s_cbranch_scc1 {l_whole[(u + 1) % COPIES]}")
            else:
                l_leave = e.label("leave")
                stubs.append((l_leave, l_masked[(u + 1) % COPIES], l_tail[(u + 1) % 2]))
                e.raw(f"s_cmp_le_u32 {sr(T_REM)}, {sr(S_EVT)}")
                e.raw(f"s_cbranch_scc1 {l_leave}")
            if not masked and u < COPIES - 1:
                at.append((strip(e.ds), pool.next % pool.size))
        # writes of dS may be under way here that are not behind the prologue: waits made without them wait for more
        assert ([t for t in strip(e.ds) if not t.startswith("ds")], pool.next % pool.size) == at[0], (e.ds, at[0])
        e.raw(f"s_branch {(l_masked if masked else l_whole)[0]}")
    for l_leave, l_to, l_end in stubs:
        e.raw(l_leave + ":")
        e.raw(f"s_cmp_lg_u32 {sr(T_REM)}, 0")
        e.raw(f"s_cbranch_scc1 {l_to}")
        e.raw(f"s_branch {l_end}")
    e.raw(l_mask + ":")
    gen_mask_routine(e)
    for buf in range(2):
        e.raw(l_tail[buf] + ":")
        gen_tail(e, buf)
        e.raw(f"s_branch {l_done}")
    for wait in e.waits:
        gen_polls(e, *wait)
    e.raw(l_done + ":")
    e.comment("---- what the epilogue needs, from LDS")
    e.raw(f"s_add_u32 {sr(T_X)}, {sr(S_LDS)}, {PBLK + 256 * 32}")
    e.raw(f"v_mov_b32 {vr(TMP)}, {sr(T_X)}")
    for i in range(3):
        e.raw(f"ds_read_b128 {vr(160 + 4 * i, 4)}, {vr(TMP)} offset:{32 + 16 * i}")
    e.raw("s_waitcnt lgkmcnt(0)")
    for word, dst in ((U_DKPTR, kv.S_DKPTR), (U_DKPTR + 1, kv.S_DKPTR + 1), (U_DVPTR, kv.S_DVPTR), (U_DVPTR + 1, kv.S_DVPTR + 1),
                      (U_RS32, kv.S_RS32), (U_SCALE, kv.S_SCALE), (U_FLAGS, S_FLAGS), (U_DKLP, kv.S_DKLP), (U_DKLP + 1, kv.S_DKLP + 1),
                      (U_DVLP, kv.S_DVLP), (U_DVLP + 1, kv.S_DVLP + 1)):
        e.raw(f"v_readfirstlane_b32 {sr(dst)}, {vr(160 + word - 8)}")
    kv.epilogue(e, ragged_tiles=False)
    return e


def main():
    e = generate()
    clob = [f"v{i}" for i in range(256) if not (kv.IN_V <= i < kv.IN_V + 16)] + [f"a{i}" for i in range(256)]
    clob += [f"s{i}" for i in range(64, 96)]
    write_inc(sys.stdout, "gen_bwd_one_asm.py" + (" 64" if D == 64 else ""), "ST_ONE_FAST" + ("64" if D == 64 else ""), e, LDS_BYTES, clob)


if __name__ == "__main__":
    main()
