"""How ring backwards are split over workgroups (host logic, no launch): st_ring_bwd with the workspace the library asks for and
st_ring_bwd_noalloc promise the same bits, so both have to make the same plan, for every dtype, mask, mode and visited subset;
and what the plan stores has to fit what was asked for, which is no more than some plan of the share can use."""
import ctypes as C
import random
import time

import pytest

from paper_2407_00611_amd import api
from util import launcher_switch

F32, BF16, STEPWISE, FUSED = 0, 1, 0, 1
I64, I32 = C.c_int64, C.c_int32
_plan = C.CDLL(api.library_path()).st_testing_bwd_plan
_plan.restype, _plan.argtypes = C.c_int, [C.POINTER(api.st_ring_desc), C.POINTER(I32), I32, I32, I32, I64, C.POINTER(I64), I32]
PER_LAUNCH = 12                                                # values per launch, the last one the bytes of partial sums


class Share:
    def __init__(self, dtype, B, Hq, Hkv, D, Sq, Sk, offsets, q_offset=0, causal=True, seg=0, q2=0):
        n = len(offsets)
        self.offsets = (I64 * n)(*offsets)
        self.tables = (C.c_void_p * n)(*[0x10000] * n)
        self.d = api.st_ring_desc(dtype, B, Hq, Hkv, D, Sq, Sk, q_offset, int(causal), 0.1, n, self.tables, self.tables,
                                  Sk * Hkv * D, Hkv * D, D, Sk * Hkv * D, Hkv * D, D, self.offsets, seg, q2)
        up = lambda x: (x + 255) // 256 * 256
        self.base = up(B * Sq * Hq * 4) + 1024 + (up(B * Sq * Hq * D * 2) if dtype == BF16 else 0)     # Delta, counters, scaled Q
        self.text = f"{('f32', 'bf16')[dtype]} {B} x {Hq}/{Hkv} x {D}, {Sq} rows at {q_offset} ({seg}, {q2}), {n} x {Sk}, causal {causal}"

    def last_position(self):
        d = self.d
        return d.q_offset2 + d.Sq - d.q_seg - 1 if d.q_seg else d.q_offset + d.Sq - 1

    def size(self, mode):
        return int(api._lib.st_ring_workspace_bytes(C.byref(self.d), mode, 1))

    def plan(self, order, mode, assign, workspace):
        out = (I64 * (PER_LAUNCH * 256))()
        n = _plan(C.byref(self.d), (I32 * max(len(order), 1))(*order), len(order), mode, int(assign), workspace, out, len(out))
        assert n >= 0
        return [tuple(out[i:i + PER_LAUNCH]) for i in range(0, n, PER_LAUNCH)]


def _check(share, rng):
    n = len(share.offsets)
    some = rng.sample(range(n), rng.randint(1, n))
    for mode in (FUSED, STEPWISE):
        size = share.size(mode)
        for order in (list(range(n)), list(reversed(range(n))), some):
            for assign in (False, True):
                asked = share.plan(order, mode, assign, size)
                assert asked == share.plan(order, mode, assign, -1), f"noalloc plans otherwise: {share.text}, order {order}, mode {mode}"
                assert asked == share.plan(order, mode, assign, size + (200 << 20)), f"more room, another plan: {share.text}"
                assert all(x[-1] <= size - share.base for x in asked), share.text
                less = share.base + max([x[-1] for x in asked], default=0) // 2     # short of it: fewer workgroups, not more memory
                assert all(x[-1] <= less - share.base for x in share.plan(order, mode, assign, less)), share.text


def _ring(dtype, B, Hq, Hkv, D, S, n, rank, causal=True):
    return Share(dtype, B, Hq, Hkv, D, S, S, [S * j for j in range(n)], S * rank, causal)


@pytest.mark.parametrize("share", [
    _ring(F32, 1, 24, 3, 64, 678, 3, 0), _ring(F32, 2, 16, 2, 128, 512, 8, 0),        # 512 to 1023 query tiles, few key tiles
    Share(BF16, 1, 32, 4, 64, 4096, 32768, [0]),                                       # many keys, few of them seen
    _ring(BF16, 1, 1, 1, 128, 694, 8, 0, False), _ring(BF16, 1, 4, 4, 64, 2408, 2, 0, False)],  # no mask
    ids=lambda s: s.text)
def test_shares_whose_two_plans_differed(share):
    assert any(x[8] > 0 or x[9] > 1 or x[1] > 1 for x in share.plan(list(range(len(share.offsets))), FUSED, False, -1)), "meant to be split"
    _check(share, random.Random(1))


def test_random_shares():
    rng = random.Random(2407)
    split = 0
    for _ in range(400):
        dtype = rng.choice([F32, BF16])
        D = rng.choice([32, 64, 80, 128, 256]) if dtype == F32 else rng.choice([64, 128])
        hkv, g, B = rng.choice([1, 1, 2, 3, 8]), rng.choice([1, 1, 2, 4, 8]), rng.choice([1, 1, 2])
        S, n = int(2 ** rng.uniform(4, 10 if dtype == F32 else 13)), rng.choice([1, 2, 3, 4, 8, 16, 70])
        rank, causal = rng.randrange(n), rng.random() < 0.7
        if rng.random() < 0.25:                                # two runs of rows
            m = max(S // 2, 1)
            share = Share(dtype, B, hkv * g, hkv, D, 2 * m, m, [m * j for j in range(2 * n)], rank * m, causal, m, (2 * n - 1 - rank) * m)
        elif rng.random() < 0.3:                               # chunks of another length, anywhere
            share = Share(dtype, B, hkv * g, hkv, D, S, max(1, int(S * rng.uniform(0.1, 4))), [rng.randint(-S, 4 * S) for _ in range(n)], rng.randint(0, 2 * S), causal)
        else:
            share = _ring(dtype, B, hkv * g, hkv, D, S, n, rank, causal)
        split += any(x[-1] > 0 for x in share.plan(list(range(len(share.offsets))), FUSED, False, -1))
        _check(share, rng)
    assert split > 100


def test_the_common_launch_is_planned_where_the_launcher_takes_it():
    """A dQ walk of at most six 64-key tiles runs on the general kernel, in a launch of its own: a plan that counts on both passes
    in one would leave the key tiles whole and get neither (causal 2 x 6/3 heads x 259 rows: 38 us, split 28 and 7)."""
    rng = random.Random(66)
    pairs = 0
    for _ in range(600):
        D, hkv, g, B = rng.choice([64, 128]), rng.choice([1, 1, 2, 3, 8]), rng.choice([1, 1, 2, 4, 8]), rng.choice([1, 1, 2])
        S, n = rng.randint(16, 500), rng.choice([1, 2, 3])
        share = _ring(BF16, B, hkv * g, hkv, D, S, n, rng.randrange(n), rng.random() < 0.7)
        for mode in (-1, FUSED):
            for x in share.plan(list(range(n)), mode, False, -1):
                pairs += x[10]
                assert not x[10] or x[0] * ((S + 63) // 64) > 6, share.text
    assert pairs > 50
    assert Share(BF16, 2, 6, 3, 128, 259, 259, [0]).plan([0], -1, False, -1)[0][8] > 0        # split


def test_a_tie_goes_to_the_common_launch():
    """It is one launch less, and what the model has against it is too much rather than too little: 3 heads x 786 rows, last of 16
    ranks, 88 us together and 94 and a gap apart, was planned apart for want of 5 %."""
    share = _ring(BF16, 1, 3, 3, 128, 786, 16, 15)
    assert all(x[10] for x in share.plan(list(range(16)), FUSED, False, -1))


def test_key_tiles_that_fill_the_chip_by_themselves():
    """The common launch is looked for with every way to split them: 2 x 8/4 heads x 1728 rows x 573 keys, three blocks 172 us
    together and 224 in launches of their own."""
    share = Share(BF16, 2, 8, 4, 128, 1728, 573, [0, 573, 1146], 1146)
    assert all(x[10] and x[8] for x in share.plan([0, 1, 2], -1, False, -1))


def test_small_shares_ask_for_little():
    assert _ring(F32, 1, 1, 1, 64, 128, 4, 3).size(FUSED) <= 1 << 20              # 40 KB of it Delta and what surrounds it
    assert _ring(F32, 1, 8, 2, 128, 512, 8, 7).size(FUSED) <= 48 << 20
    assert _ring(BF16, 1, 4, 4, 64, 69, 8, 7).size(FUSED) <= 2 << 20


def _block_size(share, k_offset):
    d = share.d
    b = api.st_block_desc(d.dtype, d.B, d.Hq, d.Hkv, d.D, d.Sq, d.Sk, d.q_offset, k_offset, d.causal, d.scale, d.q_seg, d.q_offset2)
    return int(api._lib.st_attn_block_bwd_workspace_bytes(C.byref(b)))


def test_block_backwards():
    """One workspace, sized for any chunk of the ring, holds the plan of every other one; and it is no larger than some plan uses."""
    rng = random.Random(611)
    for _ in range(300):
        D, hkv, g, B = rng.choice([64, 128]), rng.choice([1, 1, 2, 3, 8]), rng.choice([1, 1, 2, 4, 8]), rng.choice([1, 1, 2])
        S, n = int(2 ** rng.uniform(4, 13)), rng.choice([1, 2, 3, 8])
        rank, causal, m = rng.randrange(n), rng.random() < 0.7, max(S // 2, 1)
        share = _ring(BF16, B, hkv * g, hkv, D, S, n, rank, causal) if rng.random() < 0.7 else \
            Share(BF16, B, hkv * g, hkv, D, 2 * m, m, [m * j for j in range(2 * n)], rank * m, causal, m, (2 * n - 1 - rank) * m)
        order = list(range(len(share.offsets)))
        best = share.plan(order, -1, False, -1)
        base = (B * share.d.Sq * hkv * g * D * 2 + 255) // 256 * 256
        for j in order:
            size = _block_size(share, share.offsets[j])
            assert share.plan(order, -1, False, size) == best == share.plan(order, -1, False, size + (200 << 20)), share.text
            assert causal or size - base == max(x[-1] for x in best), share.text
    assert _block_size(_ring(BF16, 1, 2, 2, 128, 320, 2, 1), 0) <= 8 << 20
    assert _block_size(_ring(BF16, 2, 16, 16, 64, 512, 8, 5), 0) <= 4 << 20


def test_what_a_plan_costs():
    """Every call plans, and the backwards below are some 80 to 625 us of GPU work.  Sizing them took 0.7 to 1.7 ms, planning two chunks of
    a causal ring 0.15 ms, while the model of the one walk was simulated job by job for every number of chunks; now 40 to 110 us
    and 10.  The bounds lie between, for the best of several runs."""
    def best(f):
        times = []
        for _ in range(12):
            start = time.perf_counter()
            f()
            times.append(time.perf_counter() - start)
        return min(times) * 1e6

    for heads, D, S in ((32, 128, 512), (32, 64, 256), (64, 128, 256), (24, 64, 512)):
        share = _ring(BF16, 1, heads, heads, D, S, 64, 3, False)
        assert best(lambda: share.size(FUSED)) < 400, share.text
    for share in (_ring(BF16, 1, 32, 32, 128, 1024, 32, 31), _ring(BF16, 1, 32, 32, 128, 2048, 16, 15)):
        assert best(lambda: share.plan([3, 7], FUSED, True, -1)) < 60, share.text
        assert best(lambda: share.size(FUSED)) < 70, share.text


def test_shares_whose_rows_the_one_walk_does_not_take():
    """Its loop keeps the bytes of 256 rows of K in 32 bits.  Rows further apart are planned in two passes, as well as if there were no
    other way: split, and in a workspace of that size.  (2 x 16 heads of 64 x 512 rows x 8 chunks, batches of 4 heads otherwise.)"""
    def share(stride):
        s = _ring(BF16, 2, 16, 16, 64, 512, 8, 5)
        s.d.k_stride_s = stride
        return s
    order = list(range(8))
    near, far = share((1 << 21) - 1), share(1 << 21)
    assert all(x[9] < 0 for x in near.plan(order, FUSED, True, -1))
    with launcher_switch("one_walk", 0, 1):
        two, size = far.plan(order, FUSED, True, -1), near.size(FUSED)
        assert two == near.plan(order, FUSED, True, -1) and any(x[10] or x[8] > 0 for x in two)
    assert far.plan(order, FUSED, True, -1) == two and far.size(FUSED) == size
    _check(far, random.Random(5))
