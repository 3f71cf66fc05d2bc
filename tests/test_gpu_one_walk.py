"""Ring backwards that make dK, dV and dQ in one walk over the key tiles, against the fp64 oracle and the two passes: dQ is passed on from
key tile to key tile of a KV head, two blocks behind the one in hand, so what can go wrong lies at the ends of walks (1 to 7 blocks, the
loop has six copies of one, of head size 64 four), at blocks that reach beyond the shard, at tiles whose walks are shorter than the one before, and in chains
longer than an XCD has workgroups.  Tolerance: the bf16 bounds of assert_close_wide."""
import pytest
import torch

import paper_2407_00611_amd as st
import synth_inputs as si
from oracle import attention as oa
from test_backward_plans import BF16, FUSED, Share, _ring
from util import assert_close_wide, host, launcher_switch, positions, upload

#        B, Hq, Hkv,  Sq,  Sk,  n, q_offset, (q_seg, q_offset2), causal
CASES = [(1, 1, 1, 1, 256, 1, 255, (0, 0), True),                  # one row
         (1, 2, 1, 33, 256, 2, 256, (0, 0), True),                 # a ragged block of one row first, the diagonal last
         (1, 3, 1, 64, 256, 1, 0, (0, 0), True),                   # most keys are seen by nobody
         (1, 6, 2, 96, 256, 3, 100, (0, 0), True),                 # the diagonal crosses two tiles; one head more than a power of two
         (1, 2, 2, 128, 256, 3, 0, (0, 0), False),
         (1, 4, 4, 160, 512, 2, 700, (0, 0), True),
         (2, 4, 2, 223, 256, 4, 801, (0, 0), True),                # batch 2, offsets at no boundary
         (1, 2, 2, 300, 768, 2, 1236, (0, 0), True),
         (1, 4, 2, 512, 256, 8, 256, (256, 1792), True),           # two runs
         (1, 2, 1, 330, 256, 6, 100, (130, 1200), True),           # two runs of unlike length, their boundary inside a block
         (1, 16, 16, 256, 256, 40, 39 * 256, (0, 0), True),        # chains of 40 tiles, two heads in a batch
         (1, 2, 1, 512, 256, 2, -200, (0, 0), True),               # rows that see nothing: no sums of theirs
         (1, 4, 2, 400, 256, 1, -100, (170, 120), True),           # the same and two runs
         (1, 12, 12, 200, 256, 5, 1080, (0, 0), False),
         (1, 24, 3, 64, 256, 66, 65 * 256, (0, 0), True)]          # two launches


def _share(c, D):
    B, Hq, Hkv, Sq, Sk, n, q0, (seg, q2), causal = c
    w = si.Workload("one_walk", 420 + Sq % 50, "bf16", B, Hq, Hkv, D, Sq, Sk, n, q0, causal, True, q_seg=seg, q_offset2=q2)
    return w, si.make_inputs(w), [w.k_offset(j) for j in range(n)]


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("c", CASES, ids=[f"h{c[1]}_{c[2]}_q{c[3]}_n{c[5]}" for c in CASES])
def test_all_gradients_in_one_walk(c, D):
    B, Hq, Hkv, Sq, Sk, n, q0, (seg, q2), causal = c
    print(f"[one walk] {c} D={D}", flush=True)
    w, inp, koffs = _share(c, D)
    q, ks, vs, d_o = upload(inp)
    pos, order, args = positions(w), list(range(n)), (w.q_where, koffs, causal, w.scale)
    o, lse, low = st.st_ring_fwd(q, ks, vs, *args, order)
    dq_r, dk_r, dv_r = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, *pos, causal, w.scale)

    def check(dq, dk, dv, what):
        assert_close_wide(host(dq) - 1 / 64, dq_r, f"{what} dq")          # the start costs 1e-9 per element
        for j in range(n):
            for name, x, ref in (("dk", dk[j], dk_r[j]), ("dv", dv[j], dv_r[j])):
                if ref.any():
                    assert_close_wide(host(x), ref, f"{what} {name}[{j}]")
                else:
                    assert not x.any(), f"{what} {name}[{j}]: of keys that nobody sees"

    def run(call, start):
        dq = torch.full_like(o, 1 / 64)
        dk, dv = ([torch.full(k.shape, start, device="cuda") for k in ks] for _ in range(2))
        st.st_profile_begin()
        try:
            call(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv)
        finally:
            ran = st.st_profile_end()
        return (dq, dk, dv), ran

    with launcher_switch("one_walk", 2, 1):
        size = st.st_ring_workspace_bytes(q, ks, vs, *args, st.ST_RING_FUSED, True)
        ws = lambda n_bytes: torch.full((n_bytes + 256,), 0xff, dtype=torch.uint8, device="cuda")     # NaN
        got, ran = run(lambda *a: st.st_ring_bwd(*a, workspace=ws(size)), 0.0)
        assert ran["bwd_one_bf16"][0] == (n + 63) // 64 and "bwd_dkv_bf16" not in ran, ran
        check(*got, "added")
        again, _ = run(lambda *a: st.st_ring_bwd(*a, workspace=ws(size)), 0.0)
        other, _ = run(lambda *a: st.st_ring_bwd_noalloc(*a), 0.0)
        for x in (again, other):
            assert all(torch.equal(a, b) for a, b in zip([x[0], *x[1], *x[2]], [got[0], *got[1], *got[2]]))
        lows = [[torch.empty_like(k) for k in ks] for _ in range(2)]
        last, ran = run(lambda *a: st.st_ring_bwd_last(*a, assign=True, dk_lowp=lows[0], dv_lowp=lows[1], workspace=ws(size)), float("nan"))
        assert "bwd_one_bf16" in ran
        check(*last, "assigned")
        for x, y in zip(last[1] + last[2], lows[0] + lows[1]):
            assert torch.equal(x.to(torch.bfloat16), y)
        # a workspace without room for the sums' way from tile to tile: two passes
        base = (B * Hq * Sq * 4 + 255) // 256 * 256 + 1024 + (q.numel() * 2 + 255) // 256 * 256
        less, ran = run(lambda *a: st.st_ring_bwd(*a, workspace=ws(base)), 0.0)
        assert "bwd_one_bf16" not in ran
        check(*less, "two passes")


#          heads of a batch; B, Hq, Hkv, Sq, Sk, n, q_offset, (q_seg, q_offset2), causal
BATCHES = [(2, (1, 16, 16, 96, 256, 3, 672, (0, 0), True)),
           (3, (2, 12, 12, 70, 256, 12, 3002, (0, 0), True)),      # 36 tiles a batch: more than an XCD has workgroups
           (3, (1, 48, 24, 64, 512, 2, 0, (0, 0), False)),
           (4, (2, 32, 16, 100, 256, 9, 1000, (50, 2254), True)),  # the last chunks are seen by one run, or by nobody
           (5, (1, 5, 5, 128, 256, 2, 384, (0, 0), True)),         # one batch: seven XCDs have none
           (8, (2, 32, 32, 64, 256, 5, 1216, (0, 0), True)),
           (8, (1, 24, 24, 160, 256, 4, 0, (0, 0), False))]


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("heads,c", BATCHES, ids=[f"{b}_of_{c[0]}x{c[2]}_n{c[5]}" for b, c in BATCHES])
def test_batches_of_heads(heads, c, D):
    """A ticket of an XCD is a tile of one of the heads of its batch, the heads in turn.  Which ones are walked together changes no bit;
    the planner takes one head or all of an XCD's (3, 4 and 8 for 24, 32 and 64)."""
    B, Hq, Hkv, Sq, Sk, n, q0, (seg, q2), causal = c
    print(f"[one walk] batches of {heads}: {c} D={D}", flush=True)
    w, inp, koffs = _share(c, D)
    q, ks, vs, d_o = upload(inp)
    order, args = list(range(n)), (w.q_where, koffs, causal, w.scale)
    o, lse, low = st.st_ring_fwd(q, ks, vs, *args, order)
    share = Share(BF16, B, Hq, Hkv, D, Sq, Sk, koffs, q0, causal, seg, q2)

    def run():
        dq, dk, dv = torch.zeros_like(o), [torch.empty(k.shape, device="cuda") for k in ks], [torch.empty(k.shape, device="cuda") for k in ks]
        st.st_ring_bwd_last(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv, assign=True)
        return dq, dk, dv

    with launcher_switch("one_walk", 2, 1):
        got = []
        for batch in (heads, 1):
            with launcher_switch("one_heads", batch, 0):
                assert [x[9] for x in share.plan(order, FUSED, True, -1)] == [-batch]
                got.append(run())
    for a, b in zip(*[[x[0], *x[1], *x[2]] for x in got]):
        assert torch.equal(a, b)
    dq_r, dk_r, dv_r = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, *positions(w), causal, w.scale)
    assert_close_wide(host(got[0][0]), dq_r, "dq")
    for j in range(n):
        for name, x, ref in (("dk", got[0][1][j], dk_r[j]), ("dv", got[0][2][j], dv_r[j])):
            if ref.any():
                assert_close_wide(host(x), ref, f"{name}[{j}]")
            else:
                assert not x.any(), f"{name}[{j}]"


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("layout", ["k_heads_first", "v_heads_first", "k_packed", "all_heads_first"])
def test_any_memory_layout(layout, causal, D):
    """K lies in LDS here and V in registers, the other way round than in the dK/dV loop, and head size 64 reads K a second time: with
    strides of K and V unlike each other, batch 2, grouped heads and (causal) the chunks in another order, the same bits as dense."""
    print(f"[one walk] {layout}, causal {causal}, D={D}", flush=True)
    n = 3
    w, inp, koffs = _share((2, 6, 3, 200, 512, n, 3 * 512 - 200 if causal else 0, (0, 0), causal), D)
    q, ks, vs, d_o = upload(inp)
    args = (w.q_where, koffs, causal, w.scale)
    heads_first = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)

    def packed(t):                                                  # beside other data: rows four heads further apart
        wide = torch.full((*t.shape[:2], t.shape[2] + 4, D), float("nan"), dtype=t.dtype, device="cuda")
        wide[:, :, 2:-2] = t
        return wide[:, :, 2:-2]

    same = lambda t: t
    how_q, how_k, how_v, how_do = {"k_heads_first": (same, heads_first, same, packed), "v_heads_first": (packed, same, heads_first, same),
                                   "k_packed": (heads_first, packed, heads_first, same), "all_heads_first": (heads_first,) * 4}[layout]
    o, lse, low = st.st_ring_fwd(q, ks, vs, *args, list(range(n)))

    def run(q, ks, vs, d_o, low, order):
        dq, dk, dv = torch.zeros_like(o), [torch.zeros(k.shape, device="cuda") for k in ks], [torch.zeros(k.shape, device="cuda") for k in ks]
        st.st_profile_begin()
        try:
            st.st_ring_bwd(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv)
        finally:
            ran = st.st_profile_end()
        assert "bwd_one_bf16" in ran
        return [dq, *dk, *dv]

    with launcher_switch("one_walk", 2, 1):
        want = run(q, ks, vs, d_o, low, [0, 1, 2])
        got = run(how_q(q), [how_k(x) for x in ks], [how_v(x) for x in vs], how_do(d_o), how_do(low), [2, 0, 1] if causal else [0, 1, 2])
    assert all(torch.equal(x, y) for x, y in zip(got, want))
    dq_r, dk_r, dv_r = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, *positions(w), causal, w.scale)
    assert_close_wide(host(want[0]), dq_r, "dq")
    for j in range(n):
        assert_close_wide(host(want[1 + j]), dk_r[j], f"dk[{j}]")
        assert_close_wide(host(want[1 + n + j]), dv_r[j], f"dv[{j}]")


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
def test_one_walk_in_a_graph(D):
    """Replays with eager work between them, each compared with the eager result; the counts start anew in every launch."""
    w, inp, koffs = _share((1, 8, 8, 256, 256, 6, 1280, (0, 0), True), D)
    q, ks, vs, d_o = upload(inp)
    args, order = (w.q_where, koffs, True, w.scale), list(range(6))
    with launcher_switch("one_walk", 2, 1):
        o, lse, low = st.st_ring_fwd(q, ks, vs, *args, order)
        ws = torch.empty(st.st_ring_workspace_bytes(q, ks, vs, *args, st.ST_RING_FUSED, True) + 256, dtype=torch.uint8, device="cuda")
        dq, dk, dv = torch.zeros_like(o), [torch.empty(k.shape, device="cuda") for k in ks], [torch.empty(k.shape, device="cuda") for k in ks]

        def step():
            dq.zero_()
            st.st_ring_bwd_last(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv, assign=True, workspace=ws)

        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            step()
            torch.cuda.synchronize()
            want = [x.clone() for x in (dq, *dk, *dv)]
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                step()
        for _ in range(4):
            for x in (dq, *dk, *dv):
                x.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip((dq, *dk, *dv), want))
            step()


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
def test_a_wait_that_gives_up_is_not_silent(D):
    """With a single poll a wait, tiles go on before the one ahead of them has counted a pair.  The launch ends, its gradients are NaN, all
    of them, and the next one in the same workspace is right."""
    print(f"[one walk] waits of one poll, D={D}", flush=True)
    w, inp, koffs = _share((1, 8, 8, 256, 256, 8, 2048, (0, 0), True), D)
    q, ks, vs, d_o = upload(inp)
    args, order = (w.q_where, koffs, True, w.scale), list(range(8))
    with launcher_switch("one_walk", 2, 1):
        o, lse, low = st.st_ring_fwd(q, ks, vs, *args, order)
        ws = torch.empty(st.st_ring_workspace_bytes(q, ks, vs, *args, st.ST_RING_FUSED, True) + 256, dtype=torch.uint8, device="cuda")

        def step():
            dq, dk, dv = torch.zeros_like(o), [torch.zeros(k.shape, device="cuda") for k in ks], [torch.zeros(k.shape, device="cuda") for k in ks]
            dkl, dvl = ([torch.zeros_like(k) for k in ks] for _ in range(2))
            st.st_ring_bwd_last(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv, assign=True, dk_lowp=dkl, dv_lowp=dvl, workspace=ws)
            torch.cuda.synchronize()
            return [dq, *dk, *dv, *dkl, *dvl]

        want = step()
        with launcher_switch("one_polls", 1, 1 << 21):
            assert all(x.isnan().all() for x in step())
        assert not any(x.isnan().any() for x in want) and all(torch.equal(x, y) for x, y in zip(step(), want))


@pytest.mark.gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Sq,q0,n", [(64, 0, 1), (128, 256, 3), (192, 256, 2)])
def test_keys_that_no_row_sees_may_hold_anything(Sq, q0, n, D):
    """A key tile meets 256 keys, seen or not, and 0 times a NaN is one: what lies behind the last key that a row sees (here at the
    end of a 64-key tile, where the forward ends) must not reach dQ, as it does not in two passes.  Bit for bit what finite keys give."""
    print(f"[one walk] keys nobody sees, {Sq} rows at {q0}, {n} chunks, D={D}", flush=True)
    w, inp, koffs = _share((1, 4, 2, Sq, 256, n, q0, (0, 0), True), D)
    q, ks, vs, d_o = upload(inp)
    args, order = (w.q_where, koffs, True, w.scale), list(range(n))
    o, lse, low = st.st_ring_fwd(q, ks, vs, *args, order)

    def grads(ks, vs):
        dq, dk, dv = torch.zeros_like(o), [torch.zeros(k.shape, device="cuda") for k in ks], [torch.zeros(k.shape, device="cuda") for k in ks]
        st.st_profile_begin()
        try:
            st.st_ring_bwd(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv)
        finally:
            ran = st.st_profile_end()
        assert "bwd_one_bf16" in ran
        return [dq, *dk, *dv]

    with launcher_switch("one_walk", 2, 1):
        want = grads(ks, vs)
        for bad in (float("nan"), float("inf")):
            other = [[x.clone() for x in xs] for xs in (ks, vs)]
            for xs in other:
                for j, x in enumerate(xs):
                    x[:, max(q0 + Sq - koffs[j], 0):] = bad
            assert any((x != y).any() for x, y in zip(other[0], ks))
            assert all(torch.equal(x, y) for x, y in zip(grads(*other), want))


def test_where_one_walk_is_planned():
    """By the work of the longest chain: not where an XCD has no head, nor for few tiles, nor for chunks that overlap, tiles of fewer
    keys than the loop takes, or more sums than there is room for."""
    def batch(share):
        p = share.plan(list(range(len(share.offsets))), FUSED, True, -1)[0]
        return max(-p[9], 0), p[-1]
    assert batch(_ring(BF16, 1, 32, 8, 128, 4096, 32, 31))[0] == 1
    assert batch(_ring(BF16, 1, 32, 32, 128, 2048, 16, 15))[0] in (1, 4)
    assert batch(_ring(BF16, 1, 32, 32, 128, 512, 8, 7))[0] == 4
    assert batch(_ring(BF16, 2, 12, 4, 128, 1000, 6, 5))[0] == 0
    assert batch(_ring(BF16, 1, 16, 4, 128, 4096, 8, 7))[0] == 0
    assert batch(_ring(BF16, 1, 32, 8, 128, 1024, 8, 0))[0] == 0
    assert batch(Share(BF16, 1, 32, 8, 128, 4096, 4096, [2048 * j for j in range(32)], 64000))[0] == 0
    assert batch(_ring(BF16, 1, 32, 8, 128, 16384, 8, 7))[0] == 1            # 256 MiB of them: more than st_ring_bwd_noalloc takes shares for
    assert batch(_ring(BF16, 1, 32, 8, 128, 32768, 4, 3))[0] == 0
    assert batch(_ring(BF16, 1, 24, 24, 64, 16384, 8, 3, False))[0] in (1, 3)
    heads, size = batch(_ring(BF16, 1, 32, 8, 128, 4096, 32, 31))
    # 16 KiB a pair of head and block, two more a KV head, and less than 1 MiB of counts
    assert 0 <= size - 16384 * (32 * 128 + 2 * 8) < 1 << 20


@pytest.mark.parametrize("share,heads", [(_ring(BF16, 1, 16, 16, 128, 1024, 8, 7), 2), (_ring(BF16, 1, 24, 24, 64, 16384, 8, 3, False), 3),
                                         (_ring(BF16, 2, 16, 16, 64, 512, 8, 5), 4), (_ring(BF16, 1, 48, 48, 128, 512, 8, 7), 6),
                                         (_ring(BF16, 1, 64, 64, 64, 512, 8, 7), 8)], ids=lambda x: x.text if isinstance(x, Share) else str(x))
def test_batches_that_are_planned(share, heads):
    """All heads of an XCD at once where chains are short (the others run one head's tiles behind each other: the case above)."""
    assert share.plan(list(range(len(share.offsets))), FUSED, True, -1)[0][9] == -heads
