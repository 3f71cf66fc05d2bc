"""Masked and ragged tiles in the hand-scheduled bf16 forward, against the fp64 oracle: chunk lengths around the 64-key tile,
query counts around the 64 rows of a wavefront and the 256 of a workgroup, the diagonal at every alignment, shards in two
runs that meet inside a tile, walks without a single tile that all rows see, and splits that cut the masked part.
Tolerance: the bf16 bounds of assert_close."""
import numpy as np
import pytest
import torch

import paper_2407_00611_amd as st
import synth_inputs as si
from oracle import attention as oa
from util import assert_close, assert_close_wide, host, positions, upload

pytestmark = pytest.mark.gpu

#        D, Hq, Hkv, Sq, Sk, n, q_offset, causal, (q_seg, q_offset2)
CASES = [(128, 1, 1, 1, 64, 1, 63, True, (0, 0)),
         (128, 2, 1, 65, 65, 2, 65, True, (0, 0)),
         (128, 1, 1, 255, 127, 3, 126, True, (0, 0)),
         (128, 3, 1, 257, 129, 2, 0, False, (0, 0)),
         (128, 1, 1, 300, 64, 6, 30, True, (0, 0)),              # every tile is crossed, some rows see nothing
         (128, 2, 2, 512, 192, 4, 256, True, (200, 600)),         # two runs that meet inside a query tile
         (128, 1, 1, 40, 448, 2, 880, True, (0, 0)),
         (64, 2, 1, 1, 500, 1, 20, True, (0, 0)),
         (64, 1, 1, 320, 500, 2, 690, True, (0, 0)),
         (64, 2, 2, 257, 449, 3, 0, False, (0, 0)),
         (64, 1, 1, 300, 130, 4, 100, True, (33, 360)),
         # no causal mask: ragged chunks, and two runs inside a query tile whose distance does not fit 30 bits
         (128, 1, 1, 256, 129, 4, 0, False, (100, 3 << 29)),
         (64, 2, 1, 200, 129, 4, 0, False, (70, 1 << 31))]


def _check(w, inp, orders, mode=st.ST_RING_FUSED, close=assert_close, **kw):
    q, ks, vs, _ = upload(inp)
    q_pos, k_pos = positions(w)
    koffs = [w.k_offset(j) for j in range(w.n_chunks)]
    o_ref, lse_ref = oa.attention_forward(inp.q, inp.k, inp.v, q_pos, k_pos, w.causal, w.scale)
    for order in orders:
        o, lse, low = st.st_ring_fwd(q, ks, vs, w.q_where, koffs, w.causal, w.scale, order, None, mode)
        close(host(o), o_ref, *kw.get("args", ()), "o")
        close(host(lse), lse_ref, *kw.get("args", ()), "lse", lse=True)
        assert torch.equal(low, o.to(torch.bfloat16))


@pytest.mark.parametrize("mode", [st.ST_RING_FUSED, st.ST_RING_STEPWISE], ids=["fused", "stepwise"])
@pytest.mark.parametrize("c", CASES, ids=[f"d{c[0]}_q{c[3]}_k{c[4]}" for c in CASES])
def test_forward_at_tile_edges(c, mode):
    D, Hq, Hkv, Sq, Sk, n, q0, causal, (seg, q2) = c
    w = si.Workload("masks", 320 + Sq % 50, "bf16", 1, Hq, Hkv, D, Sq, Sk, n, q0, causal, False, q_seg=seg, q_offset2=q2)
    print(f"[masks] {c} mode {mode}", flush=True)
    _check(w, si.make_inputs(w), [list(range(n)), list(range(n))[::-1]], mode, args=("bf16",))


@pytest.mark.parametrize("D", [128, 64])
def test_rows_that_meet_their_first_key_late(D):
    """Every tile is masked (the shard's 256 rows start before the chunk's keys do) and every score lies some hundred
    log2 units below zero: the exponent reference of a row must come from the first block in which it sees a key."""
    w = si.Workload("late", 330, "bf16", 1, 1, 1, D, 256, 512, 1, -100, True, False)
    inp = si.make_inputs(w)
    # a common direction: <q, k> = -3 D plus noise, so scale * log2 e * <q, k> is about -49 (D = 128) and below;
    # with four times the keys, below -190: exp2 of it is zero in fp32
    for a, bits in ((inp.q, inp.q_bits), (inp.k[0], inp.k_bits[0])):
        a[:] = si.bf16_bits_to_f32(si.f32_to_bf16_bits(a * 0.25 + (1.0 if a is inp.q else -12.0 * np.sqrt(128 / D))))
        bits[:] = si.f32_to_bf16_bits(a)
    q_pos, k_pos = positions(w)
    _, lse_ref = oa.attention_forward(inp.q, inp.k, inp.v, q_pos, k_pos, True, w.scale)
    assert np.isneginf(lse_ref[..., :100]).all() and lse_ref[..., 100:].max() < -100     # exp2 underflows at -149
    _check(w, inp, [[0]], close=lambda x, r, what, lse=False: assert_close_wide(x, r, what, lse=lse))


#        D, Sq, Sk, n, q_offset, causal
EQUAL = [(128, 300, 300, 1, 0, True), (64, 520, 520, 2, 0, True), (128, 200, 130, 3, 0, False), (64, 270, 500, 2, 700, True)]


@pytest.mark.parametrize("mode", [st.ST_RING_FUSED, st.ST_RING_STEPWISE], ids=["fused", "stepwise"])
@pytest.mark.parametrize("c", EQUAL, ids=[f"d{c[0]}_q{c[1]}_k{c[2]}" for c in EQUAL])
def test_the_largest_probability_carries_no_rounding(c, mode):
    """A row's exponent reference is its maximum, so a key that holds it has P = 1 in bf16.  A row that sees one key returns
    its V bit for bit; where all keys are alike O is the mean of the visible V to fp32 accuracy: every P is 1, and the row
    sum is off by the rounding of scores of at most 32 log2 units summed in 8 steps, 8 * 32 * 2^-24 * ln 2 = 1.1e-5."""
    D, Sq, Sk, n, q0, causal = c
    w = si.Workload("equal", 342, "bf16", 1, 2, 1, D, Sq, Sk, n, q0, causal, False)
    print(f"[equal keys] {c} {mode}", flush=True)
    inp = si.make_inputs(w)
    for k, bits in zip(inp.k, inp.k_bits):
        k[:], bits[:] = inp.k[0][:, :1], inp.k_bits[0][:, :1]
    q, ks, vs, _ = upload(inp)
    q_pos, k_pos = positions(w)
    o_ref, _ = oa.attention_forward(inp.q, inp.k, inp.v, q_pos, k_pos, causal, w.scale)
    o, _, _ = st.st_ring_fwd(q, ks, vs, q0, [w.k_offset(j) for j in range(n)], causal, w.scale, list(range(n)), None, mode)
    assert np.abs(host(o) - o_ref).max() <= 2e-5 * np.abs(o_ref).max()
    if causal and q0 == 0:
        assert torch.equal(o[:, 0], vs[0][:, 0].float().expand(1, 2, D))


def test_split_cuts_the_masked_part():
    """One head, so the walk of every query tile is split sixteen ways and some splits hold masked tiles only."""
    w = si.Workload("split_masks", 331, "bf16", 1, 1, 1, 128, 700, 700, 3, 1400, True, False)
    st.st_profile_begin()
    _check(w, si.make_inputs(w), [[0, 1, 2], [2, 0, 1]], args=("bf16",))
    assert "combine" in st.st_profile_end(), "this share was meant to be split"


@pytest.mark.parametrize("D", [128, 64])
def test_the_state_of_an_empty_share_stays_out(D):
    """65 query tiles, more than have numbers of shares of their own: the plan counts the tiles of the last rows, and of the
    first query tile, which sees one key tile, some shares have none.  They leave their O unwritten, here NaN, behind an lse of
    -inf."""
    Sq = 65 * 256
    w = si.Workload("empty_shares", 343, "bf16", 1, 1, 1, D, Sq, 4096, 1, -200, True, False)
    inp = si.make_inputs(w)
    q, ks, vs, _ = upload(inp)
    b_o, b_l = q.numel() * 4, Sq * 4
    need = st.st_ring_workspace_bytes(q, ks, vs, w.q_offset, [0], True, w.scale, st.ST_RING_FUSED, False)
    shares = need // (b_o + b_l)
    assert shares > 1, "this share was meant to be split"
    ws = torch.full((need + 256,), 0xff, dtype=torch.uint8, device="cuda")
    o, lse, low = st.st_ring_fwd(q, ks, vs, w.q_offset, [0], True, w.scale, [0], workspace=ws)
    first, empty = (-ws.data_ptr()) % 256, 0
    for y in range(shares):
        state = ws[first + y * (b_o + b_l):first + (y + 1) * (b_o + b_l)].view(torch.float32)
        if torch.isneginf(state[b_o // 4:b_o // 4 + 256]).all():
            assert torch.isnan(state[:256 * D]).all()
            empty += 1
    assert empty > 0, "every share of the first query tile had a tile"
    o_ref, lse_ref = oa.attention_forward(inp.q, inp.k, inp.v, *positions(w), True, w.scale)
    assert_close(host(o), o_ref, "bf16", "o")
    assert_close(host(lse), lse_ref, "bf16", "lse", lse=True)
    assert torch.equal(low, o.to(torch.bfloat16))


def _backward(w, inp, mode, assign=None):
    q, ks, vs, d_o = upload(inp)
    koffs = [w.k_offset(j) for j in range(w.n_chunks)]
    order = list(range(w.n_chunks))
    args = (w.q_where, koffs, w.causal, w.scale, order)
    o, lse, low = st.st_ring_fwd(q, ks, vs, *args, None, mode)
    dq = torch.full_like(o, 0.25)                       # gradients are added to what is there
    dk = [torch.full(k.shape, float("nan") if assign else -0.5, device="cuda") for k in ks]
    dv = [x.clone() for x in dk]
    lows = None
    if assign is None:
        st.st_ring_bwd(q, ks, vs, d_o, low, lse, *args, dq, dk, dv, mode)
    else:
        lows = [[torch.empty_like(k) for k in ks] for _ in range(2)]
        st.st_ring_bwd_last(q, ks, vs, d_o, low, lse, *args, dq, dk, dv, assign=assign, dk_lowp=lows[0], dv_lowp=lows[1], mode=mode)
        for x, y in zip(dk + dv, lows[0] + lows[1]):
            assert torch.equal(x.to(torch.bfloat16), y)
    base = 0.0 if assign else -0.5
    q_pos, k_pos = positions(w)
    ref = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, q_pos, k_pos, w.causal, w.scale)
    assert_close(host(dq) - 0.25, ref[0], "bf16", "dq")
    for j in range(w.n_chunks):
        # few keys and hundreds of rows: gradients well above 1, bounded relative to the largest
        assert_close_wide(host(dk[j]) - base, ref[1][j], f"dk[{j}]")
        assert_close_wide(host(dv[j]) - base, ref[2][j], f"dv[{j}]")


@pytest.mark.parametrize("how", ["add", "assign", "add_lowp", "stepwise"])
@pytest.mark.parametrize("c", CASES, ids=[f"d{c[0]}_q{c[3]}_k{c[4]}" for c in CASES])
def test_backward_at_tile_edges(c, how):
    D, Hq, Hkv, Sq, Sk, n, q0, causal, (seg, q2) = c
    w = si.Workload("masks", 320 + Sq % 50, "bf16", 1, Hq, Hkv, D, Sq, Sk, n, q0, causal, True, q_seg=seg, q_offset2=q2)
    print(f"[masks backward] {c} {how}", flush=True)
    _backward(w, si.make_inputs(w), st.ST_RING_STEPWISE if how == "stepwise" else st.ST_RING_FUSED,
              {"assign": True, "add_lowp": False}.get(how))


def test_backward_split_over_workgroups():
    """One head against 60 tiles: the dQ pass is split, and its sums are the same from call to call and from st_ring_bwd to
    st_ring_bwd_noalloc; with a workspace of the unsplit size it runs unsplit, with room for one partial sum its first
    share adds to dq itself."""
    w = si.Workload("split_bwd", 332, "bf16", 1, 2, 1, 128, 300, 640, 6, 6 * 640 - 300, True, True)
    inp = si.make_inputs(w)
    _backward(w, inp, st.ST_RING_FUSED)
    q, ks, vs, d_o = upload(inp)
    koffs = [w.k_offset(j) for j in range(w.n_chunks)]
    args = (w.q_where, koffs, w.causal, w.scale)
    order = list(range(w.n_chunks))
    need = st.st_ring_workspace_bytes(q, ks, vs, *args, st.ST_RING_FUSED, True)
    n_o = (q.numel() * 4 + 255) // 256 * 256
    base = (w.Hq * w.Sq * 4 + 255) // 256 * 256 + 1024 + n_o // 2       # Delta, the counters, the scaled copy of Q
    assert need > base + n_o
    o, lse, low = st.st_ring_fwd(q, ks, vs, *args, order)
    got, launches = [], []
    for ws in (None, None, "noalloc", base, base + n_o):
        st.st_profile_begin()
        dq = torch.zeros_like(o)
        dk = [torch.zeros(k.shape, device="cuda") for k in ks]
        dv = [torch.zeros(k.shape, device="cuda") for k in ks]
        if ws == "noalloc":
            st.st_ring_bwd_noalloc(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv)
        else:
            buf = None if ws is None else torch.empty(ws + 256, dtype=torch.uint8, device="cuda")
            st.st_ring_bwd(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv, workspace=buf)
        launches.append(st.st_profile_end())
        got.append(dq)
    assert ["add_parts" in x for x in launches] == [True, True, True, False, True]
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    assert_close(host(got[3]), host(got[0]), "bf16", "dq unsplit")
    assert_close(host(got[4]), host(got[0]), "bf16", "dq of two shares and one partial sum")


@pytest.mark.parametrize("how", ["add", "assign", "add_lowp", "stepwise"])
@pytest.mark.parametrize("D", [128, 64])
def test_key_tiles_split_over_workgroups(D, how):
    """Grouped heads against two short chunks: four key tiles, each walked by several workgroups whose sums are added up;
    the causal shard leaves some shares of some tiles without a block, and a chunk in the future without any."""
    w = si.Workload("split_kv", 333, "bf16", 1, 4, 1, D, 1070, 300, 3, -200, True, True)
    print(f"[key tile split] D={D} {how}", flush=True)
    st.st_profile_begin()
    _backward(w, si.make_inputs(w), st.ST_RING_STEPWISE if how == "stepwise" else st.ST_RING_FUSED,
              {"assign": True, "add_lowp": False}.get(how))
    assert "add_kv_parts" in st.st_profile_end(), "the key tiles of this share were meant to be split"


def test_block_backward_with_and_without_room_for_partial_sums():
    w = si.Workload("split_block", 334, "bf16", 1, 8, 1, 128, 1024, 256, 1, 0, True, True)
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    q_pos, k_pos = positions(w)
    need = st.st_attn_block_bwd_workspace_bytes(q, ks[0], 0, 0, True, w.scale)
    small = q.numel() * 2
    assert need > small
    o, lse = st.st_attn_block_fwd(q, ks[0], vs[0], 0, 0, True, w.scale)
    delta = st.st_attn_delta(d_o, o)
    ref = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, q_pos, k_pos, True, w.scale)
    for size in (need, small):
        dq, dk, dv = torch.zeros_like(o), torch.zeros(ks[0].shape, device="cuda"), torch.zeros(ks[0].shape, device="cuda")
        st.st_profile_begin()
        st.st_attn_block_bwd(q, ks[0], vs[0], d_o, lse, delta, 0, 0, True, w.scale, dq, dk, dv,
                             workspace=torch.empty(size + 256, dtype=torch.uint8, device="cuda"))
        assert ("add_kv_parts" in st.st_profile_end()) == (size == need)
        assert_close(host(dq), ref[0], "bf16", "dq")
        assert_close_wide(host(dk), ref[1][0], "dk")
        assert_close_wide(host(dv), ref[2][0], "dv")


@pytest.mark.parametrize("assign", [True, False])
def test_listed_chunks_that_nobody_sees(assign):
    """Chunks in the shard's future, first, last and between the others in visit order: assigned to zero, or left as they
    are, and rounded, in the same launch as the chunks that have rows."""
    w = si.Workload("future", 335, "bf16", 1, 2, 1, 64, 130, 130, 5, 130, True, True)
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    koffs = [w.k_offset(j) for j in range(5)]
    order = [3, 0, 4, 1, 2]
    o, lse, low = st.st_ring_fwd(q, ks, vs, w.q_where, koffs, True, w.scale, order)
    dq = torch.zeros_like(o)
    dk = [torch.full(k.shape, float("nan") if assign else 1.25, device="cuda") for k in ks]
    dv = [x.clone() for x in dk]
    lk, lv = [torch.empty_like(k) for k in ks], [torch.empty_like(k) for k in ks]
    st.st_ring_bwd_last(q, ks, vs, d_o, low, lse, w.q_where, koffs, True, w.scale, order, dq, dk, dv, assign=assign,
                        dk_lowp=lk, dv_lowp=lv)
    q_pos, k_pos = positions(w)
    ref = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, q_pos, k_pos, True, w.scale)
    assert_close(host(dq), ref[0], "bf16", "dq")
    for j in range(5):
        for x, y, r in ((dk[j], lk[j], ref[1][j]), (dv[j], lv[j], ref[2][j])):
            assert torch.equal(x.to(torch.bfloat16), y)
            assert_close_wide(host(x) - (0.0 if assign else 1.25), r, f"chunk {j}")
            if j > 1:
                assert (x == (0.0 if assign else 1.25)).all()


@pytest.mark.parametrize("D,n,Sk", [(128, 64, 70), (64, 33, 64), (128, 17, 130)])
def test_walk_of_many_chunks(D, n, Sk):
    """A lane per chunk builds the walk: sums over all 64 lanes, over a row of 16 and one lane more, over two rows and one;
    the shard sits where the first chunks are seen whole, the middle ones in part and the last ones not at all."""
    w = si.Workload("many_chunks", 340, "bf16", 1, 1, 1, D, 300, Sk, n, (n // 2) * Sk + 13, True, False)
    print(f"[many chunks] D={D} n={n} Sk={Sk}", flush=True)
    rng = np.random.default_rng(n)
    _check(w, si.make_inputs(w), [list(range(n)), [int(x) for x in rng.permutation(n)]], args=("bf16",))


#       D, Hq, Hkv, Sq, Sk, n, q_offset, causal, (q_seg, q_offset2)
PAIRS = [(128, 4, 4, 300, 700, 4, 3 * 700 + 400, True, (0, 0)),
         (128, 6, 2, 200, 513, 6, 0, False, (0, 0)),
         (64, 4, 4, 333, 500, 6, 1700, True, (0, 0)),               # the last chunks are hidden
         (64, 8, 8, 260, 600, 4, 500, True, (130, 1500))]           # two runs of rows


@pytest.mark.parametrize("how", ["add", "assign", "add_lowp"])
@pytest.mark.parametrize("c", PAIRS, ids=[f"d{c[0]}_q{c[3]}_k{c[4]}" for c in PAIRS])
def test_both_backward_passes_in_one_launch(c, how):
    """Few key tiles with short walks leave compute units for the dQ pass beside them: one launch holds both."""
    D, Hq, Hkv, Sq, Sk, n, q0, causal, (seg, q2) = c
    w = si.Workload("pair", 341, "bf16", 1, Hq, Hkv, D, Sq, Sk, n, q0, causal, True, q_seg=seg, q_offset2=q2)
    print(f"[pair] {c} {how}", flush=True)
    st.st_profile_begin()
    _backward(w, si.make_inputs(w), st.ST_RING_FUSED, {"assign": True, "add_lowp": False}.get(how))
    assert "bwd_bf16" in st.st_profile_end(), "this share was meant to take the common launch"
