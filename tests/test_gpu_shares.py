"""Launches that are split over workgroups.  Where query tiles have unlike walks (a causal mask, two runs of rows) each tile has a
number of workgroups of its own, and the two runs have tiles of their own.  Forward and backward against the fp64 oracle, on
workspaces full of NaN: with the room that is asked for, with less, and with none for partial sums; and st_ring_bwd_noalloc,
which has to compute the bits of the first.  That a launch was split as it was meant to be is read off the kernels that ran."""
import pytest
import torch

import paper_2407_00611_amd as st
import synth_inputs as si
from oracle import attention as oa
from test_backward_plans import BF16, F32, FUSED, Share
from util import assert_close, assert_close_wide, host, positions, upload

pytestmark = pytest.mark.gpu

# dtype, B, Hq, Hkv, D, Sq, Sk, n, q_offset, (q_seg, q_offset2), causal, whether the forward is split, and how the backward is with
# the room that is asked for and with room for one dQ: Q, K: partial sums of dQ, of dK and dV; O: the first share of a query tile adds
# to dQ itself; P: both passes in one launch
CASES = [("bf16", 1, 2, 1, 128, 1500, 1500, 1, 0, (0, 0), True, True, "QKP", "KP"),                # the diagonal alone: 1 to 6 tiles' worth
         ("bf16", 2, 2, 2, 64, 1300, 700, 3, 650, (0, 0), True, True, "QKP", "QOP"),
         ("bf16", 1, 2, 1, 128, 200, 100, 8, 100, (100, 600), True, True, "QP", "QOP"),            # a tile per run
         ("bf16", 2, 1, 1, 128, 1030, 515, 6, 0, (515, 2575), True, True, "QKP", "QOP"),           # three tiles per run, ragged ends of three rows
         ("bf16", 1, 3, 1, 64, 1026, 513, 6, 1026, (513, 1539), True, True, "QKP", "P"),           # the runs touch; ragged ends of one row
         ("bf16", 1, 1, 1, 128, 700, 350, 5, 0, (257, 1300), True, True, "QKP", "QOP"),            # runs of unlike length
         ("bf16", 1, 1, 1, 64, 16384, 320, 8, -9000, (0, 0), True, True, "QKP", "KP"),             # 64 tiles, the first half of them sees nothing
         ("bf16", 1, 1, 1, 64, 16400, 320, 8, -9000, (0, 0), True, True, "QKP", "KP"),             # 65: one number for all
         # few key tiles with unlike walks: split into shares of one size, found through runs of tiles (of which there are
         # more than five in the first case: the last one is mixed), beside hidden chunks, with dQ in the same launch
         ("bf16", 1, 4, 1, 128, 1500, 100, 18, 0, (0, 0), True, True, "QKP", "KP"),
         ("bf16", 1, 8, 1, 64, 900, 450, 8, 450, (450, 2700), True, True, "QKP", "KP"),
         ("bf16", 2, 4, 2, 128, 1280, 640, 4, 0, (0, 0), True, True, "QKP", "KP"),
         ("bf16", 1, 8, 1, 128, 300, 2000, 2, 1800, (0, 0), True, True, "QKP", "P"),
         ("bf16", 1, 4, 1, 64, 600, 6000, 1, 0, (0, 0), True, True, "KP", "KP"),                   # most keys are seen by nobody
         ("bf16", 1, 4, 2, 128, 259, 259, 1, 0, (0, 0), True, True, "QK", ""),                     # a dQ walk too short for the common launch
         # no mask: every tile has the same number, which nothing looks up
         ("bf16", 1, 1, 1, 128, 694, 694, 8, 0, (0, 0), False, True, "QKP", "QOP"),
         ("bf16", 1, 4, 4, 64, 2408, 2408, 2, 0, (0, 0), False, True, "QP", "QOP"),
         ("f32", 1, 1, 1, 64, 1210, 1210, 1, 0, (0, 0), True, True, "QKP", "P"),
         ("f32", 2, 1, 1, 128, 140, 70, 12, 70, (70, 700), True, True, "QP", "QOP"),
         ("f32", 1, 1, 1, 256, 2048, 256, 3, -100, (0, 0), True, True, "QKP", "KP"),
         ("f32", 1, 8, 1, 40, 700, 70, 12, 0, (0, 0), True, False, "KP", "KP"),                    # few key tiles, split as well; some keys seen by nobody
         ("f32", 2, 4, 1, 256, 333, 333, 2, 100, (0, 0), True, True, "KP", "KP"),
         ("f32", 1, 24, 3, 64, 678, 678, 3, 0, (0, 0), True, False, "KP", "KP"),                   # 528 query tiles
         ("f32", 1, 2, 1, 64, 300, 300, 4, 0, (0, 0), False, True, "QKP", "P")]


def _profiled(call):
    st.st_profile_begin()
    try:
        call()
    finally:
        ran = set(st.st_profile_end())
    return ran


@pytest.mark.parametrize("c", CASES, ids=[f"{c[0]}_d{c[4]}_q{c[5]}_seg{c[9][0]}{'' if c[10] else '_full'}" for c in CASES])
def test_tiles_with_shares_of_their_own(c):
    dtype, B, Hq, Hkv, D, Sq, Sk, n, q0, (seg, q2), causal, split, flags, flags_less = c
    w = si.Workload("shares", 360 + Sq % 100, dtype, B, Hq, Hkv, D, Sq, Sk, n, q0, causal, True, q_seg=seg, q_offset2=q2)
    print(f"[shares] {c}", flush=True)
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    koffs = [w.k_offset(j) for j in range(n)]
    args = (w.q_where, koffs, causal, w.scale)
    order = list(range(n))
    pos = positions(w)
    o_r, lse_r = oa.attention_forward(inp.q, inp.k, inp.v, *pos, causal, w.scale)
    dq_r, dk_r, dv_r = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, *pos, causal, w.scale)
    full = [st.st_ring_workspace_bytes(q, ks, vs, *args, st.ST_RING_FUSED, back) for back in (False, True)]
    plans = Share(BF16 if dtype == "bf16" else F32, B, Hq, Hkv, D, Sq, Sk, koffs, q0, causal, seg, q2)
    up = lambda x: (x + 255) // 256 * 256
    ws = lambda size: torch.full((size + 256,), 0xff, dtype=torch.uint8, device="cuda")
    outs = []
    ran = _profiled(lambda: outs.extend(st.st_ring_fwd(q, ks, vs, *args, order, workspace=ws(full[0]))))
    o, lse, low = outs
    assert ("combine" in ran) == split, f"the forward of this share was meant to be {'split' if split else 'whole'}: {ran}"
    assert_close(host(o), o_r, dtype, "o")
    assert_close(host(lse), lse_r, dtype, "lse", lse=dtype == "bf16")
    assert torch.equal(low, o.to(low.dtype))

    def close(dk, dv, what=""):
        for j in range(n):
            if dtype == "f32":
                assert_close(host(dk[j]), dk_r[j], dtype, f"{what}dk[{j}]")
                assert_close(host(dv[j]), dv_r[j], dtype, f"{what}dv[{j}]")
            else:                                                          # hundreds of rows add into few keys
                assert_close_wide(host(dk[j]), dk_r[j], f"{what}dk[{j}]")
                assert_close_wide(host(dv[j]), dv_r[j], f"{what}dv[{j}]")

    def backward(call):
        dq = torch.full_like(o, 1 / 64)
        dk, dv = ([torch.zeros(k.shape, device="cuda") for k in ks] for _ in range(2))
        ran = _profiled(lambda: call(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv))
        return dq, dk, dv, ran

    got = []
    for size, want in ((full[1], flags), (plans.base + up(q.numel() * 4), flags_less), (plans.base, "P" if "P" in flags else "")):
        dq, dk, dv, ran = backward(lambda *a: st.st_ring_bwd(*a, workspace=ws(size)))
        assert ("add_parts" in ran, "add_kv_parts" in ran, "bwd_bf16" in ran or "bwd_f32" in ran) == tuple(x in want for x in "QKP"), \
            f"meant to be split as {want!r}: {ran}"
        assert plans.plan(order, FUSED, False, size + 256)[0][3] == ("O" in want)
        assert_close(host(dq) - 1 / 64, dq_r, dtype, "dq")                # the start costs 1e-9 per element
        close(dk, dv)
        got.append((dq, dk, dv))
    if dtype == "bf16":                                                    # assigned and rounded, hidden chunks too
        dq = torch.full_like(o, 1 / 64)
        dk, dv = ([torch.full(k.shape, float("nan"), device="cuda") for k in ks] for _ in range(2))
        lows = [[torch.empty_like(k) for k in ks] for _ in range(2)]
        st.st_ring_bwd_last(q, ks, vs, d_o, low, lse, *args, order, dq, dk, dv, assign=True, dk_lowp=lows[0], dv_lowp=lows[1], workspace=ws(full[1]))
        if not causal or koffs[-1] <= plans.last_position():               # with hidden chunks in the table the plan may be another one
            assert torch.equal(dq, got[0][0])
        assert_close(host(dq) - 1 / 64, dq_r, dtype, "dq")
        for j in range(n):
            assert torch.equal(dk[j].to(torch.bfloat16), lows[0][j]) and torch.equal(dv[j].to(torch.bfloat16), lows[1][j])
        close(dk, dv, "assigned ")
    dq, dk, dv, ran = backward(lambda *a: st.st_ring_bwd_noalloc(*a))
    assert torch.equal(dq, got[0][0])
    for x, y in zip(dk + dv, got[0][1] + got[0][2]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,Sq", [("bf16", 1500), ("f32", 1210)])
def test_states_a_tile_does_not_have_are_left_alone(dtype, Sq):
    """Tiles of a causal shard have unlike numbers of shares; the pass that folds them reads only those a tile has, so nothing is
    written in the place of the others."""
    B, Hq, Hkv, D = 1, 2, 1, 128 if dtype == "bf16" else 64
    w = si.Workload("shares", 361, dtype, B, Hq, Hkv, D, Sq, Sq, 1, 0, True, True)
    q, ks, vs, _ = upload(si.make_inputs(w))
    args = (q, ks, vs, 0, [0], True, w.scale)
    size = st.st_ring_workspace_bytes(*args, st.ST_RING_FUSED, False)
    up = lambda x: (x + 255) // 256 * 256
    o_bytes, state = up(q.numel() * 4), up(q.numel() * 4) + up(B * Hq * Sq * 4)
    buf = torch.full((size + 256,), 0xff, dtype=torch.uint8, device="cuda")
    st.st_ring_fwd(*args, [0], workspace=buf)
    at = -buf.data_ptr() % 256
    n = size // state
    assert n >= 3
    lse = [buf[at + y * state + o_bytes:at + y * state + o_bytes + 4 * B * Hq * Sq].view(torch.float32).view(B, Hq, Sq) for y in range(n)]
    written = [int((~x.isnan()).sum()) for x in lse]                    # rows of the tiles that have a share y
    assert written[0] > written[n - 1] and all(x >= y for x, y in zip(written, written[1:])), written
