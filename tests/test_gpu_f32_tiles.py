"""fp32 kernels at the edges of their 32 x 32 tiles and of the padded head sizes, against the fp64 oracle: one row
more or less than a tile, every padded size with and without zero-filled columns, shards in two runs, more tiles than
wavefronts, forwards split over workgroups, and values that are no numbers behind a mask.  Tolerance: the fp32
bounds of assert_close (1e-5 relative; sums of at most 1300 terms, each rounded at 6e-8)."""
import numpy as np
import pytest
import torch

import paper_2407_00611_amd as st
import synth_inputs as si
from oracle import attention as oa
from util import assert_close, host, positions, upload

pytestmark = pytest.mark.gpu

#        D,  Hq, Hkv, Sq, Sk, n, q_offset, causal, (q_seg, q_offset2)
CASES = [(8, 1, 1, 1, 31, 2, 40, True, (0, 0)),
         (32, 2, 1, 33, 32, 2, 31, True, (0, 0)),
         (40, 2, 2, 31, 33, 1, 0, False, (0, 0)),
         (96, 3, 1, 64, 65, 3, 131, True, (0, 0)),
         (104, 1, 1, 65, 96, 2, 0, False, (0, 0)),
         (128, 4, 2, 70, 64, 4, 32, True, (35, 186)),
         (136, 1, 1, 34, 66, 2, 98, True, (0, 0)),
         (256, 2, 1, 40, 90, 2, 20, True, (9, 140)),
         (64, 2, 1, 64, 640, 2, 1216, True, (0, 0))]


def _share(w, mode=st.ST_RING_FUSED):
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    koffs = [w.k_offset(j) for j in range(w.n_chunks)]
    order = list(range(w.n_chunks))
    o, lse, _ = st.st_ring_fwd(q, ks, vs, w.q_where, koffs, w.causal, w.scale, order, None, mode)
    dq = torch.zeros_like(o)
    dk = [torch.zeros_like(k) for k in ks]
    dv = [torch.zeros_like(k) for k in ks]
    st.st_ring_bwd(q, ks, vs, d_o, o, lse, w.q_where, koffs, w.causal, w.scale, order, dq, dk, dv, mode)
    return inp, (o, lse, dq, dk, dv)


@pytest.mark.parametrize("c", CASES, ids=[f"d{c[0]}_q{c[3]}_k{c[4]}" for c in CASES])
def test_share_at_tile_edges(c):
    D, Hq, Hkv, Sq, Sk, n, q0, causal, (seg, q2) = c
    w = si.Workload("f32_tiles", 300 + D, "f32", 1, Hq, Hkv, D, Sq, Sk, n, q0, causal, True, q_seg=seg, q_offset2=q2)
    print(f"[f32 tiles] {c}", flush=True)
    inp, (o, lse, dq, dk, dv) = _share(w)
    q_pos, k_pos = positions(w)
    o_r, lse_r = oa.attention_forward(inp.q, inp.k, inp.v, q_pos, k_pos, causal, w.scale)
    dq_r, dk_r, dv_r = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, q_pos, k_pos, causal, w.scale)
    assert_close(host(o), o_r, "f32", "o")
    assert_close(host(lse), lse_r, "f32", "lse")
    assert_close(host(dq), dq_r, "f32", "dq")
    for j in range(n):
        assert_close(host(dk[j]), dk_r[j], "f32", f"dk[{j}]")
        assert_close(host(dv[j]), dv_r[j], "f32", f"dv[{j}]")


def test_split_forward_and_a_workspace_too_small_for_it():
    """A few query tiles against long chunks: the fused forward splits the table over workgroups when the workspace
    has room for their states, and walks it in one launch when there is none."""
    w = si.Workload("f32_split", 310, "f32", 1, 2, 2, 128, 64, 512, 4, 3 * 512, True, True)
    inp = si.make_inputs(w)
    q, ks, vs, _ = upload(inp)
    args = (q, ks, vs, w.q_where, [w.k_offset(j) for j in range(4)], True, w.scale)
    one = (q.numel() + w.Hq * w.Sq) * 4
    assert st.st_ring_workspace_bytes(*args, st.ST_RING_FUSED, False) >= 2 * one
    q_pos, k_pos = positions(w)
    o_r, lse_r = oa.attention_forward(inp.q, inp.k, inp.v, q_pos, k_pos, True, w.scale)
    for ws in (None, torch.empty(256, dtype=torch.uint8, device="cuda")):
        st.st_profile_begin()
        o, lse, low = st.st_ring_fwd(*args, list(range(4)), workspace=ws)
        assert ("combine" in st.st_profile_end()) == (ws is None)
        assert_close(host(o), o_r, "f32", "o")
        assert_close(host(lse), lse_r, "f32", "lse")
        assert torch.equal(o, low)


#           D,  Sq, Sk, n, q_offset, causal, shares
FWD_SPLIT = [(128, 64, 512, 4, 4 * 512 - 64, True, 8), # eight turns, four chunks
             (128, 100, 1024, 1, 924, True, 4),        # one chunk
             (64, 33, 1000, 2, 0, False, 8),           # turns that reach over two chunks, ragged last tiles
             (256, 40, 300, 3, 860, True, 8)]          # four wavefronts per workgroup


@pytest.mark.parametrize("c", FWD_SPLIT, ids=[f"d{c[0]}_q{c[1]}_k{c[2]}" for c in FWD_SPLIT])
def test_every_share_of_a_split_forward_has_work(c):
    """The plan counts turns of tiles and the launch hands them out: no partial state is empty, whatever the number of
    chunks, and an infinity behind a mask edge reaches exactly the rows that see it, whichever share met it."""
    D, Sq, Sk, n, q0, causal, shares = c
    w = si.Workload("f32_shares", 313, "f32", 1, 2, 1, D, Sq, Sk, n, q0, causal, False)
    inp = si.make_inputs(w)
    q, ks, vs, _ = upload(inp)
    args = (q0, [w.k_offset(j) for j in range(n)], causal, w.scale)
    up = lambda x: (x + 255) // 256 * 256
    b_o, b_l = up(q.numel() * 4), up(w.Hq * Sq * 4)
    need = st.st_ring_workspace_bytes(q, ks, vs, *args, st.ST_RING_FUSED, False)
    assert need == shares * (b_o + b_l)
    ws = torch.full((need + 256,), 0xff, dtype=torch.uint8, device="cuda")                   # NaN
    o, lse, _ = st.st_ring_fwd(q, ks, vs, *args, list(range(n)), workspace=ws)
    o_r, lse_r = oa.attention_forward(inp.q, inp.k, inp.v, *positions(w), causal, w.scale)
    assert_close(host(o), o_r, "f32", "o")
    assert_close(host(lse), lse_r, "f32", "lse")
    first = (-ws.data_ptr()) % 256
    for y in range(shares):
        at = first + y * (b_o + b_l) + b_o
        part = ws[at:at + w.Hq * Sq * 4].view(torch.float32)
        assert torch.isfinite(part).any(), f"share {y} met no key"
    if not causal:
        return
    bad = q0 + Sq // 2                                  # the position of a query row in the middle
    v2 = [v.clone() for v in vs]
    v2[bad // Sk][:, bad % Sk, :, 3] = float("inf")
    v2[(bad + 1) // Sk][:, (bad + 1) % Sk, :, 4] = float("nan")
    o2, lse2, _ = st.st_ring_fwd(q, ks, v2, *args, list(range(n)))
    i = bad - q0
    assert torch.equal(lse, lse2) and torch.equal(o[:, :i], o2[:, :i])
    assert torch.isposinf(o2[:, i:, :, 3]).all() and torch.isnan(o2[:, i + 1:, :, 4]).all()
    keep = [d for d in range(D) if d not in (3, 4)]
    assert torch.equal(o[..., keep], o2[..., keep]) and torch.equal(o[:, i, :, 4], o2[:, i, :, 4])


def test_values_that_are_no_numbers_stay_behind_the_mask():
    """Rows that a causal mask hides from a query (or queries it hides from a key) may hold anything: the results of
    every row that does not see them are the ones without them, bit for bit; a row that sees one is no number."""
    w = si.Workload("f32_nan", 311, "f32", 1, 2, 1, 72, 70, 70, 1, 0, True, True)
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    bad = 45                                            # a key, and the query row at the same position
    q2, k2, v2, d2 = q.clone(), ks[0].clone(), vs[0].clone(), d_o.clone()
    v2[:, bad, :, 3] = float("inf")
    v2[:, bad, :, 70] = float("nan")

    def run(q, k, v, d_o):
        o, lse, _ = st.st_ring_fwd(q, [k], [v], 0, [0], True, w.scale, [0])
        dq = torch.zeros_like(o)
        dk, dv = torch.zeros_like(k), torch.zeros_like(v)
        st.st_ring_bwd(q, [k], [v], d_o, clean_o, clean_lse, 0, [0], True, w.scale, [0], dq, [dk], [dv])
        return o, lse, dq, dk, dv

    clean_o, clean_lse, _ = st.st_ring_fwd(q, ks, vs, 0, [0], True, w.scale, [0])
    ref = run(q, ks[0], vs[0], d_o)
    o, lse, dq, _, _ = run(q, ks[0], v2, d_o)
    assert torch.equal(o[:, :bad], ref[0][:, :bad]) and torch.equal(lse, ref[1]) and torch.equal(dq[:, :bad], ref[2][:, :bad])
    assert torch.isposinf(o[:, bad:, :, 3]).all() and torch.isnan(o[:, bad:, :, 70]).all()
    keep = [d for d in range(72) if d not in (3, 70)]
    assert torch.equal(o[..., keep], ref[0][..., keep])
    k2[:, bad, :, 5] = float("nan")
    _, _, dq, _, _ = run(q, k2, vs[0], d_o)
    assert torch.equal(dq[:, :bad], ref[2][:, :bad]) and torch.isnan(dq[:, bad:]).all()
    # a query row reaches the keys up to its own position only
    q2[:, bad, :, 0] = float("nan")
    _, _, _, dk, dv = run(q2, ks[0], vs[0], d_o)
    assert torch.equal(dk[:, bad + 1:], ref[3][:, bad + 1:]) and torch.equal(dv[:, bad + 1:], ref[4][:, bad + 1:])
    assert torch.isnan(dk[:, :bad + 1]).all() and torch.isnan(dv[:, :bad + 1]).all()
    d2[:, bad, :, 9] = float("inf")
    _, _, _, dk, dv = run(q, ks[0], vs[0], d2)
    assert torch.equal(dk[:, bad + 1:], ref[3][:, bad + 1:]) and torch.equal(dv[:, bad + 1:], ref[4][:, bad + 1:])
    assert torch.isposinf(dv[:, :bad + 1, :, 9]).all()


@pytest.mark.parametrize("D", [32, 64, 88, 128, 136, 192, 256])
def test_no_numbers_behind_the_mask_in_every_block_of_columns(D):
    """A lane owns blocks of neighbouring columns, as many as the padded head size has multiples of 32: an infinity in any of them
    reaches the rows that see it, once, and no other column."""
    w = si.Workload("f32_cols", 313, "f32", 1, 1, 1, D, 40, 40, 1, 0, True, True)
    q, ks, vs, d_o = upload(si.make_inputs(w))
    bad, cols = 21, sorted({c for b in range(0, D, 16) for c in (b, b + 7, min(b + 13, D - 1)) if c < D})
    rest = [d for d in range(D) if d not in cols]
    v2, d2 = vs[0].clone(), d_o.clone()
    v2[:, bad, :, cols] = float("inf")
    d2[:, bad, :, cols] = float("-inf")
    o, lse, _ = st.st_ring_fwd(q, ks, vs, 0, [0], True, w.scale, [0])
    o2, _, low = st.st_ring_fwd(q, ks, [v2], 0, [0], True, w.scale, [0])
    assert torch.equal(o2[:, :bad], o[:, :bad]) and torch.equal(o2[..., rest], o[..., rest]) and torch.equal(low, o2)
    assert torch.isposinf(o2[:, bad:][..., cols]).all()
    out = []
    for x in (d_o, d2):
        g = [torch.zeros_like(o), torch.zeros_like(ks[0]), torch.zeros_like(vs[0])]
        st.st_ring_bwd(q, ks, vs, x, o, lse, 0, [0], True, w.scale, [0], g[0], [g[1]], [g[2]])
        out.append(g[2])
    assert torch.equal(out[0][:, bad + 1:], out[1][:, bad + 1:]) and torch.equal(out[0][..., rest], out[1][..., rest])
    assert torch.isneginf(out[1][:, :bad + 1][..., cols]).all()


@pytest.mark.parametrize("D,Sq,Sk", [(72, 45, 70), (128, 33, 33), (256, 63, 40), (64, 1, 1)])
def test_infinities_in_the_last_row_of_a_ragged_tile(D, Sq, Sk):
    """Every query sees the last key and every key the last query; rows that a ragged tile lacks must not multiply what they
    hold by zero: an infinity arrives as one, and the other columns are what they are without it, bit for bit."""
    w = si.Workload("f32_inf", 312, "f32", 1, 2, 1, D, Sq, Sk, 2, 0, False, True)
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    koffs = [w.k_offset(j) for j in range(2)]
    args = (0, koffs, False, w.scale, [0, 1])
    v2, d2 = [v.clone() for v in vs], d_o.clone()
    v2[0][:, -1, :, 3], v2[1][:, -1, :, D - 1] = float("inf"), float("-inf")
    d2[:, -1, :, 5] = float("inf")
    o, lse, _ = st.st_ring_fwd(q, ks, vs, *args)
    o2, lse2, _ = st.st_ring_fwd(q, ks, v2, *args)
    assert torch.isposinf(o2[..., 3]).all() and torch.isneginf(o2[..., D - 1]).all() and torch.equal(lse, lse2)
    keep = [d for d in range(D) if d not in (3, D - 1)]
    assert torch.equal(o[..., keep], o2[..., keep])
    dvs = []
    for x in (d_o, d2):
        dq, dk, dv = torch.zeros_like(o), [torch.zeros_like(k) for k in ks], [torch.zeros_like(v) for v in vs]
        st.st_ring_bwd(q, ks, vs, x, o, lse, *args, dq, dk, dv)
        dvs.append(dv)
    keep = [d for d in range(D) if d != 5]
    for a, b in zip(*dvs):
        assert torch.isposinf(b[..., 5]).all() and torch.equal(a[..., keep], b[..., keep])


#           D,  Sq,  Sk, n, q_offset, causal, (q_seg, q_offset2)
DQ_SPLIT = [(128, 64, 300, 4, 3 * 300, True, (0, 0)),       # a few query tiles against long chunks
            (64, 33, 1000, 1, 0, True, (0, 0)),             # one chunk; all but its first turn is hidden
            (40, 65, 520, 2, 100, True, (33, 900)),         # two runs of query rows
            (256, 31, 260, 3, 0, False, (0, 0)),            # four wavefronts per workgroup, ragged last tiles
            (96, 40, 700, 2, 20, True, (0, 0))]             # a chunk whose first rows see nothing of it


@pytest.mark.parametrize("c", DQ_SPLIT, ids=[f"d{c[0]}_q{c[1]}_k{c[2]}" for c in DQ_SPLIT])
def test_split_dq_and_a_workspace_without_room_for_it(c):
    """An under-filled dQ launch is split over the keys when the workspace has room for the partial sums, and not
    otherwise; both add to what dq holds, and st_ring_bwd_noalloc adds up as the split launch does."""
    D, Sq, Sk, n, q0, causal, (seg, q2) = c
    w = si.Workload("f32_dq_split", 320 + D, "f32", 1, 2, 1, D, Sq, Sk, n, q0, causal, True, q_seg=seg, q_offset2=q2)
    print(f"[f32 dq split] {c}", flush=True)
    inp = si.make_inputs(w)
    q, ks, vs, d_o = upload(inp)
    koffs, order = [w.k_offset(j) for j in range(n)], list(range(n))
    args = (q, ks, vs, w.q_where, koffs, causal, w.scale)
    o, lse, _ = st.st_ring_fwd(*args, order)
    q_pos, k_pos = positions(w)
    dq_r, _, _ = oa.attention_backward(inp.q, inp.k, inp.v, inp.d_o, q_pos, k_pos, causal, w.scale)
    full = st.st_ring_workspace_bytes(*args, st.ST_RING_FUSED, True)
    base = (w.Hq * Sq * 4 + 255) // 256 * 256 + 1024          # Delta and the counters, without partial sums
    assert full - base >= q.numel() * 4, "this share was meant to split"

    def run(workspace=None):
        dq = torch.full_like(o, 1 / 64)
        grads = (dq, [torch.zeros_like(k) for k in ks], [torch.zeros_like(v) for v in vs])
        if workspace is None:
            st.st_ring_bwd_noalloc(q, ks, vs, d_o, o, lse, *args[3:], order, *grads)
        else:
            st.st_ring_bwd(q, ks, vs, d_o, o, lse, *args[3:], order, *grads, workspace=workspace)
        return dq

    one = (q.numel() * 4 + 255) // 256 * 256                  # room for one partial sum: the first share adds to dq itself
    split, two, whole = (run(torch.full((n,), 0xff, dtype=torch.uint8, device="cuda")) for n in (full, base + one, base))   # 0xff..: NaN
    for dq in (split, two, whole):
        assert_close(host(dq) - 1 / 64, dq_r, "f32", "dq")    # the start costs 1e-9 per element
    assert torch.equal(run(), split)


def test_backward_of_more_key_tiles_than_one_grid_dimension_takes():
    """4.2 million key tiles of two heads: more workgroups than the 2^32 threads of one dimension of a grid hold.  Only the first
    64 keys are seen, the results are those of a chunk of these 64, bit for bit, and nothing else is written."""
    Sk, Sq, H, D = 32 * ((1 << 22) + 5), 40, 2, 8
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 35 GB of device memory")
    gen = torch.Generator(device="cuda").manual_seed(91)
    rand = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    q, d_o = rand(1, Sq, H, D), rand(1, Sq, H, D)
    k, v, dk, dv = (torch.empty((1, Sk, H, D), device="cuda") for _ in range(4))
    for t in (k, v):
        t[:, :64] = rand(1, 64, H, D)
    o, lse = st.st_attn_block_fwd(q, k[:, :64], v[:, :64], 0, 0, True, 0.3)
    delta = st.st_attn_delta(d_o, o)
    got = []
    for n in (64, Sk):
        dq = torch.zeros_like(q)
        g = [dk, dv] if n == Sk else [torch.empty((1, n, H, D), device="cuda") for _ in range(2)]
        for x in g:
            x[:, :64] = 0.0
            x[:, -1] = 7.0 if n == Sk else 0.0
        st.st_attn_block_bwd(q, k[:, :n], v[:, :n], d_o, lse, delta, 0, 0, True, 0.3, dq, *g)
        got.append([dq] + [x[:, :64].clone() for x in g])
    assert float(dk[:, -1].min()) == float(dv[:, -1].max()) == 7.0
    for name, x, y in zip(("dq", "dk", "dv"), *got):
        same, live = torch.equal(x, y), bool(x.abs().max() > 0)
        assert live and same, name
