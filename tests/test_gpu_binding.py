"""The native half of the wrapper takes plain tensors, lists and numbers and leaves every other accepted form to the ctypes
half: both make the same call (results bit for bit), and what was refused stays refused with the same error."""
import numpy as np
import pytest
import torch

import paper_2407_00611_amd as st
import synth_inputs as si
from paper_2407_00611_amd import api
from util import upload

pytestmark = pytest.mark.gpu


class Watched:
    """the native half, and what it answered: a status, or None where it left the call to ctypes"""
    NAMES = {"ring_fwd", "ring_bwd", "block_fwd", "block_bwd", "merge", "combine", "delta", "cast"}

    def __init__(self, half):
        self.half, self.took, self.left = half, set(), set()

    def __getattr__(self, name):
        def call(*args):
            status = getattr(self.half, name)(*args)
            (self.left if status is None else self.took).add(name)
            return status
        return call


class Wrapped(torch.Tensor):
    """a subclass: the native half does not look into it"""


def _share(dtype="bf16"):
    w = si.Workload("binding", 371, dtype, 2, 4, 2, 64, 200, 100, 3, 0, True, True, q_seg=100, q_offset2=200)
    q, ks, vs, d_o = upload(si.make_inputs(w))
    return w, q, ks, vs, d_o


def _run(w, q, ks, vs, d_o, offsets, where, scale, causal, order, stream=None):
    shape, kv = tuple(q.shape), tuple(ks[0].shape)
    o, lse, low = torch.empty(shape, device="cuda"), torch.empty((w.B, w.Hq, w.Sq), device="cuda"), torch.empty(shape, dtype=d_o.dtype, device="cuda")
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    st.st_ring_fwd(q, ks, vs, where, offsets, causal, scale, order, [0] * len(order), o_acc=o, lse=lse, o_lowp=low, workspace=ws, stream=stream)
    out = [o, lse, low]
    for way in ("add", "last", "noalloc"):
        dq = torch.zeros(shape, device="cuda")
        dk, dv = ([torch.zeros(kv, device="cuda") for _ in ks] for _ in range(2))
        args = (q, ks, vs, d_o, low, lse, where, offsets, causal, scale, order, dq, dk, dv)
        if way == "add":
            st.st_ring_bwd(*args, workspace=ws, stream=stream)
        elif way == "noalloc":
            st.st_ring_bwd_noalloc(*args, stream=stream)
        else:
            lk, lv = ([torch.empty(kv, dtype=d_o.dtype, device="cuda"), None, torch.empty(kv, dtype=d_o.dtype, device="cuda")] for _ in range(2))
            st.st_ring_bwd_last(*args, assign=True, dk_lowp=lk, dv_lowp=lv, workspace=ws, stream=stream)
            out += [x for x in lk + lv if x is not None]
        out += [dq] + dk + dv
    part, pl = torch.empty_like(o), torch.empty_like(lse)
    st.st_attn_block_fwd(q, ks[1], vs[1], where, offsets[1], causal, scale, part, pl, stream=stream)
    acc, al = o.clone(), lse.clone()
    st.st_attn_merge(acc, al, part, pl, st.ST_BF16, low.clone(), stream=stream)
    delta = st.st_attn_delta(d_o, low, torch.empty_like(lse), stream=stream)
    dq, dk, dv = torch.zeros_like(o), torch.zeros(kv, device="cuda"), torch.zeros(kv, device="cuda")
    st.st_attn_block_bwd(q, ks[1], vs[1], d_o, lse, delta, where, offsets[1], causal, scale, dq, dk, dv, workspace=ws, stream=stream)
    both, bl = torch.empty_like(o[:, :50]).contiguous(), torch.empty((w.B, w.Hq, 50), device="cuda")
    st.st_attn_combine([o, part], [lse, pl], 20, 50, st.ST_F32, both, bl, stream=stream)
    torch.cuda.synchronize()
    return out + [part, pl, acc, al, delta, dq, dk, dv, both, bl, st.st_cast_from_f32(dq, st.ST_BF16, torch.empty_like(low), stream=stream)]


def test_both_halves_make_the_same_call(monkeypatch):
    w, q, ks, vs, d_o = _share()
    offsets, order = [w.k_offset(j) for j in range(3)], [2, 0, 1]
    watched = lambda: monkeypatch.setattr(api, "_binding", Watched(native)) or api._binding
    native = api._binding
    seen = watched()
    plain = _run(w, q, ks, vs, d_o, offsets, w.q_where, w.scale, True, order)
    assert seen.took == Watched.NAMES and not seen.left, "plain arguments go the short way"
    uses_q = {"ring_fwd", "ring_bwd", "block_fwd", "block_bwd"}
    # the calls that each form leaves to ctypes
    forms = {"tuples and a parameter": (set(), (torch.nn.Parameter(q), tuple(ks), tuple(vs), d_o, tuple(offsets), tuple(w.q_where), w.scale, True, tuple(order))),
             "numpy numbers, a list, an int": (uses_q, (q, ks, vs, d_o, list(np.array(offsets)), list(w.q_where), np.float64(w.scale), 1, list(np.array(order)))),
             "a subclass": (uses_q | {"delta"}, (q.as_subclass(Wrapped), ks, vs, d_o.as_subclass(Wrapped), offsets, w.q_where, w.scale, True, order))}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for name, (left, form) in forms.items():
        for stream in (None, side, side.cuda_stream):
            print(f"[binding] {name}", flush=True)
            seen = watched()
            with torch.cuda.stream(side if stream is not None else torch.cuda.current_stream()):      # tensors are made there too
                got = _run(w, *form, stream=stream)
            left_now = Watched.NAMES if isinstance(stream, int) else left          # a bare handle is ctypes' as well
            assert seen.left == left_now and seen.took == Watched.NAMES - left_now, name
            for x, y in zip(plain, got):
                assert torch.equal(x, y), name

    class Declines:
        def __getattr__(self, _):
            return lambda *a: None
    monkeypatch.setattr(api, "_binding", Declines())
    for x, y in zip(plain, _run(w, q, ks, vs, d_o, offsets, w.q_where, w.scale, True, order)):
        assert torch.equal(x, y)


def test_what_is_refused():
    w, q, ks, vs, d_o = _share()
    offsets, order = [w.k_offset(j) for j in range(3)], [0, 1, 2]
    o, lse, low = torch.empty(q.shape, device="cuda"), torch.empty((w.B, w.Hq, w.Sq), device="cuda"), torch.empty_like(q)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    fwd = lambda ks=ks, vs=vs, o=o, lse=lse, order=order, q=q, where=w.q_where: st.st_ring_fwd(
        q, ks, vs, where, offsets, True, w.scale, order, o_acc=o, lse=lse, o_lowp=low, workspace=ws)
    with pytest.raises(ValueError, match="one K, one V"):
        fwd(ks=ks[:2])
    with pytest.raises(ValueError, match="share shape"):
        fwd(vs=vs[:2] + [vs[2][:, :50]])
    with pytest.raises(ValueError, match="o_acc"):
        fwd(o=o[:, :100])
    with pytest.raises(ValueError, match="lse"):
        fwd(lse=lse.double())
    with pytest.raises(ValueError, match="D dimension"):
        fwd(q=q.transpose(1, 3).contiguous().transpose(1, 3))
    with pytest.raises(TypeError):
        fwd(q=q.half(), ks=[k.half() for k in ks], vs=[v.half() for v in vs])
    for bad in ([0, 0, 1], [0, 1, 3]):
        with pytest.raises(st.StarTrailError) as e:
            fwd(order=bad)
        assert e.value.status == 1 and "st_ring_fwd" in str(e.value)
    with pytest.raises(st.StarTrailError):
        fwd(where=(100, 100, 0))                     # the second run before the first
    with pytest.raises(ValueError):
        st.st_cast_from_f32(o, st.ST_BF16, low[:, :100])


def test_a_tensor_whose_memory_may_not_be_touched_raises():
    """Its accessors throw inside the native half, which is called through C: the error reaches Python as one."""
    w, q, ks, vs, d_o = _share()
    src, dst = torch.ones(64, device="cuda"), torch.zeros(64, dtype=torch.bfloat16, device="cuda")
    barred = torch.ones(64, device="cuda")
    torch._C._set_throw_on_mutable_data_ptr(barred)
    with pytest.raises(RuntimeError, match="data pointer"):
        st.st_cast_from_f32(barred, st.ST_BF16, dst)
    k = ks[1].clone()
    torch._C._set_throw_on_mutable_data_ptr(k)
    o, lse, low = torch.empty(q.shape, device="cuda"), torch.empty((w.B, w.Hq, w.Sq), device="cuda"), torch.empty_like(q)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    with pytest.raises(RuntimeError, match="data pointer"):
        st.st_ring_fwd(q, [ks[0], k, ks[2]], vs, w.q_where, [w.k_offset(j) for j in range(3)], True, w.scale, [0, 1, 2], o_acc=o, lse=lse,
                       o_lowp=low, workspace=ws)
    st.st_cast_from_f32(src, st.ST_BF16, dst)           # and the library goes on
    assert float(dst.float().sum()) == 64
