"""Forward workspaces that are missing, short or off the 256-byte boundary, through the C entry point: shares that can do
without one run on fewer workgroups, small shares and tables of more than 64 chunks take the least they have always asked
for and refuse less.  Every accepted call against the fp64 oracle."""
import ctypes as C

import pytest
import torch

import paper_2407_00611_amd as st
import synth_inputs as si
from oracle import attention as oa
from paper_2407_00611_amd import api
from util import assert_close, host, positions, upload

pytestmark = pytest.mark.gpu


class Share:
    def __init__(self, dtype, Hq, D, Sq, Sk, n):
        self.w = w = si.Workload("workspace", 350, dtype, 1, Hq, 1, D, Sq, Sk, n, 0, False, False)
        inp = si.make_inputs(w)
        self.q, self.ks, self.vs, _ = upload(inp)
        self.koffs = [w.k_offset(j) for j in range(n)]
        self.ref = oa.attention_forward(inp.q, inp.k, inp.v, *positions(w), w.causal, w.scale)
        up = lambda x: (x + 255) // 256 * 256
        self.state = up(self.q.numel() * 4) + up(Hq * Sq * 4)          # one partial O and lse
        self.full = st.st_ring_workspace_bytes(self.q, self.ks, self.vs, 0, self.koffs, False, w.scale, st.ST_RING_FUSED, False)
        self.buf = torch.full((self.full + 1024,), 0xff, dtype=torch.uint8, device="cuda")      # NaN as floats

    def run(self, offset, nbytes):
        """Status of the fused forward with `nbytes` of workspace, `offset` bytes beyond a boundary (None: no workspace);
        the result is checked where there is one."""
        w, q = self.w, self.q
        r = api._Ring(q, self.ks, self.vs, 0, self.koffs, False, w.scale)
        o = torch.full(q.shape, float("nan"), device="cuda")
        lse = torch.full((w.B, w.Hq, w.Sq), float("nan"), device="cuda")
        p = None if offset is None else (self.buf.data_ptr() + 255) // 256 * 256 + offset
        assert p is None or p + nbytes <= self.buf.data_ptr() + self.buf.numel()
        tq = api._view(q)
        got = api._lib.st_ring_fwd(C.byref(r.desc), C.byref(tq), api._i32_array(list(range(w.n_chunks))), None, w.n_chunks,
                                   st.ST_RING_FUSED, api._ptr(o), api._ptr(lse), None, C.c_void_p(p), nbytes, api._stream(None))
        torch.cuda.synchronize()
        if got == 0:
            assert_close(host(o), self.ref[0], w.dtype, "o")
            assert_close(host(lse), self.ref[1], w.dtype, "lse", lse=True)
        return got


#        dtype, Hq, D, Sq, Sk, n
FREE = [("f32", 2, 128, 64, 512, 4), ("bf16", 2, 128, 256, 640, 1), ("bf16", 16, 64, 2100, 320, 2), ("f32", 1, 64, 40, 33, 2)]


@pytest.mark.parametrize("c", FREE, ids=[f"{c[0]}_q{c[3]}_n{c[5]}" for c in FREE])
def test_shares_that_can_do_without(c):
    s = Share(*c)
    assert s.run(None, 0) == 0
    assert s.run(0, s.full) == 0
    assert s.run(16, s.full) == 0
    for states in (1, 2, 3):
        assert s.run(0, min(states * s.state + 128, s.full)) == 0


#         dtype, Hq, D, Sq, Sk, n, states asked for
LEAST = [("bf16", 2, 128, 300, 640, 2, 3), ("bf16", 4, 64, 512, 704, 2, 3), ("f32", 1, 128, 40, 64, 70, 1),
         ("bf16", 1, 128, 200, 64, 66, 1)]


@pytest.mark.parametrize("c", LEAST, ids=[f"{c[0]}_q{c[3]}_n{c[5]}" for c in LEAST])
def test_shares_that_ask_for_some(c):
    s = Share(*c[:6])
    least = c[6] * s.state
    assert s.full > least, "this share was meant to be given more by the present plan"
    assert s.run(None, 0) == 5 and s.run(0, least - 1) == 5 and s.run(16, s.full) == 3
    assert s.run(0, least) == 0 and s.run(0, s.full) == 0
