"""GPU: router and dispatch of a few tokens, at the edges of their forms: one and several token fragments, pools of
both lane widths, selection in one workgroup and in several, one-chunk and several-chunk index maps with and without
a copy, rows of 16 bytes and of odd words, in float and bfloat16."""
import numpy as np
import pytest

from oracle import unipool_oracle as O
from synth import workloads as W
from tests.gpu_util import TOL, check_selection, dev, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

CASES = [
    # (E, k, d_model, T, dtype)
    (8, 1, 64, 1, "bf16"), (8, 8, 64, 16, "bf16"), (24, 2, 192, 17, "bf16"), (192, 2, 1536, 4, "bf16"),
    (256, 8, 128, 16, "bf16"), (264, 3, 448, 5, "bf16"), (264, 8, 128, 33, "bf16"), (512, 8, 1024, 48, "bf16"),
    (512, 1, 64, 64, "bf16"), (512, 8, 128, 64, "bf16"), (392, 4, 320, 31, "bf16"), (64, 4, 128, 64, "bf16"),
    (90, 3, 64, 64, "bf16"), (16, 2, 64, 128, "bf16"), (200, 5, 128, 128, "bf16"),
    (8, 2, 64, 128, "f32"), (5, 3, 37, 65, "f32"), (300, 8, 30, 129, "f32"), (512, 4, 24, 255, "f32"),
    (40, 1, 33, 256, "f32"),
    (512, 1, 64, 72, "bf16"), (512, 1, 64, 73, "bf16"), (288, 2, 64, 128, "f32"), (296, 2, 64, 128, "f32"),
    (512, 2, 128, 63, "bf16"),
]


@pytest.mark.parametrize("router", ["norm", "softmax"])
@pytest.mark.parametrize("E,k,d,T,dtype", CASES, ids=["%s-E%d-k%d-d%d-T%d" % (c[4], *c[:4]) for c in CASES])
def test_route_and_permute(E, k, d, T, dtype, router):
    import torch
    import paper_2605_06665_amd as U
    w = W.Workload("few-tokens", L=1, E=E, d=d, f=64, k=k, T=T, dtype=dtype, seed=2000 + E + k + d + T, c=2.4)
    sh = U.Shape(T=T, d_model=d, d_ff=64, E=E, k=k, L=1, dtype=U.BF16 if dtype == "bf16" else U.F32, sigma=0.9, c=w.c,
                 eps=w.eps, alpha_pool=w.alpha, router=U.ROUTER_SOFTMAX if router == "softmax" else U.ROUTER_NORM)
    x, wr = W.gen_x(w, 0), W.gen_w_router(w, 0)
    ref = O.route(x, wr, k, 0.9, w.c, w.eps, router=router)
    xd, wd = dev(x, dtype), dev(wr, dtype)
    i32 = dict(dtype=torch.int32, device="cuda")
    idx = torch.full((T, k), -1, **i32)
    gate = torch.full((T, k), float("nan"), device="cuda")
    logits = torch.full((T, E), float("nan"), device="cuda")
    counts = torch.full((E,), -1, **i32)
    psum = torch.full((E,), float("nan"), device="cuda")
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    U.route(sh, xd, wd, idx, gate, logits, counts, psum, ws)
    tol = TOL[dtype]
    assert rel_err(host(logits), ref["z"]) <= tol
    gi = host(idx)
    check_selection(ref["z"], ref["idx"], gi, k, scores=ref["s"], got_gate=host(gate), tol=tol)
    assert np.array_equal(host(counts), np.bincount(gi.ravel(), minlength=E))
    assert rel_err(host(psum), ref["psum"]) <= tol
    # rows in the order of (expert, token): a stable sort of the slots by expert
    order = np.argsort(gi.ravel(), kind="stable")
    rows = np.empty(T * k, dtype=np.int64)
    rows[order] = np.arange(T * k)
    for copy in (False, True):
        ws.fill_(0xff)
        off, ros, sor = (torch.full((n,), -1, **i32) for n in (E + 1, T * k, T * k))
        xp = torch.full((T * k, d), float("nan"), dtype=xd.dtype, device="cuda")
        U.permute(sh, xd if copy else None, idx, counts, xp if copy else None, off, ros, sor, ws)
        assert np.array_equal(host(off), np.concatenate([[0], np.cumsum(host(counts))]))
        assert np.array_equal(host(ros), rows) and np.array_equal(host(sor), order)
        if copy:
            assert np.array_equal(host(xp), host(xd)[order // k])
