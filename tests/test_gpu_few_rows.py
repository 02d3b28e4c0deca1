"""GPU: the expert FFN forward of calls with few rows per expert, at the edges of its forms: one and several row
fragments, more rows than one pass over the weights holds, split and whole reductions, reductions shorter than the
four parts, empty experts in front, between and at the end."""
import numpy as np
import pytest

from tests.gpu_util import TOL, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

# name: (T, k, d, f, rows of every expert; they add up to T k)
CASES = {
    "one-token-one-step": (1, 1, 64, 64, [0, 1, 0]),                       # a reduction of one step, four parts
    "fragment-edges": (16, 3, 192, 320, [16, 0, 15, 1, 16]),
    "repeated-selections": (16, 8, 128, 192, [0, 100, 28] + [0] * 5),                # more rows than tokens: several passes
    "two-fragments": (64, 2, 448, 64, [17] * 4 + [32, 0, 28] + [0] * 9),
    "three-passes": (64, 4, 128, 256, [65, 0, 33] + [2] * 79),
    "whole-reductions": (64, 8, 256, 192, [1] * 300 + [0] * 5 + [33, 40, 64, 31, 32, 12] + [0] * 201),
    "pool-of-512": (48, 8, 1024, 704, [1, 0] * 192 + [2] * 64 + [0] * 63 + [64]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_few_rows(name):
    import torch
    import paper_2605_06665_amd as U
    T, k, d, f, counts = CASES[name]
    E, S = len(counts), T * k
    assert sum(counts) == S and E <= 512
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    g = torch.Generator().manual_seed(E + T)
    x = torch.randn((T, d), generator=g).to(torch.bfloat16)
    wgu = (torch.randn((E, 2 * f, d), generator=g) * d ** -0.5).to(torch.bfloat16)
    wd = (torch.randn((E, d, f), generator=g) * f ** -0.5).to(torch.bfloat16)
    slots = torch.randperm(S, generator=g).to(torch.int32)
    xp = x[(slots // k).long()].contiguous()
    sh = U.Shape(T=T, d_model=d, d_ff=f, E=E, k=k, L=1, dtype=U.BF16, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0,
                 router=0)
    ws = torch.empty(U.workspace_bytes(sh), dtype=torch.uint8, device="cuda:0")
    goff, gslots, gwgu, gwd = torch.from_numpy(off).cuda(), slots.cuda(), wgu.cuda(), wd.cuda()
    runs = []
    for gather in (False, True):
        # a row more than there are: it has to stay as it is
        a, b, h = (torch.full((S + 1, f), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
        y = torch.full((S + 1, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        if gather:
            U.expert_ffn_fwd_gather(sh, x.cuda(), gslots, goff, gwgu, gwd, a, b, h, y, ws)
        else:
            U.expert_ffn_fwd(sh, xp.cuda(), goff, gwgu, gwd, a, b, h, y, ws)
        runs.append([host(t) for t in (a, b, h, y)])
    a, b, h = (torch.full((S + 1, f), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
    U.expert_ffn_recompute(sh, xp.cuda(), goff, gwgu, a, b, h, ws)
    for i, t in enumerate((a, b, h)):
        assert np.array_equal(host(t), runs[0][i], equal_nan=True)
    for m, n in zip(*runs):
        assert np.array_equal(m, n, equal_nan=True) and np.isnan(m[S]).all() and np.isfinite(m[:S]).all()
    ga, gb, gh, gy = (r[:S] for r in runs[0])
    for e, n in enumerate(counts):
        if n == 0:
            continue
        r = slice(int(off[e]), int(off[e + 1]))
        z = xp[r].double().numpy() @ wgu[e].double().numpy().T
        ra, rb = z[:, :f], z[:, f:]
        rh = ra / (1 + np.exp(-ra)) * rb
        ry = gh[r].astype(np.float64) @ wd[e].double().numpy().T
        for got, want in ((ga, ra), (gb, rb), (gh, rh), (gy, ry)):
            assert rel_err(got[r], want) <= TOL["bf16"], (name, e)
