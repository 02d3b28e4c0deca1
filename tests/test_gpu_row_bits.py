"""GPU: a token's bits do not depend on how many tokens share the call: logits, selection, gates and expert outputs of the
forms for a few tokens and rows, against a call of many tokens, which takes the tile kernels."""
import pytest

from tests.gpu_util import has_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

MANY = 600


def _shape(T, E, d, f, k, router=0):
    import paper_2605_06665_amd as U
    return U.Shape(T=T, d_model=d, d_ff=f, E=E, k=k, L=1, dtype=U.BF16, sigma=0.9, c=2.0, eps=1e-6, alpha_pool=0.0,
                   router=router)


@pytest.mark.parametrize("E,k,d", [(8, 1, 64), (64, 2, 256), (192, 2, 1536), (264, 3, 448), (512, 8, 1024)])
@pytest.mark.parametrize("router", [0, 1])
def test_router(E, k, d, router):
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(E + d)
    x = torch.randn((MANY, d), generator=g).to(torch.bfloat16).cuda()
    w = (torch.randn((E, d), generator=g) * d ** -0.5).to(torch.bfloat16).cuda()

    def run(T):
        sh = _shape(T, E, d, 64, k, router)
        idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
        gate, z = torch.full((T, k), float("nan"), device="cuda"), torch.full((T, E), float("nan"), device="cuda")
        cnt, ps = torch.empty(E, dtype=torch.int32, device="cuda"), torch.empty(E, device="cuda")
        ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
        U.route(sh, x[:T], w, idx, gate, z, cnt, ps, ws)
        return idx, gate, z

    many = run(MANY)
    for T in (1, 15, 16, 17, 33, 64, 65, 128, 129):
        for few, whole in zip(run(T), many):
            assert torch.equal(few, whole[:T]), T


# one wavefront per workgroup with 4, 8, 12 or 16 steps in flight, with half of the registers, four wavefronts per
# workgroup; reductions that do not come out even; a pool larger than the caches
@pytest.mark.parametrize("E,d,f,k", [(8, 64, 64, 1), (64, 512, 1024, 2), (24, 768, 768, 2), (48, 832, 1472, 3),
                                     (64, 1536, 704, 2), (200, 320, 1088, 8)])
def test_experts(E, d, f, k):
    import numpy as np
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(E + d)
    x = torch.randn((MANY, d), generator=g).to(torch.bfloat16).cuda()
    wgu = torch.empty((E, 2 * f, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, d ** -0.5)
    wd = torch.empty((E, d, f), dtype=torch.bfloat16, device="cuda").normal_(0.0, f ** -0.5)
    # a fifth of the experts takes half of the slots
    rng = np.random.default_rng(E)
    bias = np.where(np.arange(E) < E // 5, 1.5, 0.0)
    idx = np.argsort(-(bias + rng.gumbel(size=(MANY, E))), axis=1)[:, :k]

    def run(T):
        sh = _shape(T, E, d, f, k)
        picks = idx[:T].reshape(-1)
        order = np.argsort(picks, kind="stable").astype(np.int32)
        off = np.concatenate([[0], np.cumsum(np.bincount(picks, minlength=E))]).astype(np.int32)
        a, b, h = (torch.full((T * k, f), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3))
        y = torch.full((T * k, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
        U.expert_ffn_fwd_gather(sh, x, torch.from_numpy(order).cuda(), torch.from_numpy(off).cuda(), wgu, wd, a, b, h, y, ws)
        out = []
        for t in (a, b, h, y):                      # rows in slot order
            s = torch.empty_like(t)
            s[torch.from_numpy(order).long().cuda()] = t
            out.append(s)
        return out

    many = run(MANY)
    assert all(bool(torch.isfinite(t).all()) for t in many)
    for T in (1, 2, 5, 16, 17, 40, 64):
        for few, whole in zip(run(T), many):
            assert torch.equal(few, whole[:T * k]), T
