"""GPU: accumulated weight gradients on both sides of the size from which they are streamed past the caches: experts
without rows are added until the gradients are larger, and the others keep their bits."""
import pytest

from tests.gpu_util import TOL, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

D, F, K, T = 512, 1024, 2, 150


@pytest.mark.parametrize("aligned", [True, False])
def test_both_sides_of_the_line(aligned):
    import torch
    import paper_2605_06665_amd as U
    few = (160 << 20) // (12 * D * F)               # 12 bytes of gradient per weight pair of an expert: 160 MiB at most
    g = torch.Generator().manual_seed(3)
    S = T * K
    counts = torch.bincount(torch.randint(0, few - 1, (S,), generator=g), minlength=few)    # the last one empty as well
    off = torch.cat([torch.zeros(1, dtype=torch.long), counts.cumsum(0)]).to(torch.int32)

    def rows(n):
        return torch.randn((S, n), generator=g).to(torch.bfloat16).cuda()

    dy, xp, a, b, h = rows(D), rows(D), rows(F), rows(F), rows(F)
    old = torch.randn((few, 3 * F * D), generator=g).cuda()
    got = []
    for E in (few, few + 2):
        sh = U.Shape(T=T, d_model=D, d_ff=F, E=E, k=K, L=1, dtype=U.BF16, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0, router=0)
        assert bool(U.tile_forms(sh) & U.binding.WGRAD_STREAMED) == (E > few)
        offsets = torch.cat([off, off[-1:].repeat(E - few)]).cuda()
        wgu, wd = (torch.zeros(n, dtype=torch.bfloat16, device="cuda") for n in ((E, 2 * F, D), (E, D, F)))
        pad = 0 if aligned else 1                    # the other form of the stores
        buf = [torch.full((E * n + pad,), 7.0, device="cuda") for n in (2 * F * D, F * D)]
        dgu, dd = buf[0][pad:].view(E, 2 * F, D), buf[1][pad:].view(E, D, F)
        dgu[:few] = old[:, :2 * F * D].view(few, 2 * F, D)
        dd[:few] = old[:, 2 * F * D:].view(few, D, F)
        dx, dact = (torch.empty((S, n), dtype=torch.bfloat16, device="cuda") for n in (D, 2 * F))
        ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
        U.expert_ffn_bwd(sh, dy, xp, a, b, h, offsets, wgu, wd, dx, dact, dgu, dd, ws)
        assert bool((dgu[few:] == 7.0).all()) and bool((dd[few:] == 7.0).all())
        got.append((dgu[:few].clone(), dd[:few].clone()))
    for p, q in zip(*got):
        assert torch.equal(p, q)
    e = int(counts.argmax())
    r = slice(int(off[e]), int(off[e + 1]))
    want = old[e, 2 * F * D:].double().view(D, F) + dy[r].double().T @ h[r].double()
    assert rel_err(host(got[0][1][e]), host(want)) <= TOL["f32"]     # bfloat16 operands, float sums of a few dozen terms
    empty = few - 1
    assert torch.equal(got[0][0][empty].flatten(), old[empty, :2 * F * D])
