"""GPU: the sum over the router gradient's partial products, four values at a time where the output is aligned to 16
bytes, one otherwise: numbers of parts on both sides of a group of eight, bitwise the same result from both forms."""
import numpy as np
import pytest

from tests.gpu_util import TOL, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("T", [1, 255, 2048, 2049, 2400, 16384])
def test_both_forms(T):
    import torch
    import paper_2605_06665_amd as U
    E, d, k = 40, 192, 2
    g = torch.Generator().manual_seed(T)
    x = torch.randn((T, d), generator=g).to(torch.bfloat16).cuda()
    wr = torch.randn((E, d), generator=g).to(torch.bfloat16).cuda()
    sh = U.Shape(T=T, d_model=d, d_ff=64, E=E, k=k, L=1, dtype=U.BF16, sigma=0.9, c=2.0, eps=1e-6, alpha_pool=0.0, router=0)
    i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(device="cuda")
    idx, gate, z = torch.empty((T, k), **i32), torch.empty((T, k), **f32), torch.empty((T, E), **f32)
    cnt, ps = torch.empty(E, **i32), torch.empty(E, **f32)
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    U.route(sh, x, wr, idx, gate, z, cnt, ps, ws)
    dgate = torch.randn((T, k), generator=g).cuda()
    outs = []
    for shift in (0, 1):
        buf = torch.full((E * d + 2,), float("nan"), **f32)
        dw, ds = buf[shift:shift + E * d].view(E, d), torch.full((1,), float("nan"), **f32)
        dx = torch.zeros((T, d), dtype=torch.bfloat16, device="cuda")
        U.route_bwd(sh, x, wr, z, idx, dgate, torch.zeros(E, **f32), dw, ds, dx, False, ws)
        outs.append((host(dw), host(ds), host(dx)))
        assert np.isnan(host(buf[shift + E * d:])).all() and np.isnan(host(buf[:shift])).all()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    # d_sigma and dW in double from the same logits: s = sigma c relu(z) / (|z| + eps)
    zd = z.double().cpu()
    n = zd.norm(dim=1, keepdim=True)
    ds_ = torch.zeros_like(zd).scatter_(1, idx.long().cpu(), dgate.double().cpu())
    zh = zd / (n + 1e-6)
    dzh = ds_ * 0.9 * 2.0 * (zh > 0)
    dz = dzh / (n + 1e-6) - zd * (dzh * zd).sum(1, keepdim=True) / ((n + 1e-6) ** 2 * n)
    assert rel_err(outs[0][0], (dz.T @ x.double().cpu()).numpy()) <= TOL["bf16"]
    want = float((ds_ * 2.0 * zh.clamp_min(0)).sum())
    # T k float terms of about unit size, summed in a tree
    assert abs(float(outs[0][1][0]) - want) <= 1e-5 * float((ds_.abs() * 2.0 * zh.clamp_min(0)).sum()) + 1e-6
