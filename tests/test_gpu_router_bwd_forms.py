"""GPU: the sum over the router gradient's partial products, four values at a time where the output is aligned to 16
bytes, one otherwise: numbers of parts on both sides of a group of eight, bitwise the same result from both forms.
dx of the router added to what is there: the sum is rounded once.  Operands of pools that are not a multiple of 8 at
addresses that are not a multiple of 16."""
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


def _route_bwd_inputs(T, E, d, k, seed):
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((T, d), generator=g).to(torch.bfloat16).cuda()
    wr = torch.randn((E, d), generator=g).to(torch.bfloat16).cuda()
    sh = U.Shape(T=T, d_model=d, d_ff=64, E=E, k=k, L=1, dtype=U.BF16, sigma=0.9, c=2.0, eps=1e-6, alpha_pool=0.0, router=0)
    z = x.float() @ wr.float().T
    idx = torch.topk(z, k, dim=1).indices.to(torch.int32).contiguous()
    dgate = torch.randn((T, k), generator=g).cuda()
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    # dz as the library defines it, rounded to bfloat16
    zd = z.double()
    n = zd.norm(dim=1, keepdim=True)
    ds = torch.zeros_like(zd).scatter_(1, idx.long(), dgate.double())
    dzh = ds * 0.9 * 2.0 * (zd > 0)
    dz = dzh / (n + 1e-6) - zd * (dzh * zd).sum(1, keepdim=True) / ((n + 1e-6) ** 2 * n)
    return sh, x, wr, z.contiguous(), idx, dgate, ws, dz.to(torch.bfloat16).double()


@pytest.mark.parametrize("E,d,T", [(90, 192, 777), (3, 64, 33), (8, 320, 129), (64, 192, 300), (96, 832, 2049)])
def test_accumulated_dx_is_rounded_once(E, d, T):
    """dx starts as minus the rounded product, so what is left is the product's own rounding error: a product that is
    rounded before the addition leaves zeros."""
    import torch
    import paper_2605_06665_amd as U
    sh, x, wr, z, idx, dgate, ws, dz = _route_bwd_inputs(T, E, d, 2, E + T)
    f32 = dict(device="cuda")
    dw, ds = torch.empty((E, d), **f32), torch.empty(1, **f32)
    dx = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    U.route_bwd(sh, x, wr, z, idx, dgate, None, dw, ds, dx, False, ws)
    product = dz @ wr.double()
    rounded = dx.clone()
    dx.neg_()
    U.route_bwd(sh, x, wr, z, idx, dgate, None, dw, ds, dx, True, ws)
    left = product - rounded.double()
    # float sums of at most 96 terms: 1e-5 of the product is ample; half of it more for the rounding of what is left.
    # dz is computed in float by the library, so a few of its values round the other way (about 5e-4 of them, times E
    # of a row): rows with one are off by a share of the product, all others are not
    bad = (dx.double() - left).abs() > 2e-5 * product.abs().amax(dim=1, keepdim=True) + 2.0 ** -8 * left.abs()
    assert float(left.abs().max()) > 0
    assert float(bad.any(dim=1).double().mean()) <= 0.2
    assert float((dx == 0).double().mean()) <= 0.5


@pytest.mark.parametrize("E,d,T", [(90, 192, 33), (3, 64, 256), (13, 128, 257), (90, 192, 2049)])
@pytest.mark.parametrize("shifted", ["x", "w_router", "dx", "all"])
def test_odd_pools_take_any_alignment(E, d, T, shifted):
    import torch
    import paper_2605_06665_amd as U
    sh, x, wr, z, idx, dgate, ws, dz = _route_bwd_inputs(T, E, d, 2, E + T)
    dx0 = torch.randn((T, d), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()

    def place(name, t):
        if shifted not in (name, "all"):
            return t.clone(), None
        buf = torch.full((t.numel() + 2,), float("nan"), dtype=t.dtype, device="cuda")
        v = buf[1:-1].view(t.shape)
        v.copy_(t)
        return v, buf

    px, pw, (pdx, around) = place("x", x)[0], place("w_router", wr)[0], place("dx", dx0)
    dw, ds = torch.full((E, d), float("nan"), device="cuda"), torch.full((1,), float("nan"), device="cuda")
    U.route_bwd(sh, px, pw, z, idx, dgate, None, dw, ds, pdx, True, ws)
    # float sums, and a few values of dz that round the other way (2^-8 of one term)
    assert rel_err(host(dw), host(dz.T @ x.double())) <= 1e-3
    want = dx0.double() + dz @ wr.double()
    assert float((pdx.double() - want).norm() / want.norm()) <= 1.02 * float((want.to(torch.bfloat16).double() - want).norm() / want.norm())
    assert bool(torch.isfinite(ds).all())
    if around is not None:
        assert bool(torch.isnan(around[0])) and bool(torch.isnan(around[-1]))


@pytest.mark.parametrize("E,T,k,d", [(1, 300, 1, 64), (3, 1000, 2, 64), (4, 1000, 2, 192), (5, 17, 1, 128), (32, 400, 2, 320),
                                     (40, 129, 3, 64), (128, 400, 2, 192), (136, 70, 2, 320), (256, 15, 1, 64),
                                     (257, 300, 3, 64), (264, 33, 8, 192), (512, 9, 8, 128), (512, 700, 8, 192),
                                     (200, 17000, 1, 64),
                                     # 2048, 2049 and 4125 partial sums of d_sigma: whole and cut rounds of its loads
                                     (8, 32768, 1, 64), (8, 32784, 1, 64), (264, 33000, 1, 64)])
@pytest.mark.parametrize("router", [0, 1])
def test_blocks_of_tokens(E, T, k, d, router):
    """Blocks of 8, 16 and 64 tokens with ends inside them, logits and dx in tiles of 128 x 128 and 128 x 256 whose rows
    and columns end inside a tile, chunks of 128 and 256 tokens: logits, d_sigma, router gradient and dx in double."""
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(E + T)
    x = torch.randn((T, d), generator=g).to(torch.bfloat16).cuda()
    wr = (torch.randn((E, d), generator=g) * (1.0 if router == 0 else d ** -0.5)).to(torch.bfloat16).cuda()
    sh = U.Shape(T=T, d_model=d, d_ff=64, E=E, k=k, L=1, dtype=U.BF16, sigma=0.9, c=2.0, eps=1e-6, alpha_pool=0.0, router=router)
    i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(device="cuda")
    idx, gate, z = torch.empty((T, k), **i32), torch.empty((T, k), **f32), torch.full((T + 1, E), float("nan"), **f32)
    cnt, ps = torch.empty(E, **i32), torch.empty(E, **f32)
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    U.route(sh, x, wr, idx, gate, z, cnt, ps, ws)
    assert torch.isnan(z[T]).all()
    xd, wd = x.double().cpu(), wr.double().cpu()
    assert rel_err(host(z[:T]), (xd @ wd.T).numpy()) <= 1e-5
    dgate, coef = torch.randn((T, k), generator=g), torch.randn(E, generator=g) * 0.1
    dw, dsg = torch.full((E, d), float("nan"), **f32), torch.full((1,), float("nan"), **f32)
    dx = torch.full((T + 1, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    U.route_bwd(sh, x, wr, z, idx, dgate.cuda(), coef.cuda(), dw, dsg, dx, False, ws)
    assert torch.isnan(dx[T].float()).all()
    zd = z[:T].double().cpu()
    ds = coef.double().expand(T, E).clone().scatter_add_(1, idx.long().cpu(), dgate.double())
    if router == 0:
        n = zd.norm(dim=1, keepdim=True)
        s = 2.0 * (zd / (n + 1e-6)).clamp_min(0)
        dzh = ds * 0.9 * 2.0 * (zd > 0)
        dz = dzh / (n + 1e-6) - zd * (dzh * zd).sum(1, keepdim=True) / ((n + 1e-6) ** 2 * n)
        # at most T E float terms, summed in a tree of wavefronts and blocks
        assert abs(float(dsg) - float((ds * s).sum())) <= 1e-5 * float((ds * s).abs().sum()) + 1e-6
    else:
        p = torch.softmax(zd, 1)
        dz = p * (ds - (ds * p).sum(1, keepdim=True))
        assert float(dsg) == 0.0
    # (one expert: dz cancels to rounding noise of its terms)
    if E > 1:
        assert rel_err(host(dw), (dz.T @ xd).numpy()) <= TOL["bf16"] and rel_err(host(dx[:T]), (dz @ wd).numpy()) <= TOL["bf16"]
    else:
        assert np.isfinite(host(dw)).all() and np.isfinite(host(dx[:T])).all()


@pytest.mark.parametrize("T", [130816, 130817, 131072])
@pytest.mark.parametrize("accumulate", [False, True])
def test_dx_of_many_tokens_of_a_large_pool(T, accumulate):
    """Both sides of the line from which dx goes in tiles of 256 x 256 (eight rounds of them on 256 compute units: 512 row tiles of
    d_model 1024), the last one of a single row or full: sampled rows in double, and the bits of the first tokens alone, in tiles of 128 x 128."""
    import torch
    import paper_2605_06665_amd as U
    E, d = 448, 1024
    sh, x, wr, z, idx, dgate, ws, dz = _route_bwd_inputs(T, E, d, 2, 7)
    f32 = dict(device="cuda")
    dw, ds = torch.empty((E, d), **f32), torch.empty(1, **f32)
    dx = torch.full((T + 1, d), 0.5 if accumulate else float("nan"), dtype=torch.bfloat16, device="cuda")
    U.route_bwd(sh, x, wr, z, idx, dgate, None, dw, ds, dx, accumulate, ws)
    assert bool((dx[T] == 0.5).all() if accumulate else torch.isnan(dx[T]).all())
    few = 1000
    sh2 = U.Shape(T=few, d_model=d, d_ff=64, E=E, k=2, L=1, dtype=U.BF16, sigma=0.9, c=2.0, eps=1e-6, alpha_pool=0.0, router=0)
    dx2 = torch.full((few, d), 0.5, dtype=torch.bfloat16, device="cuda")
    U.route_bwd(sh2, x[:few], wr, z[:few], idx[:few], dgate[:few], None, dw, ds, dx2, accumulate, ws)
    assert torch.equal(dx[:few], dx2)
    rows = torch.tensor([0, 127, 128, 255, 256, 65535, T - 257, T - 256, T - 255, T - 1], device="cuda")
    want = dz[rows] @ wr.double() + (0.5 if accumulate else 0.0)
    assert rel_err(host(dx[rows]), host(want)) <= TOL["bf16"]
