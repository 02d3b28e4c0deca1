"""GPU: float products over pools of any size (the search for a row tile by wavefronts up to 64 experts and by the workgroup
beyond, the list of tiles cut into eight parts, one tile and less than eight), widths that are a multiple of four and not, and weight gradients over
layers of which one is not aligned to 16 bytes."""
import numpy as np
import pytest

from tests.gpu_util import TOL, dev, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("E,d,f,rows", [(1, 20, 12, [5]), (3, 64, 68, [0, 1, 130]), (7, 33, 40, [64, 0, 65, 3, 0, 32, 31]),
                                        (64, 24, 21, [i % 5 for i in range(64)]), (65, 36, 32, [0] * 64 + [70]),
                                        (130, 16, 20, [(7 * i) % 67 for i in range(130)]),
                                        (511, 12, 8, [i % 3 for i in range(511)]),
                                        (512, 8, 16, [33] + [0] * 509 + [1, 66]), (66, 20, 12, [1] + [0] * 64 + [129]),
                                        (12, 252, 500, [40 + 9 * i for i in range(12)])])
@pytest.mark.parametrize("shift", [0, 1])
def test_products(E, d, f, rows, shift):
    import torch
    import paper_2605_06665_amd as U
    rng = np.random.default_rng(E)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    S = int(off[-1])
    x, dy = rng.standard_normal((S, d)), rng.standard_normal((S, d))
    wgu, wd = rng.standard_normal((E, 2 * f, d)) * d ** -0.5, rng.standard_normal((E, d, f)) * f ** -0.5
    sh = U.Shape(T=S, d_model=d, d_ff=f, E=E, k=1, L=1, dtype=U.F32, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0, router=0)
    ws = torch.empty(U.workspace_bytes(sh), dtype=torch.uint8, device="cuda:0")

    def f32(a):
        return dev(a.astype(np.float32), "f32")

    gx, gdy, gwgu, gwd, goff = f32(x), f32(dy), f32(wgu), f32(wd), dev(off)
    a, b, h = (torch.full((S, f), float("nan"), device="cuda:0") for _ in range(3))
    y, dx = (torch.full((S, d), float("nan"), device="cuda:0") for _ in range(2))
    dact = torch.full((S, 2 * f), float("nan"), device="cuda:0")
    U.expert_ffn_fwd(sh, gx, goff, gwgu, gwd, a, b, h, y, ws)
    U.expert_ffn_bwd(sh, gdy, gx, a, b, h, goff, gwgu, gwd, dx, dact, None, None, ws)
    # two layers with the same rows, the second one's tensors `shift` floats further on

    def moved(t):
        buf = torch.empty(t.numel() + shift, device="cuda:0")
        buf[shift:].copy_(t.flatten())
        return buf[shift:]

    second = [moved(t) for t in (gx, dact, h, gdy)]
    tabs = [torch.tensor([p.data_ptr(), q.data_ptr()], dtype=torch.int64, device="cuda:0")
            for p, q in zip((gx, dact, h, gdy), second)]
    toff = torch.tensor([goff.data_ptr()] * 2, dtype=torch.int64, device="cuda:0")
    dwgu, dwd = torch.full((E, 2 * f, d), float("nan"), device="cuda:0"), torch.full((E, d, f), float("nan"), device="cuda:0")
    U.expert_wgrad(sh, 2, *tabs, toff, dwgu, dwd, False, ws)
    gx, gdy, a, b, h, y, dx, dact, dwgu, dwd = (host(t).astype(np.float64) for t in
                                                (gx, gdy, a, b, h, y, dx, dact, dwgu, dwd))
    for e in range(E):
        r = slice(int(off[e]), int(off[e + 1]))
        want_gu, want_d = 2 * dact[r].T @ gx[r], 2 * gdy[r].T @ h[r]
        assert rel_err(dwgu[e], want_gu) <= TOL["f32"] and rel_err(dwd[e], want_d) <= TOL["f32"], e
        if rows[e] == 0:
            continue
        z = x[r] @ wgu[e].T
        sg = 1 / (1 + np.exp(-a[r]))
        dh = dy[r] @ wd[e]
        want = np.concatenate([dh * b[r] * sg * (1 + a[r] * (1 - sg)), dh * a[r] * sg], axis=1)
        for got, w in ((a[r], z[:, :f]), (b[r], z[:, f:]), (y[r], h[r] @ wd[e].T), (dact[r], want), (dx[r], dact[r] @ wgu[e])):
            assert rel_err(got, w) <= TOL["f32"], e


def test_weight_gradients_of_skewed_pools_use_the_whole_card():
    """As many rows take about as long whether they are spread evenly or half of them are with the first six experts of 32 (4500
    rows, 320 x 640, two layers: 137 and 139 us; 332 against 155 where the experts were cut into eight parts in order)."""
    import torch
    import paper_2605_06665_amd as U
    E, d, f, S, L = 32, 320, 640, 4500, 2
    sh = U.Shape(T=S, d_model=d, d_ff=f, E=E, k=1, L=L, dtype=U.F32, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0, router=0)
    ws = torch.empty(U.workspace_bytes(sh), dtype=torch.uint8, device="cuda:0")
    x, dy, h, dact = (torch.randn((S, n), device="cuda:0") for n in (d, d, f, 2 * f))
    dwgu, dwd = torch.empty((E, 2 * f, d), device="cuda:0"), torch.empty((E, d, f), device="cuda:0")

    def best_time(rows):
        off = torch.from_numpy(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)).cuda()
        tabs = [torch.tensor([t.data_ptr()] * L, dtype=torch.int64, device="cuda:0") for t in (x, dact, h, dy, off)]
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                U.expert_wgrad(sh, L, *tabs, dwgu, dwd, False, ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    even = [S // E + (i < S % E) for i in range(E)]
    skewed = [375] * 6 + [86] * 25 + [100]
    assert sum(skewed) == S
    assert best_time(skewed) <= 1.5 * best_time(even)
