"""GPU: float mode at any address: every tensor of a step's entry points shifted by one float from where it can be read
four values at a time gives the bits of the aligned call."""
import pytest

from tests.gpu_util import has_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

# widths that are multiples of 4, so that only the addresses decide; the second one takes 64 x 64 tiles
SIZES = [(5, 2, 36, 40, 70), (3, 1, 128, 256, 2500)]


class Bench:
    """Tensors by name, each at an address that is a multiple of 16 or one float further on."""

    def __init__(self, shifted):
        self.shifted = shifted

    def put(self, name, t):
        import torch
        shift = 1 if self.shifted in (name, "all") else 0
        buf = torch.full((t.numel() + 4,), float("nan"), device="cuda")
        v = buf[shift:shift + t.numel()].view(t.shape)
        v.copy_(t)
        return v

    def out(self, name, *shape):
        import torch
        return self.put(name, torch.zeros(shape, device="cuda"))


def _run(E, k, d, f, T, shifted):
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(E + d)
    S, n = T * k, lambda *s: torch.randn(s, generator=g)      # noqa: E731
    m = Bench(shifted)
    x, wr = m.put("x", n(T, d)), m.put("w_router", n(E, d))
    wgu, wd = m.put("w_gate_up", n(E, 2 * f, d) * 0.1), m.put("w_down", n(E, d, f) * 0.1)
    sh = U.Shape(T=T, d_model=d, d_ff=f, E=E, k=k, L=1, dtype=U.F32, sigma=0.9, c=2.0, eps=1e-6, alpha_pool=0.0, router=0)
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    idx, cnt, off = torch.empty((T, k), **i32), torch.empty(E, **i32), torch.empty(E + 1, **i32)
    ros, sor = torch.empty(S, **i32), torch.empty(S, **i32)
    z, gate, ps = m.out("logits", T, E), m.out("gate", T, k), m.out("psum", E)
    U.route(sh, x, wr, idx, gate, z, cnt, ps, ws)
    xp = m.out("x_perm", S, d)
    U.permute(sh, x, idx, cnt, xp, off, ros, sor, ws)
    a, b, h, y = m.out("a", S, f), m.out("b", S, f), m.out("h", S, f), m.out("y", S, d)
    U.expert_ffn_fwd(sh, xp, off, wgu, wd, a, b, h, y, ws)
    a2, b2, h2, y2 = m.out("a", S, f), m.out("b", S, f), m.out("h", S, f), m.out("y", S, d)
    U.expert_ffn_fwd_gather(sh, x, sor, off, wgu, wd, a2, b2, h2, y2, ws)
    dy = m.put("dy", n(S, d))
    dxp, dact = m.out("dx_perm", S, d), m.out("d_act", S, 2 * f)
    dwgu, dwd = m.put("d_w_gate_up", n(E, 2 * f, d)), m.put("d_w_down", n(E, d, f))
    U.expert_ffn_bwd(sh, dy, xp, a, b, h, off, wgu, wd, dxp, dact, dwgu, dwd, ws)
    # two layers in one reduction: this one, and one whose tensors are all aligned
    pairs = [(t, t.clone()) for t in (xp, dact, h, dy, off)]
    tabs = [torch.tensor([t.data_ptr() for t in p], dtype=torch.int64, device="cuda") for p in pairs]
    gwgu, gwd = m.out("d_w_gate_up", E, 2 * f, d), m.out("d_w_down", E, d, f)
    U.expert_wgrad(sh, 2, *tabs, gwgu, gwd, False, ws)
    dw, ds, dx = m.out("d_w_router", E, d), torch.empty(1, device="cuda"), m.put("dx", n(T, d))
    U.route_bwd(sh, x, wr, z, idx, m.put("dgate", n(T, k)), m.put("aux", n(E)), dw, ds, dx, True, ws)
    torch.cuda.synchronize()
    return [idx, z, gate, ps, xp, a, b, h, y, a2, b2, h2, y2, dxp, dact, dwgu, dwd, gwgu, gwd, dw, ds, dx]


NAMES = ["x", "w_router", "w_gate_up", "w_down", "logits", "x_perm", "a", "b", "h", "y", "dy", "dx_perm", "d_act",
         "d_w_gate_up", "d_w_down", "d_w_router", "dx", "all"]


@pytest.mark.parametrize("size", SIZES, ids=["E%d-k%d-d%d-f%d-T%d" % s for s in SIZES])
def test_shifted_tensors_keep_the_bits(size):
    import torch
    want = _run(*size, None)
    assert all(bool(torch.isfinite(t.float()).all()) for t in want)
    for name in NAMES:
        for i, (p, q) in enumerate(zip(_run(*size, name), want)):
            assert torch.equal(p, q), (name, i)
