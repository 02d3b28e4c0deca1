"""GPU: weight gradients of step() with wgrad="layer", which takes several layers into one accumulation, against
begin_backward and backward_layer, which add layer by layer: one layer, some of them, uneven groups and all at once."""
import pytest

from tests.gpu_util import has_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


# E = 16, d = f = 64: a quarter of the gradients is 196608 bytes, a pair of buffers T k 192 values
@pytest.mark.parametrize("dtype,T,L,recompute,per", [("bf16", 1000, 3, False, 1), ("bf16", 150, 5, False, 2),
                                                     ("bf16", 150, 5, True, 2), ("bf16", 30, 4, False, 4),
                                                     ("bf16", 20, 11, False, 6), ("f32", 80, 5, False, 2)])
def test_groups(dtype, T, L, recompute, per):
    import torch
    import paper_2605_06665_amd as U
    from paper_2605_06665_amd.pipeline import PoolStep
    E, d, f, k = 16, 64, 64, 2
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(T)

    def rnd(*shape, std=1.0):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=g).to(act)

    xs, wrs, gs = ([rnd(*s) for _ in range(L)] for s in ((T, d), (E, d), (T, d)))
    wgu, wd = rnd(E, 2 * f, d, std=0.1), rnd(E, d, f, std=0.1)
    sig = [1.0] * L
    ps = PoolStep(T, d, f, E, k, L, U.BF16 if dtype == "bf16" else U.F32, 2.6, 1e-6, 0.01, device="cuda:0", wgrad="layer",
                  recompute=recompute)
    assert len(ps._dy) == per
    ps.step(xs, wrs, sig, wgu, wd, gs)                       # leaves the forward pass's state of every layer
    ps.begin_backward()
    for l in reversed(range(L)):
        ps.backward_layer(l, xs[l], wrs[l], sig[l], wgu, wd, gs[l])
    want = [t.clone() for t in (ps.d_w_gate_up, ps.d_w_down, *(st.dx for st in ps.layers))]
    for t in (ps.d_w_gate_up, ps.d_w_down, *ps._dy, *ps._dact):
        t.fill_(float("nan"))                                # nothing of an earlier step is read
    ps.step(xs, wrs, sig, wgu, wd, gs)
    got = (ps.d_w_gate_up, ps.d_w_down, *(st.dx for st in ps.layers))
    for a, b in zip(got[2:], want[2:]):
        assert torch.equal(a, b)
    for a, b in zip(got[:2], want[:2]):
        # the same products in another order of float sums: about sqrt(n) 2^-24 of terms of the size of the result; n up to
        # T L, a few hundred per expert
        assert (a - b).norm() <= 2e-6 * b.norm() and torch.isfinite(a).all()
