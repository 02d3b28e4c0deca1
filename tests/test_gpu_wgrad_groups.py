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
    ps.step(xs, wrs, sig, wgu, wd, gs)                       # leaves the forward pass's state of every layer
    assert len(ps._dy) == per
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


def _small_step(dev="cuda:0", **kw):
    import torch
    import paper_2605_06665_amd as U
    from paper_2605_06665_amd.pipeline import PoolStep
    T, L, E, d, f, k = 30, 4, 16, 64, 64, 2
    g = torch.Generator().manual_seed(T)

    def rnd(*shape, std=1.0):
        return (torch.randn(shape, generator=g) * std).to(torch.bfloat16).to(dev)

    args = ([rnd(T, d) for _ in range(L)], [rnd(E, d) for _ in range(L)], [1.0] * L, rnd(E, 2 * f, d, std=0.1),
            rnd(E, d, f, std=0.1), [rnd(T, d) for _ in range(L)])
    return PoolStep(T, d, f, E, k, L, U.BF16, 2.6, 1e-6, 0.01, device=dev, wgrad="layer", **kw), args


def _gradients(ps, args):
    ps.step(*args)
    return [t.clone() for t in (ps.d_w_gate_up, ps.d_w_down)]


def _agree(a, b):
    return all((p - q).norm() <= 2e-6 * q.norm() for p, q in zip(a, b))           # as above


def test_the_caller_says_how_many_layers(monkeypatch):
    """Buffers of further layers are made by the first step() and not by a caller's own loop over the layers; wgrad_layers
    sets their number; without memory for them, and in a recording that is the first step, layers go one by one."""
    import torch
    ps, args = _small_step()
    for l in range(4):
        ps.forward_layer(l, args[0][l], args[1][l], 1.0, args[3], args[4])
    ps.aux_loss()
    ps.begin_backward()
    for l in reversed(range(4)):
        ps.backward_layer(l, args[0][l], args[1][l], 1.0, args[3], args[4], args[5][l])
    ps.end_backward()
    want = [t.clone() for t in (ps.d_w_gate_up, ps.d_w_down)]
    assert len(ps._dy) == len(ps._dact) == 1
    assert _agree(_gradients(ps, args), want) and len(ps._dy) == 4
    for n in (1, 3, 9):
        ps, args = _small_step(wgrad_layers=n)
        assert _agree(_gradients(ps, args), want) and len(ps._dy) == min(n, 4)
    ps, args = _small_step()

    def no_memory(per):
        raise torch.OutOfMemoryError("none left")

    monkeypatch.setattr(ps, "_take_layers", no_memory)
    assert _agree(_gradients(ps, args), want) and len(ps._dy) == 1
    # the kernels have run, this object has not
    ps, args = _small_step()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        ps.step(*args)
    assert len(ps._dy) == 1
    assert _agree(_gradients(ps, args), want) and len(ps._dy) == 4       # an eager step makes them, the recording keeps its own
    for _ in range(3):
        ps.d_w_gate_up.fill_(float("nan"))
        ps.d_w_down.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert _agree((ps.d_w_gate_up, ps.d_w_down), want)
        assert _agree(_gradients(ps, args), want)
