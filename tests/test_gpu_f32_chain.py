"""GPU: float sums are the index-order chain of fused multiply-adds, bit for bit, whatever the tile: logits of float mode
and of bfloat16 pools that are not a multiple of 8 (whose products the float kernel takes)."""
import numpy as np
import pytest

from tests.gpu_util import has_gpu, host

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _chain(x, w):
    """acc = fma(x_i, w_i, acc) in float32, i ascending.  In 64-bit mantissas a product of two floats is exact and the
    sum is off by 2^-40 of a float's last place at most, so the one rounding to float is the chain's."""
    x, w = x.astype(np.longdouble), w.astype(np.longdouble)
    acc = np.zeros((x.shape[0], w.shape[0]), dtype=np.float32)
    for i in range(x.shape[1]):
        acc = (x[:, i:i + 1] * w[:, i] + acc.astype(np.longdouble)).astype(np.float32)
    return acc


# 32 x 32 tiles with whole and ragged reductions, 64 x 64 tiles; vector and value-by-value loads
@pytest.mark.parametrize("dtype,T,E,d", [("f32", 33, 5, 70), ("f32", 129, 40, 36), ("f32", 4100, 252, 44), ("f32", 4100, 250, 41),
                                         ("bf16", 33, 5, 64), ("bf16", 129, 90, 128), ("bf16", 4100, 250, 64)])
def test_logits_are_the_chain(dtype, T, E, d):
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(T + E + d)
    act = torch.float32 if dtype == "f32" else torch.bfloat16
    x, w = (torch.randn(s, generator=g).to(act).cuda() for s in ((T, d), (E, d)))
    sh = U.Shape(T=T, d_model=d, d_ff=64, E=E, k=1, L=1, dtype=U.F32 if dtype == "f32" else U.BF16, sigma=0.9, c=2.0, eps=1e-6,
                 alpha_pool=0.0, router=0)
    i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(device="cuda")
    z = torch.full((T, E), float("nan"), **f32)
    ws = torch.empty(U.workspace_bytes(sh), dtype=torch.uint8, device="cuda")
    U.route(sh, x, w, torch.empty((T, 1), **i32), torch.empty((T, 1), **f32), z, torch.empty(E, **i32), torch.empty(E, **f32), ws)
    assert np.array_equal(host(z), _chain(host(x), host(w)))
