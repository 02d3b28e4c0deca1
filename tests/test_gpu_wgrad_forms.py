"""GPU: weight gradients of the experts in all forms: tiles of 128 x 128 and 256 x 256, both gradients in one launch and
in two, written and added, over layers by table and one layer by its pointers; widths that end inside a tile, reductions
that run over layer boundaries, shorter than a block of 32 rows, of one row and of none.  In double from the same bfloat16
values: float sums of up to n terms of either sign are off by about sqrt(n) 2^-24 of them, 3e-6 of the largest result.
Every case says which form it is meant to run in, written and added, and fails if the rule comes to choose another."""
import numpy as np
import pytest

from tests.gpu_util import has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

EDGES = [0, 1, 31, 32, 33, 64, 5, 95, 96, 97, 0, 130, 200]
# name: (d, f, rows of every expert in every layer, form written, form added): s tiles of 128 x 128, b of 256 x 256, b2 in a
# launch each, + past the caches
CASES = {
    "one-tile": (64, 64, [EDGES], "b", "b"),
    "three-layers": (192, 128, [EDGES, EDGES[::-1], [7] * len(EDGES)], "s", "s"),
    "layers-shorter-than-a-block": (64, 192, [[1] * 5 + [0] * 3, [2] * 8, [0] * 4 + [3] * 4, [40] * 8], "s", "s"),
    "odd-widths": (320, 448, [[30 * i for i in range(9)]] * 2, "s", "s"),
    "whole-tiles": (256, 512, [[900, 1100, 0, 1000, 950, 1050]], "s", "s"),
    "empty": (64, 64, [[0, 0, 0]], "b", "b"),
    "written-large-added-small": (320, 320, [[449 + i % 5 for i in range(215)]], "b+", "s+"),
    # large tiles with all four passes of old values, whole ones and ones that end inside, both ways
    "large-odd-widths": (576, 1088, [[600, 0, 1, 1200], [1, 900, 31, 0], [700] * 4, [0, 0, 2400, 33]] * 2, "b", "b"),
    "large-streamed": (1024, 1088, [[200 + i for i in range(16)], [0] * 8 + [390] * 8] * 4, "b+", "b+"),
    "two-launches": (320, 512, [[500 + i % 41 for i in range(480)]] * 8, "b2+", "b2+"),
}


def _form(U, sh, n_layers, accumulate):
    m, b = U.tile_forms(sh, n_layers, accumulate), U.binding
    return ("s" if m & b.SMALL_WGRAD else "b2" if m & b.WGRAD_TWO_LAUNCHES else "b") + ("+" if m & b.WGRAD_STREAMED else "")


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_weight_gradients(name, accumulate):
    import torch
    import paper_2605_06665_amd as U
    d, f, layers, written, added = CASES[name]
    E, L = len(layers[0]), len(layers)
    g = torch.Generator(device="cuda").manual_seed(E + d)

    def rnd(*shape):
        return torch.empty(shape, device="cuda").normal_(0.0, 1.0, generator=g).to(torch.bfloat16)

    offs = [np.concatenate([[0], np.cumsum(r)]).astype(np.int32) for r in layers]
    S = max(int(o[-1]) for o in offs)
    sh = U.Shape(T=max(S, 1), d_model=d, d_ff=f, E=E, k=1, L=1, dtype=U.BF16, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0,
                 router=0)
    assert _form(U, sh, L, accumulate) == (added if accumulate else written)
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    # (layers with the same list of rows have the same operands)
    made = {id(r): [rnd(max(S, 1), n) for n in (d, f, d, 2 * f)] for r in layers}
    x, h, dy, da = ([made[id(r)][i] for r in layers] for i in range(4))
    goff = [torch.from_numpy(o).cuda() for o in offs]

    def tab(ts):
        return torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device="cuda")

    old = [torch.empty((E, *s), device="cuda").normal_(0.0, 1.0, generator=g) for s in ((2 * f, d), (d, f))]
    got = [t.clone() if accumulate else torch.full_like(t, float("nan")) for t in old]
    U.expert_wgrad(sh, L, tab(x), tab(da), tab(h), tab(dy), tab(goff), *got, accumulate, ws)
    outs = [got]
    if accumulate and L == 1 and S > 0:                     # the same through the backward call of one layer
        one = [t.clone() for t in old]
        a, b = rnd(S, f), rnd(S, f)
        wgu, wd = rnd(E, 2 * f, d), rnd(E, d, f)
        dact, dx = torch.empty_like(da[0]), torch.empty_like(x[0])
        U.expert_ffn_bwd(sh, dy[0], x[0], a, b, h[0], goff[0], wgu, wd, dx, dact, *one, ws)
        outs.append(one)
        acts = [da, [dact]]
    else:
        acts = [da]
    for got, act in zip(outs, acts):
        for e in (range(E) if E < 50 else (0, 1, 7, 100, E - 1)):
            want = [t[e].double().cpu().numpy() * accumulate for t in old]
            for l in range(L):
                r = slice(int(offs[l][e]), int(offs[l][e + 1]))
                want[0] = want[0] + (act[l][r].double().T @ x[l][r].double()).cpu().numpy()
                want[1] = want[1] + (dy[l][r].double().T @ h[l][r].double()).cpu().numpy()
            for t, w in zip(got, want):
                assert rel_err(host(t[e]), w) <= 1e-5, (name, e)
        assert all(torch.isfinite(t).all() for t in got)
