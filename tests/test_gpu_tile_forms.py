"""GPU: the two tile sizes of the row-grouped products (256 x 256, 128 x 128) at the edges of rows, columns and
reductions: row counts around the 16-row units, 32-row strips and both tiles, column counts that end inside a tile,
reductions of one, two and three stages, one or both tables in a call.  Everything is compared with float64, and the row
after the last has to stay as it is.  Every case says which of its four products (gate and up, down, dH, dX) are meant to run
in which size, and fails if the rule comes to choose another."""
import numpy as np
import pytest

from tests.gpu_util import TOL, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 112, 113, 127, 128, 129, 144, 160, 255, 256, 257, 300, 0]
# name: (d, f, rows of every expert, size of each product's tiles: s 128 x 128, b 256 x 256)
CASES = {
    "one-stage": (64, 64, EDGES, "ssss"),
    "two-stages-three-blocks": (128, 192, EDGES, "ssss"),
    "odd-columns": (320, 448, EDGES, "ssss"),
    "big-tiles-fill-the-chip": (1024, 256, [200 + 3 * i for i in range(70)], "bbsb"),
    "small-rows": (576, 320, [i % 60 for i in range(200)], "ssss"),
    "one-hot-expert": (192, 640, [0] * 7 + [2000] + [5] * 30, "bsss"),
    "long-reduction": (256, 2112, [150, 90, 129, 47], "ssss"),
    # the same edges in large tiles: the products with d_ff columns, whose reductions are d_model long, then the others, whose
    # reductions are d_ff and 2 d_ff long; columns that fill the tiles and that end in their first, second and last quarter
    "big-one-stage": (64, 512, EDGES * 4, "bsbs"),
    "big-two-stages": (128, 448, EDGES * 4, "bsbs"),
    "big-odd-columns": (64, 832, EDGES * 4, "bsbs"),
    "big-down-one-stage": (512, 64, EDGES * 4, "sbsb"),
    "big-down-two-stages": (448, 128, EDGES * 4, "sbsb"),
    "big-down-odd-columns": (320, 192, EDGES * 4, "bbsb"),
    "big-all": (512, 512, EDGES * 4, "bbbb"),
    # tables of large tiles, which give every expert an even number of places: short last laps of the dealing in both
    # directions, experts without rows, counts around the class width, one expert with nearly all rows, full tables
    "big-seven": (64, 4864, [5, 0, 700, 1, 256, 257, 16], "bsbs"),
    "big-nine-equal": (3840, 64, [33] * 9, "sbsb"),
    "big-backward-lap": (64, 2688, [17 * i for i in range(13)], "bsbs"),
    "big-forward-lap": (1856, 64, [(37 * i) % 91 for i in range(19)], "sbsb"),
    "big-class-change": (512, 576, [2047, 2048, 2049, 2175, 2176, 4095, 4096, 0, 1, 15], "bbbb"),
    "big-hot": (448, 448, [0] * 60 + [9000] + [3] * 50, "bbbb"),
    "big-511": (64, 512, [(37 * i) % 300 for i in range(511)], "bsbs"),
    "big-512-many-empty": (512, 64, [0] * 300 + [(41 * i) % 400 for i in range(211)] + [0], "sbsb"),
    "big-alone": (64, 1792, [5000], "bsbs"),
    # a reduction of 4096 (dX), in which the workgroups of a pair of row tiles meet
    "big-pairs": (1024, 2048, [300, 513, 0, 256, 700, 40, 511, 257, 0, 300, 480, 350] * 2, "bbbb"),
}


def _shape(U, d, f, counts):
    return U.Shape(T=sum(counts), d_model=d, d_ff=f, E=len(counts), k=1, L=1, dtype=U.BF16, sigma=1.0, c=1.0, eps=1e-6,
                   alpha_pool=0.0, router=0)


@pytest.mark.parametrize("name", list(CASES))
def test_products(name):
    import torch
    import paper_2605_06665_amd as U
    d, f, counts, sizes = CASES[name]
    E = len(counts)
    assert "".join("bs"[U.tile_forms(_shape(U, d, f, counts)) >> i & 1] for i in range(4)) == sizes
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    S = int(off[-1])
    g = torch.Generator().manual_seed(E + d)

    def rnd(*shape, std=1.0):
        return (torch.randn(shape, generator=g) * std).to(torch.bfloat16)

    x, dy = rnd(S, d), rnd(S, d)
    wgu, wd = rnd(E, 2 * f, d, std=d ** -0.5), rnd(E, d, f, std=f ** -0.5)
    sh = _shape(U, d, f, counts)
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda:0")
    a, b, h = (torch.full((S + 1, f), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
    y, dx = (torch.full((S + 1, d), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(2))
    dact = torch.full((S + 1, 2 * f), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    goff, gwgu, gwd = torch.from_numpy(off).cuda(), wgu.cuda(), wd.cuda()
    U.expert_ffn_fwd(sh, x.cuda(), goff, gwgu, gwd, a, b, h, y, ws)
    U.expert_ffn_bwd(sh, dy.cuda(), x.cuda(), a, b, h, goff, gwgu, gwd, dx, dact, None, None, ws)
    a, b, h, y, dx, dact = (host(t) for t in (a, b, h, y, dx, dact))
    for t in (a, b, h, y, dx, dact):
        assert np.isnan(t[S]).all() and np.isfinite(t[:S]).all()
    for e, n in enumerate(counts):
        if n == 0:
            continue
        r = slice(int(off[e]), int(off[e + 1]))
        we, de = wgu[e].double().numpy(), wd[e].double().numpy()
        z = x[r].double().numpy() @ we.T
        ra, rb = z[:, :f], z[:, f:]
        # each product from the rounded tensors it reads
        ga, gb = a[r].astype(np.float64), b[r].astype(np.float64)
        sg = 1 / (1 + np.exp(-ga))
        dh = dy[r].double().numpy() @ de
        rdact = np.concatenate([dh * gb * sg * (1 + ga * (1 - sg)), dh * ga * sg], axis=1)
        for got, want in ((a[r], ra), (b[r], rb), (h[r], ra / (1 + np.exp(-ra)) * rb),
                          (y[r], h[r].astype(np.float64) @ de.T), (dact[r], rdact),
                          (dx[r], dact[r].astype(np.float64) @ we)):
            assert rel_err(got, want) <= TOL["bf16"], (name, e)


def test_recomputation_builds_its_own_table_only():
    """expert_ffn_recompute runs the product of w_gate_up alone: where that of w_down would take the other tile size, its table
    (in the area of the router gradient's partial products, the last of the workspace) is not built."""
    import torch
    import paper_2605_06665_amd as U
    d, f, counts, sizes = CASES["one-hot-expert"]
    assert sizes[0] != sizes[1]
    sh, S, E = _shape(U, d, f, counts), sum(counts), len(counts)
    g = torch.Generator().manual_seed(1)
    x, wgu = (torch.randn(s, generator=g).to(torch.bfloat16).cuda() for s in ((S, d), (E, 2 * f, d)))
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda:0")
    a, b, h = (torch.empty((S, f), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
    U.expert_ffn_recompute(sh, x, off, wgu, a, b, h, ws)
    partials = 64 * ((E + 7) // 8 * 8) * d * 4
    assert bool((ws[-partials:] == 0xff).all())
    y = torch.empty((S, d), dtype=torch.bfloat16, device="cuda:0")
    a2, b2, h2 = (torch.empty_like(t) for t in (a, b, h))
    U.expert_ffn_fwd(sh, x, off, wgu, torch.zeros((E, d, f), dtype=torch.bfloat16, device="cuda:0"), a2, b2, h2, y, ws)
    assert not bool((ws[-partials:] == 0xff).all())                          # the forward pass has built it there
    assert torch.equal(a, a2) and torch.equal(b, b2) and torch.equal(h, h2)
