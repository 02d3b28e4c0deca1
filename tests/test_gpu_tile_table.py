"""GPU: the tile table of the grouped GEMMs over pool sizes and row counts at its edges: short last laps of the
dealing (E mod 8 in both directions), empty experts, all experts of one size class, counts on both sides of the
2048-row change of class width, one expert with nearly all rows.  At these widths all products run in tiles of 128 x 128
(test_gpu_tile_forms.py has the tables of 256-row tiles)."""
import numpy as np
import pytest

from tests.gpu_util import TOL, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

COUNTS = {
    "one-expert": [300],
    "seven": [5, 0, 700, 1, 256, 257, 16],
    "nine-equal": [33] * 9,
    "backward-lap": [17 * i for i in range(13)],                 # E = 13: the second lap is short and runs backwards
    "forward-lap": [(37 * i) % 91 for i in range(19)],           # E = 19: the third lap is short and runs forwards
    "class-change": [2047, 2048, 2049, 2175, 2176, 4095, 4096, 0, 1, 15],
    "hot": [0] * 60 + [9000] + [3] * 50,
    "511": [i % 7 for i in range(511)],
    "512-empty-but-one": [0] * 511 + [70],
}


@pytest.mark.parametrize("name", list(COUNTS))
def test_every_row_meets_its_expert(name):
    import torch
    import paper_2605_06665_amd as U
    counts = COUNTS[name]
    E, d, f = len(counts), 64, 64
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    S = int(off[-1])
    g = torch.Generator().manual_seed(len(counts))
    x = torch.randn((S, d), generator=g).to(torch.bfloat16)
    wgu = (torch.randn((E, 2 * f, d), generator=g) * 0.1).to(torch.bfloat16)
    wd = (torch.randn((E, d, f), generator=g) * 0.1).to(torch.bfloat16)
    sh = U.Shape(T=S, d_model=d, d_ff=f, E=E, k=1, L=1, dtype=U.BF16, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0,
                 router=0)
    assert U.tile_forms(sh) & 15 == 15
    ws = torch.empty(U.workspace_bytes(sh), dtype=torch.uint8, device="cuda:0")
    a, b, h = (torch.full((S, f), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
    y = torch.full((S, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    U.expert_ffn_fwd(sh, x.cuda(), torch.from_numpy(off).cuda(), wgu.cuda(), wd.cuda(), a, b, h, y, ws)
    torch.cuda.synchronize()
    for e, n in enumerate(counts):
        if n == 0:
            continue
        r = slice(int(off[e]), int(off[e + 1]))
        z = x[r].double() @ wgu[e].double().T
        ra, rb = z[:, :f], z[:, f:]
        rh = ra / (1 + torch.exp(-ra)) * rb
        for got, want in ((a, ra), (b, rb), (h, rh), (y, host(h[r]).astype(np.float64) @ wd[e].double().T.numpy())):
            assert rel_err(host(got[r]), np.asarray(want)) <= TOL["bf16"], (name, e)
