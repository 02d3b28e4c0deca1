"""GPU: dispatch of more than a few tokens in one launch and by chunks (token counts on both sides of both lines, blocks
that are not full, pools of 1 to 512 experts, rows that are not a multiple of 16 bytes, index maps alone), bit for bit
what a stable sort gives; the combine with a row shared by several wavefronts on both sides of its line, within one
rounding of the result and one per addend."""
import numpy as np
import pytest

from tests.gpu_util import has_gpu, host

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _shape(U, T, d, E, k, dtype):
    return U.Shape(T=T, d_model=d, d_ff=64, E=E, k=k, L=1, dtype=dtype, sigma=1.0, c=1.0, eps=1e-6, alpha_pool=0.0, router=0)


def _picks(rng, T, E, k, skew):
    score = rng.random((T, E))
    if skew:                        # nearly all tokens pick the same experts
        score[:, :k] += 0.9
    return np.ascontiguousarray(np.argsort(-score, axis=1)[:, :k].astype(np.int32))


# (T, E, k, d, dtype, skewed)
PERMUTES = [(257, 8, 1, 64, "bf16", False), (272, 512, 8, 128, "bf16", False), (300, 1, 1, 3, "f32", False),
            (999, 90, 3, 37, "f32", False), (1001, 12, 3, 252, "f32", True), (1025, 500, 8, 64, "bf16", False),
            (4095, 192, 2, 64, "bf16", False),
            (4096, 512, 8, 64, "bf16", True), (4096, 16, 1, 64, "bf16", True), (4096, 64, 3, 5, "f32", False),
            (4097, 64, 3, 5, "f32", False), (4097, 16, 1, 64, "bf16", True),
            # rows on both sides of 8 KiB, or of 4 KiB a pick, copies on both sides of 256 MB
            (300, 24, 2, 4096, "bf16", False), (300, 24, 2, 4160, "bf16", False), (257, 3, 1, 1023, "f32", False),
            (257, 3, 1, 1025, "f32", False), (260, 9, 3, 3071, "f32", True), (260, 9, 3, 3073, "f32", True), (3906, 64, 8, 4096, "bf16", False), (3907, 64, 8, 4096, "bf16", False)]


@pytest.mark.parametrize("copy", [True, False])
@pytest.mark.parametrize("T,E,k,d,dtype,skew", PERMUTES)
def test_permute(T, E, k, d, dtype, skew, copy):
    import torch
    import paper_2605_06665_amd as U
    rng = np.random.default_rng(T + E)
    idx = _picks(rng, T, E, k, skew)
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    sh = _shape(U, T, d, E, k, U.BF16 if dtype == "bf16" else U.F32)
    counts = np.bincount(idx.ravel(), minlength=E).astype(np.int32)
    slot_of_row = np.argsort(idx.ravel(), kind="stable").astype(np.int32)
    row_of_slot = np.empty_like(slot_of_row)
    row_of_slot[slot_of_row] = np.arange(T * k, dtype=np.int32)
    x = torch.randn((T, d), generator=torch.Generator().manual_seed(T)).to(act).cuda()
    i32 = dict(dtype=torch.int32, device="cuda")
    off, ros, sor = (torch.full((n + 1,), -7, **i32) for n in (E + 1, T * k, T * k))
    xp = torch.full((T * k + 1, d), 7.0, dtype=act, device="cuda")
    ws = torch.full((U.workspace_bytes(sh),), 0xff, dtype=torch.uint8, device="cuda")
    U.permute(sh, x, torch.from_numpy(idx).cuda(), torch.from_numpy(counts).cuda(), xp if copy else None, off, ros, sor, ws)
    assert np.array_equal(host(off)[:-1], np.concatenate([[0], np.cumsum(counts)]))
    assert np.array_equal(host(ros)[:-1], row_of_slot) and np.array_equal(host(sor)[:-1], slot_of_row)
    assert host(off)[-1] == host(ros)[-1] == host(sor)[-1] == -7
    if copy:
        assert torch.equal(xp[:-1], x[torch.from_numpy(slot_of_row // k).long().cuda()])
        assert bool((xp[-1] == 7.0).all())


def test_wide_rows_are_copied_as_fast_as_short_ones():
    """The same 262 MB as 8000 rows of 32 KiB and as 32800 rows of 8 KiB (57 and 58 us; the former 120 where a wavefront copied
    two rows one after the other)."""
    import torch
    import paper_2605_06665_amd as U
    E, k = 192, 8

    def best_time(T, d):
        sh = _shape(U, T, d, E, k, U.F32)
        idx = _picks(np.random.default_rng(T), T, E, k, False)
        picks, counts = (torch.from_numpy(v.astype(np.int32)).cuda() for v in (idx, np.bincount(idx.ravel(), minlength=E)))
        x, xp = torch.randn((T, d), device="cuda"), torch.empty((T * k, d), device="cuda")
        off, ros, sor = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (E + 1, T * k, T * k))
        ws = torch.empty(U.workspace_bytes(sh), dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                U.permute(sh, x, picks, counts, xp, off, ros, sor, ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert best_time(1000, 8192) <= 1.5 * best_time(4100, 2048)


@pytest.mark.parametrize("T,k,d,dtype", [(1, 1, 64, "bf16"), (3, 2, 512, "bf16"), (5, 3, 576, "bf16"), (2048, 8, 1088, "bf16"),
                                         (2049, 2, 1088, "bf16"), (1, 1, 1, "f32"), (7, 3, 255, "f32"), (6, 2, 257, "f32"),
                                         (9, 4, 1030, "f32"), (2048, 3, 260, "f32"), (2049, 3, 260, "f32")])
@pytest.mark.parametrize("gated", [True, False])
def test_combine(T, k, d, dtype, gated):
    import torch
    import paper_2605_06665_amd as U
    g = torch.Generator().manual_seed(T * d)
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    y = torch.randn((T * k, d), generator=g).to(act)
    ros = torch.randperm(T * k, generator=g).to(torch.int32)
    gate = torch.rand((T, k), generator=g)
    out = torch.full((T + 1, d), 7.0, dtype=act, device="cuda")
    U.combine(_shape(U, T, d, 16, k, U.BF16 if dtype == "bf16" else U.F32), y.cuda(), ros.cuda(), gate.cuda() if gated else None,
              out)
    terms = y.double()[ros.long()].reshape(T, k, d) * (gate.double()[:, :, None] if gated else 1.0)
    ref, got = terms.sum(1), out[:-1].double().cpu()
    # k products and k - 1 sums in float (half a last place is 2^-24), then eight significant bits: half a last place is 2^-8
    bound = (k + 1) * 2.0 ** -24 * terms.abs().sum(1) * 1.01 + (2.0 ** -8 * 1.01 * ref.abs() if dtype == "bf16" else 0.0)
    assert bool(((got - ref).abs() <= bound).all())
    assert bool((out[-1] == 7.0).all())
