"""Host-side checks of the C-ABI library: it loads, exports every function the header declares,
and rejects bad shapes without touching a GPU."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def U():
    import __graft_entry__ as g
    g.ensure_built()
    import paper_2605_06665_amd as U
    U.load_library()
    return U


def declared_functions():
    text = open(os.path.join(ROOT, "include", "unipool.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(unipool_[a-z_0-9]+)\s*\(", text)))


def test_header_functions_are_exported(U):
    names = declared_functions()
    assert len(names) >= 12
    lib = U.load_library()
    for n in names:
        assert hasattr(lib, n), n
    from paper_2605_06665_amd import binding
    assert sorted(binding.ENTRY_POINTS) == names


def test_workspace_size_and_shape_validation(U):
    sh = U.Shape(T=128, d_model=64, d_ff=128, E=8, k=2, L=2, dtype=U.F32, sigma=1.0, c=2.5, eps=1e-6,
                 alpha_pool=0.01)
    n = U.workspace_bytes(sh)
    assert n > 0 and n % 256 == 0
    big = U.Shape(T=32768, d_model=1536, d_ff=4096, E=192, k=2, L=24, dtype=U.BF16, sigma=1.0, c=3.8,
                  eps=1e-6, alpha_pool=0.02)
    assert U.workspace_bytes(big) > n
    for field, value, msg in (("k", 9, "k=9"), ("E", 513, "E=513"), ("T", 0, "positive"),
                              ("dtype", 7, "dtype"), ("sigma", -1.0, "sigma")):
        bad = U.Shape(T=128, d_model=64, d_ff=128, E=8, k=2, L=2, dtype=U.F32, sigma=1.0, c=2.5, eps=1e-6,
                      alpha_pool=0.01)
        setattr(bad, field, value)
        with pytest.raises(U.UniPoolError, match=msg):
            U.workspace_bytes(bad)
    bad = U.Shape(T=128, d_model=100, d_ff=128, E=8, k=2, L=2, dtype=U.BF16, sigma=1.0, c=2.5, eps=1e-6,
                  alpha_pool=0.01)
    with pytest.raises(U.UniPoolError, match="multiples of 64"):
        U.workspace_bytes(bad)


def test_null_arguments_fail_before_any_launch(U):
    sh = U.Shape(T=128, d_model=64, d_ff=128, E=8, k=2, L=2, dtype=U.F32, sigma=1.0, c=2.5, eps=1e-6,
                 alpha_pool=0.01)
    with pytest.raises(U.UniPoolError, match="NULL"):
        U.combine(sh, None, None, None, None, stream=0)
    with pytest.raises(U.UniPoolError, match="NULL"):
        U.pool_aux_loss(sh, None, None, None, None, None, None, None, stream=0)
    assert "NULL" in U.last_error()


def test_fast_path_reports_the_kernel_families(U):
    def sh(**kw):
        base = dict(T=512, d_model=128, d_ff=192, E=64, k=2, L=2, dtype=U.BF16, sigma=1.0, c=2.5, eps=1e-6,
                    alpha_pool=0.01)
        base.update(kw)
        return U.Shape(**base)
    assert U.fast_path(sh()) == 7                       # MFMA experts, MFMA router, fused router
    assert U.fast_path(sh(E=512)) == 7                  # the largest pool the fused router takes
    assert U.fast_path(sh(d_model=192)) == 3            # d_model not a multiple of 128: logits GEMM and selection in two kernels
    assert U.fast_path(sh(E=10)) == 1                   # E not a multiple of 8: plain router kernels
    assert U.fast_path(sh(dtype=U.F32)) == 0            # float mode: plain kernels throughout
    with pytest.raises(U.UniPoolError, match="k=9"):
        U.fast_path(sh(k=9))


def test_tile_forms_are_found_at_any_number_of_rows(U):
    """The choice is made on the host in every call: its time may not grow with the rows (134 million rows of one expert are
    1.5 million tiles of both sizes; loops over them took 10 ms)."""
    import time
    sh = U.Shape(T=134_000_000, d_model=8192, d_ff=64, E=1, k=1, L=1, dtype=U.BF16, sigma=1.0, c=2.5, eps=1e-6, alpha_pool=0.01)
    best = 1.0
    for _ in range(3):
        t0 = time.perf_counter()
        forms = U.tile_forms(sh)
        best = min(best, time.perf_counter() - t0)
    assert best < 1e-3
    # 64 columns (dH) are half a small tile and a quarter of a large one, 8192 whole tiles of both
    from paper_2605_06665_amd import binding as B
    assert forms & (B.SMALL_DH | B.SMALL_DX) == B.SMALL_DH
    with pytest.raises(U.UniPoolError, match="n_layers=0"):
        U.tile_forms(sh, 0, False)
    sh.dtype = U.F32
    assert U.tile_forms(sh) == 0


def test_tile_forms_of_few_rows(U):
    """Where large tiles all run at once and small ones do not get a compute unit each, few rows per expert keep the large ones
    (256 compute units, as on a host without a device)."""
    from paper_2605_06665_amd import binding as B

    def small(T, k, E, d, f, bit):
        return bool(U.tile_forms(U.Shape(T=T, d_model=d, d_ff=f, E=E, k=k, L=1, dtype=U.BF16, sigma=1.0, c=2.5, eps=1e-6,
                                         alpha_pool=0.01)) & bit)
    assert not small(141, 2, 9, 640, 2176, B.SMALL_GATE_UP)        # 31 rows, 153 large tiles or 306 small ones
    assert not small(95, 2, 31, 1280, 1536, B.SMALL_DX)            # 6 rows, 155 or 310
    assert not small(1749, 1, 33, 1088, 960, B.SMALL_DH)           # 53 rows, 132 or 264
    assert small(230, 8, 30, 1152, 192, B.SMALL_DX)                # 61 rows, 150 or 270
    assert small(95, 2, 31, 1280, 1536, B.SMALL_GATE_UP)           # 372 large tiles: two rounds
    assert small(567, 8, 23, 192, 1856, B.SMALL_DOWN)              # 46 small tiles: one each
    # fewer picks than experts: those without rows have no tiles
    assert not small(16, 4, 96, 1024, 2816, B.SMALL_DX)            # 47 experts, 187 large tiles or 374 small ones
    assert small(30, 2, 64, 768, 2048, B.SMALL_DX)                 # 39 experts, 234 small tiles: one each


def test_weight_gradients_in_two_launches_are_long(U):
    from paper_2605_06665_amd import binding as B

    def two(E, d, f, rows, n_layers=1):
        return bool(U.tile_forms(U.Shape(T=E * rows // n_layers, d_model=d, d_ff=f, E=E, k=1, L=1, dtype=U.BF16, sigma=1.0, c=2.5,
                                         eps=1e-6, alpha_pool=0.01), n_layers, False) & B.WGRAD_TWO_LAUNCHES)
    assert two(96, 1024, 2816, 5460) and two(90, 832, 1472, 4800, 8)
    assert not two(64, 768, 2048, 1024) and not two(96, 1024, 2816, 682)       # few rows
    assert not two(64, 768, 2048, 8192)                                        # 18 rounds of tiles
