"""Host side of PoolStep: which buffers it owns from the start (nothing is launched)."""
import pytest


@pytest.mark.parametrize("wgrad,L,pairs", [("layer", 6, 1), ("pool", 6, 6), ("layer", 1, 1)])
def test_backward_buffers_of_a_new_step(wgrad, L, pairs):
    import __graft_entry__ as g
    g.ensure_built()
    import paper_2605_06665_amd as U
    from paper_2605_06665_amd.pipeline import PoolStep
    ps = PoolStep(30, 64, 64, 16, 2, L, U.BF16, 2.6, 1e-6, 0.01, device="cpu", wgrad=wgrad)
    assert len(ps._dy) == len(ps._dact) == pairs
    assert sum(len(ls) for ls, _ in ps._wgrad_groups) == L
    with pytest.raises(AssertionError):
        PoolStep(30, 64, 64, 16, 2, L, U.BF16, 2.6, 1e-6, 0.01, device="cpu", wgrad="pool", wgrad_layers=2)
