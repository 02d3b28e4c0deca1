"""GPU parity of whole steps (and of the gathered forward pass) at the sizes where kernels change over or run out of
whole tiles, against the float64 oracle."""
import numpy as np
import pytest

from oracle import unipool_oracle as O
from synth import workloads as W
from tests.gpu_util import TOL, check_selection, dev, has_gpu, host, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

CASES = {
    # float contractions: 32 x 32 and 64 x 64 tiles, four values at a time or one by one, more row groups than a
    # wavefront has lanes, the router's weight gradient in one piece and cut over the tokens
    "f32-one-token": W.Workload("s", L=1, E=3, d=7, f=5, k=1, T=1, dtype="f32", seed=81, c=1.7),
    "f32-scalar-loads": W.Workload("s", L=2, E=70, d=34, f=66, k=2, T=300, dtype="f32", seed=82, c=2.6),
    "f32-many-groups": W.Workload("s", L=1, E=130, d=64, f=128, k=1, T=700, dtype="f32", seed=83, c=2.9, skew="zipf"),
    "f32-big-tiles": W.Workload("s", L=1, E=2, d=260, f=264, k=2, T=2049, dtype="f32", seed=84, c=1.2),
    "f32-mixed-alignment": W.Workload("s", L=3, E=5, d=65, f=64, k=3, T=97, dtype="f32", seed=85, c=2.0),
    # bfloat16 pools that are not a multiple of 8: rows of the logits' gradient filled up with zeros
    "bf16-three-experts": W.Workload("s", L=2, E=3, d=64, f=64, k=2, T=33, dtype="bf16", seed=86, c=1.5),
    "bf16-90-experts": W.Workload("s", L=2, E=90, d=192, f=128, k=3, T=777, dtype="bf16", seed=87, c=2.6),
    "bf16-257-experts": W.Workload("s", L=1, E=257, d=128, f=64, k=4, T=1030, dtype="bf16", seed=88, c=3.3),
}


@pytest.mark.parametrize("wgrad", ["pool", "layer"])
@pytest.mark.parametrize("name", list(CASES))
def test_step_against_oracle(name, wgrad):
    import torch
    import paper_2605_06665_amd as U
    from paper_2605_06665_amd.pipeline import PoolStep
    w, tol = CASES[name], TOL[CASES[name].dtype]
    xs, wrs, gs = ([g(w, l) for l in range(w.L)] for g in (W.gen_x, W.gen_w_router, W.gen_grad_out))
    wg, wu, wd = W.gen_pool_weights(w)
    sig = [1.0 + 0.1 * l for l in range(w.L)]
    ps = PoolStep(w.T, w.d, w.f, w.E, w.k, w.L, U.BF16 if w.dtype == "bf16" else U.F32, w.c, w.eps, w.alpha, wgrad=wgrad)
    put = lambda ts: [dev(t, w.dtype) for t in ts]   # noqa: E731
    dx_, dwr_, dg_ = put(xs), put(wrs), put(gs)
    dwgu, dwd = dev(np.concatenate([wg, wu], axis=1), w.dtype), dev(wd, w.dtype)
    ps.step(dx_, dwr_, sig, dwgu, dwd, dg_)
    torch.cuda.synchronize()
    idxs = []
    for l in range(w.L):
        z = O.router_logits(xs[l], wrs[l])
        idxs.append(check_selection(z, O.topk_select(z, w.k), host(ps.layers[l].topk_idx), w.k)[1])
    ref = O.pool_step(xs, wrs, wg, wu, wd, gs, w.k, sig, w.c, w.eps, w.alpha, idxs=idxs)
    assert np.array_equal(host(ps.counts), ref["counts"])
    for l in range(w.L):
        st, fw, bw = ps.layers[l], ref["fw"][l], ref["bw"][l]
        assert rel_err(host(st.out), fw["out"]) <= tol, "out"
        assert rel_err(host(st.dx), bw["dx"]) <= tol, "dx"
        assert rel_err(host(st.d_w_router), bw["dw_router"]) <= tol, "dw_router"
        # one sum of signed terms: its error scales with the terms, not with what they cancel to
        terms = np.linalg.norm(bw["dgate"] * fw["gate"] / sig[l])
        assert abs(float(host(st.d_sigma)[0]) - bw["dsigma"]) <= tol * max(abs(bw["dsigma"]), terms, 1e-3)
    assert rel_err(host(ps.d_w_gate_up), np.concatenate([ref["dw_gate"], ref["dw_up"]], axis=1)) <= tol
    assert rel_err(host(ps.d_w_down), ref["dw_down"]) <= tol
    # the dispatch fused into the first GEMM gives the same bits
    outs = [st.out.clone() for st in ps.layers]
    for l in range(w.L):
        ps.forward_layer(l, dx_[l], dwr_[l], sig[l], dwgu, dwd, gather=True)
    torch.cuda.synchronize()
    assert all(torch.equal(a, st.out) for a, st in zip(outs, ps.layers))
