"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on
the same seeded float32 inputs.  Tolerance: normwise relative error
max_b ||got_b - ref_b||_inf / ||ref_b||_inf <= 1e-4 for solves, forward states
and adjoints; ||.||_inf over the whole tensor for dW, db."""
import json
import math
import os
import sys

import numpy as np
import pytest

import oracle
from paper_2309_16318_amd import deeppcr, synth
from tests._util import normwise_rel_err, per_layer_rel_err

pytestmark = pytest.mark.gpu
TOL = 1e-4

torch = pytest.importorskip("torch")

# Newton solve counts of the oracle on the full-size forward workloads,
# written by tests/golden/make_newton_counts.py (oracle only).
with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden",
                       "newton_counts.json")) as _f:
    NEWTON_COUNTS = json.load(_f)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def g(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev)


def h(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


# ----------------------------------------------------------------- PCR solve
SWEEP_W = [1, 3, 4, 8, 15, 16, 17, 32, 33, 64, 128]
SWEEP_L = [1, 2, 3, 31, 64, 1000]


def _sweep_cases():
    for w in SWEEP_W:
        for L in SWEEP_L:
            for B in (1, 5):
                if B * L * w * w > (1 << 22):
                    continue
                yield w, L, B


@pytest.mark.parametrize("w,L,B", list(_sweep_cases()))
@pytest.mark.parametrize("transpose", [0, 1])
def test_pcr_solve_shape_sweep(dev, w, L, B, transpose):
    _say(f"pcr sweep w={w} L={L} B={B} transpose={transpose}")
    d = synth.random_system(B, L, w, seed=1000 + 7 * w + L + B, scale=0.9)
    x = h(deeppcr.pcr_solve_block_bidiag(g(d["J"], dev), g(d["r"], dev), transpose=transpose))
    ref = oracle.seq_solve(d["J"], d["r"], bool(transpose))
    assert normwise_rel_err(x, ref) <= TOL


@pytest.mark.parametrize("transpose", [1, 0])
def test_pcr_solve_workload(dev, transpose):
    wl = synth.WORKLOADS["pcr_solve"]
    _say(f"pcr workload B={wl.B} L={wl.L} w={wl.w} transpose={transpose}")
    d = synth.workload_inputs(wl)
    x = h(deeppcr.pcr_solve_block_bidiag(g(d["J"], dev), g(d["r"], dev), transpose=transpose))
    ref = oracle.seq_solve(d["J"], d["r"], bool(transpose))
    err = normwise_rel_err(x, ref)
    _say(f"  normwise rel err {err:.3e}")
    assert err <= TOL


def test_pcr_solve_x_aliases_r(dev):
    for L in (2, 37):
        d = synth.random_system(3, L, 16, seed=5, scale=0.9)
        r = g(d["r"], dev)
        deeppcr.pcr_solve_block_bidiag(g(d["J"], dev), r, x=r, transpose=0)
        assert normwise_rel_err(h(r), oracle.seq_solve(d["J"], d["r"])) <= TOL


def test_pcr_solve_deterministic(dev):
    d = synth.random_system(4, 300, 32, seed=8, scale=0.9)
    J, r = g(d["J"], dev), g(d["r"], dev)
    a = h(deeppcr.pcr_solve_block_bidiag(J, r, transpose=1))
    b = h(deeppcr.pcr_solve_block_bidiag(J, r, transpose=1))
    assert np.array_equal(a, b)


def test_pcr_solve_ignores_first_block(dev):
    d = synth.random_system(2, 40, 8, seed=9, scale=0.9)
    J2 = d["J"].copy()
    J2[:, 0] = np.nan
    for tr in (0, 1):
        a = h(deeppcr.pcr_solve_block_bidiag(g(d["J"], dev), g(d["r"], dev), transpose=tr))
        b = h(deeppcr.pcr_solve_block_bidiag(g(J2, dev), g(d["r"], dev), transpose=tr))
        assert np.array_equal(a, b)


# ------------------------------------------------------------------- forward
def _forward(d, dev, layer, alpha, tol=1e-5, max_iter=20, Z_init=None):
    return deeppcr.deeppcr_mlp_forward(g(d["W"], dev), g(d["bias"], dev), g(d["z0"], dev),
                                       layer=layer, alpha=alpha, tol=tol, max_iter=max_iter,
                                       Z_init=Z_init)


@pytest.mark.parametrize("layer,alpha", [(0, 1.0), (1, 0.1)])
def test_forward_tiny_workload(dev, layer, alpha):
    wl = synth.WORKLOADS["tiny_fwd"]
    d = synth.workload_inputs(wl)
    res = _forward(d, dev, layer, alpha, wl.tol, wl.max_iter)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    assert normwise_rel_err(h(res.Z), ref) <= TOL
    _, k_ref, ok, _ = oracle.newton_forward(layer, alpha, d["W"], d["bias"], d["z0"], wl.tol,
                                            wl.max_iter)
    _say(f"tiny forward layer={layer}: gpu iters {res.iters}, oracle {k_ref}")
    assert ok and abs(res.iters - k_ref) <= 1


def test_forward_mlp_workload(dev):
    wl = synth.WORKLOADS["mlp_fwd"]
    _say(f"mlp forward B={wl.B} L={wl.L} w={wl.w}")
    d = synth.workload_inputs(wl)
    res = _forward(d, dev, wl.layer, wl.alpha, wl.tol, wl.max_iter)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"])
    err = normwise_rel_err(h(res.Z), ref)
    _, k_ref, ok, _ = oracle.newton_forward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"],
                                            wl.tol, wl.max_iter)
    _say(f"  err {err:.3e}; gpu iters {res.iters}, oracle {k_ref}")
    assert err <= TOL
    assert ok and abs(res.iters - k_ref) <= 1


def test_forward_residual_workload(dev):
    wl = synth.WORKLOADS["resnet_fwd_bwd"]
    _say(f"residual forward B={wl.B} L={wl.L} w={wl.w}")
    d = synth.workload_inputs(wl)
    res = _forward(d, dev, wl.layer, wl.alpha, wl.tol, wl.max_iter)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"])
    err = normwise_rel_err(h(res.Z), ref)
    k_ref = NEWTON_COUNTS[wl.name]["solves"]
    _say(f"  err {err:.3e}; gpu iters {res.iters}, oracle {k_ref}")
    assert err <= TOL
    assert NEWTON_COUNTS[wl.name]["converged"] and abs(res.iters - k_ref) <= 1


@pytest.mark.parametrize("w,L,B", [(1, 5, 2), (3, 40, 3), (16, 100, 2), (17, 33, 2),
                                   (32, 64, 2), (64, 20, 2), (128, 9, 2),
                                   (16, 1, 3), (16, 2, 3), (16, 3, 2), (32, 1, 2), (32, 2, 5),
                                   (32, 3, 2), (32, 4, 2), (32, 5, 3), (32, 9, 3), (16, 257, 4),
                                   (32, 130, 3), (64, 3, 2), (128, 4, 2),
                                   (4, 600, 2), (2, 3000, 1)])
@pytest.mark.parametrize("layer,alpha", [(0, 1.0), (1, 0.1)])
def test_forward_shapes(dev, w, L, B, layer, alpha):
    _say(f"forward shapes w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=300 + w + L)
    res = _forward(d, dev, layer, alpha)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    assert normwise_rel_err(h(res.Z), ref) <= TOL
    _, k_ref, ok, _ = oracle.newton_forward(layer, alpha, d["W"], d["bias"], d["z0"], 1e-5, 20)
    assert ok and abs(res.iters - k_ref) <= 1


ALL_KINDS = [(0, 1.0), (1, 0.1), (2, 1.0), (3, 0.1), (4, 1.0), (5, 0.1)]


@pytest.mark.parametrize("w,L,B", [(4, 30, 2), (16, 200, 3), (32, 100, 2), (64, 40, 2),
                                   (128, 12, 2), (17, 50, 2)])
@pytest.mark.parametrize("layer,alpha", ALL_KINDS)
def test_forward_all_layer_kinds(dev, w, L, B, layer, alpha):
    """tanh, sigmoid and ReLU layers, plain and residual, through every kernel
    family (single-workgroup, fused w = 16/32, tile w = 64/128, generic)."""
    _say(f"forward kinds w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=700 + w + L + layer)
    res = _forward(d, dev, layer, alpha)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    assert normwise_rel_err(h(res.Z), ref) <= TOL
    _, k_ref, ok, _ = oracle.newton_forward(layer, alpha, d["W"], d["bias"], d["z0"], 1e-5, 20)
    assert ok and abs(res.iters - k_ref) <= 1


# Tile widths with more systems than a group's 16 (w = 64, B = 40; w = 32, B =
# 64), a whole group (w = 128, B = 16) and half of one, deep and shallow, no
# depth a multiple of the chunks.
@pytest.mark.parametrize("w,L,B", [(64, 130, 40), (64, 300, 8), (128, 203, 16), (32, 130, 64),
                                   (32, 300, 40), (32, 17, 128), (32, 33, 64)])
@pytest.mark.parametrize("layer,alpha", ALL_KINDS)
def test_forward_tile_segments(dev, w, L, B, layer, alpha):
    _say(f"forward tile segments w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=1100 + w + L + layer)
    res = _forward(d, dev, layer, alpha)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    assert normwise_rel_err(h(res.Z), ref) <= TOL


@pytest.mark.parametrize("w,L,B", [(4, 30, 2), (16, 200, 3), (32, 100, 2), (64, 40, 2),
                                   (128, 12, 2), (17, 50, 2)])
@pytest.mark.parametrize("layer,alpha", ALL_KINDS)
def test_backward_all_layer_kinds(dev, w, L, B, layer, alpha):
    _say(f"backward kinds w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=800 + w + L + layer)
    Z32 = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"]).astype(np.float32)
    _backward_check(d, Z32, dev, layer, alpha)


@pytest.mark.parametrize("w", [8, 16, 32, 64])
def test_forward_fixed_count_and_prefix_exactness(dev, w):
    """tol = 0 runs exactly max_iter iterations; after k iterations from a
    zero start the first k rows equal the sequential pass (Eq. 3 is block
    lower-triangular)."""
    L, B = 12, 3
    d = synth.mlp_inputs(B, L, w, seed=41)
    ref = oracle.seq_forward(0, 1.0, d["W"], d["bias"], d["z0"])
    for k in (1, 3, 6):
        res = _forward(d, dev, 0, 1.0, tol=0.0, max_iter=k,
                       Z_init=torch.zeros((B, L, w), device=dev))
        assert res.status == deeppcr.OK and res.iters == k
        Z = h(res.Z)
        assert normwise_rel_err(Z[:, :k], ref[:, :k]) <= 1e-6


def test_forward_warm_start_from_solution(dev):
    wl = synth.WORKLOADS["tiny_fwd"]
    d = synth.workload_inputs(wl)
    ref = oracle.seq_forward(0, 1.0, d["W"], d["bias"], d["z0"])
    res = _forward(d, dev, 0, 1.0, Z_init=g(ref, dev))
    assert res.status == deeppcr.OK and res.iters == 1
    assert normwise_rel_err(h(res.Z), ref) <= TOL


def test_forward_reports_no_convergence(dev):
    d = synth.workload_inputs(synth.WORKLOADS["tiny_fwd"])
    res = _forward(d, dev, 0, 1.0, tol=1e-5, max_iter=1)
    assert res.status == deeppcr.ENOCONV and res.iters == 1


def test_forward_reports_non_finite(dev):
    d = synth.workload_inputs(synth.WORKLOADS["tiny_fwd"])
    d = dict(d)
    d["bias"] = d["bias"].copy()
    d["bias"][3, 1] = np.nan
    res = _forward(d, dev, 0, 1.0)
    assert res.status == deeppcr.ENONFINITE and res.iters == 1


# The same reports from the multi-kernel paths, whose substitution applies the
# update itself: blocks formed from the weights on the way (w = 16), split
# weights (w = 32, 64, 128).
@pytest.mark.parametrize("w,L,B", [(16, 100, 3), (64, 40, 2), (32, 130, 64), (64, 300, 8),
                                   (128, 203, 16)])
def test_forward_status_reports_every_path(dev, w, L, B):
    _say(f"forward status reports w={w} L={L} B={B}")
    d = dict(synth.mlp_inputs(B, L, w, seed=1700 + w + L))
    res = _forward(d, dev, 0, 1.0, tol=1e-5, max_iter=1)
    assert res.status == deeppcr.ENOCONV and res.iters == 1
    d["bias"] = d["bias"].copy()
    d["bias"][L // 2, 1] = np.nan
    res = _forward(d, dev, 0, 1.0)
    assert res.status == deeppcr.ENONFINITE and res.iters == 1


def test_profiling_times_selected_classes_and_changes_nothing(dev):
    """Instrumentation on (only the products' and the substitutions' classes timed, with
    events shared at span boundaries) leaves the result bitwise unchanged."""
    _say("profiling on a w=32 forward")
    d = synth.mlp_inputs(64, 130, 32, seed=31)
    ref = _forward(d, dev, 0, 1.0)
    timed = (deeppcr.KCLASS_PCR_LEVEL, deeppcr.KCLASS_PCR_TAIL)
    deeppcr.profile_reset()
    deeppcr.profile_select(timed)
    deeppcr.profile_enable(True)
    try:
        res = _forward(d, dev, 0, 1.0)
        res2 = _forward(d, dev, 0, 1.0)
    finally:
        deeppcr.profile_enable(False)
        deeppcr.profile_select(range(len(deeppcr.KCLASS_NAMES)))
    reads = {c: deeppcr.profile_read(c) for c in range(len(deeppcr.KCLASS_NAMES))}
    deeppcr.profile_reset()
    assert res.status == deeppcr.OK and res2.status == deeppcr.OK
    assert torch.equal(res.Z, ref.Z) and torch.equal(res2.Z, ref.Z)
    for c, rd in reads.items():
        if c in timed:
            assert rd["launches"] >= 2 * res.iters and rd["ms"] > 0.0 and rd["flops"] > 0.0
        else:
            assert rd["launches"] == 0 and rd["ms"] == 0.0
    assert all(deeppcr.profile_read(c)["launches"] == 0 for c in range(len(deeppcr.KCLASS_NAMES)))


def test_forward_deterministic(dev):
    d = synth.mlp_inputs(8, 64, 32, seed=12)
    a = h(_forward(d, dev, 1, 0.1).Z)
    b = h(_forward(d, dev, 1, 0.1).Z)
    assert np.array_equal(a, b)



# ------------------------------------------- residual stopping rule (App. F.1)
def _forward_res(d, dev, layer, alpha, atol=1e-4, rtol=1e-4, max_iter=15, Z_init=None):
    return deeppcr.deeppcr_mlp_forward_residual(g(d["W"], dev), g(d["bias"], dev),
                                                g(d["z0"], dev), layer=layer, alpha=alpha,
                                                atol=atol, rtol=rtol, max_iter=max_iter,
                                                Z_init=Z_init)


# every kernel family: single workgroup (4, 16), small widths (4, 600), (8, 300),
# fused w = 16 / 32 (including L <= 2), tile w = 64 / 128, generic (17)
RES_SHAPES = [(4, 16, 1), (4, 600, 2), (8, 300, 2), (16, 200, 3), (32, 100, 2), (32, 2, 3),
              (64, 40, 2), (128, 12, 2), (17, 50, 2)]


@pytest.mark.parametrize("w,L,B", RES_SHAPES)
@pytest.mark.parametrize("layer,alpha", [(0, 1.0), (1, 0.1), (4, 1.0)])
def test_forward_residual_rule(dev, w, L, B, layer, alpha):
    """Paper defaults (atol = rtol = 1e-4, at most 15 solves): the solve count
    is within one of the oracle's, the iterate equals the oracle's Newton
    iterate after the same number of solves, and the reported residual is
    the residual of the returned iterate and meets a threshold."""
    _say(f"forward residual rule w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=900 + w + L + layer)
    res = _forward_res(d, dev, layer, alpha)
    assert res.status == deeppcr.OK
    Zg = h(res.Z)
    _, k_ref, ok, hist = oracle.newton_forward_residual(layer, alpha, d["W"], d["bias"], d["z0"],
                                                        1e-4, 1e-4, 15)
    _say(f"  gpu solves {res.iters} residual {res.residual:.3e}; oracle {k_ref} {hist[-1]:.3e}")
    assert ok and abs(res.iters - k_ref) <= 1
    if res.iters == 0:
        Zk = oracle.initial_guess(layer, alpha, *(d[k].astype(np.float64)
                                                  for k in ("W", "bias", "z0")))
    else:
        Zk, _, _, _ = oracle.newton_forward(layer, alpha, d["W"], d["bias"], d["z0"], 0.0,
                                            res.iters)
    assert normwise_rel_err(Zg, Zk) <= TOL
    r_own = oracle.residual_norm(layer, alpha, d["W"], d["bias"], d["z0"], Zg)
    assert abs(res.residual - r_own) <= 1e-5 + 1e-3 * r_own
    assert res.residual <= max(1e-4, 1e-4 * hist[0]) * (1 + 1e-3) + 1e-6
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    assert normwise_rel_err(Zg, ref) <= 1e-3
    if res.iters >= 1:
        # one solve fewer is not enough: ENOCONV with a residual above both thresholds
        prev = _forward_res(d, dev, layer, alpha, max_iter=res.iters - 1)
        assert prev.status == deeppcr.ENOCONV and prev.iters == res.iters - 1
        assert prev.residual > 1e-4


def test_forward_residual_rule_mlp_workload(dev):
    wl = synth.WORKLOADS["mlp_fwd"]
    _say(f"mlp forward, residual rule, B={wl.B} L={wl.L} w={wl.w}")
    d = synth.workload_inputs(wl)
    res = _forward_res(d, dev, wl.layer, wl.alpha)
    assert res.status == deeppcr.OK
    _, k_ref, ok, hist = oracle.newton_forward_residual(wl.layer, wl.alpha, d["W"], d["bias"],
                                                        d["z0"], 1e-4, 1e-4, 15)
    _say(f"  gpu solves {res.iters} residual {res.residual:.3e}; oracle {k_ref}")
    assert ok and abs(res.iters - k_ref) <= 1
    Zk, _, _, _ = oracle.newton_forward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"], 0.0,
                                        res.iters)
    assert normwise_rel_err(h(res.Z), Zk) <= TOL


@pytest.mark.parametrize("w,L,B", [(4, 16, 1), (8, 300, 2), (16, 200, 3), (64, 40, 2),
                                   (17, 50, 2)])
def test_forward_residual_rule_zero_solves(dev, w, L, B):
    d = synth.mlp_inputs(B, L, w, seed=950 + w)
    res = _forward_res(d, dev, 0, 1.0, atol=1e9)
    assert res.status == deeppcr.OK and res.iters == 0
    Z0 = oracle.initial_guess(0, 1.0, *(d[k].astype(np.float64) for k in ("W", "bias", "z0")))
    assert normwise_rel_err(h(res.Z), Z0) <= 1e-6
    # warm start at the root: the start already meets the threshold, Z is untouched
    ref = oracle.seq_forward(0, 1.0, d["W"], d["bias"], d["z0"]).astype(np.float32)
    res = _forward_res(d, dev, 0, 1.0, atol=1e-4, rtol=0.0, Z_init=g(ref, dev))
    assert res.status == deeppcr.OK and res.iters == 0 and res.residual <= 1e-4
    assert np.array_equal(h(res.Z), ref)


@pytest.mark.parametrize("w,L,B", [(4, 16, 1), (16, 200, 3), (64, 40, 2), (17, 50, 2)])
def test_forward_residual_rule_max_iter(dev, w, L, B):
    d = synth.mlp_inputs(B, L, w, seed=960 + w)
    res = _forward_res(d, dev, 0, 1.0, atol=0.0, rtol=0.0, max_iter=2)
    assert res.status == deeppcr.ENOCONV and res.iters == 2
    Z2, _, _, _ = oracle.newton_forward(0, 1.0, d["W"], d["bias"], d["z0"], 0.0, 2)
    assert normwise_rel_err(h(res.Z), Z2) <= TOL


@pytest.mark.parametrize("w,L,B", [(4, 16, 1), (16, 200, 3), (64, 40, 2)])
def test_forward_residual_rule_non_finite(dev, w, L, B):
    d = dict(synth.mlp_inputs(B, L, w, seed=970 + w))
    d["bias"] = d["bias"].copy()
    d["bias"][3, 1] = np.nan
    res = _forward_res(d, dev, 0, 1.0)
    assert res.status == deeppcr.ENONFINITE and res.iters == 0

# ------------------------------------------------------------------ backward
def _backward_check(d, Z32, dev, layer, alpha, tol=TOL):
    lam, dz0, dW, db = deeppcr.deeppcr_mlp_backward(g(d["W"], dev), g(d["bias"], dev),
                                                    g(d["z0"], dev), g(Z32, dev), g(d["G"], dev),
                                                    layer=layer, alpha=alpha)
    rl, rz, rW, rb = oracle.seq_backward(layer, alpha, d["W"], d["bias"], d["z0"], Z32, d["G"])
    errs = (adjoint_err(h(lam), h(dz0), rl, rz),
            normwise_rel_err(h(dW), rW, axes="all"), normwise_rel_err(h(db), rb, axes="all"))
    _say(f"  backward errs adjoints {errs[0]:.2e} dW {errs[1]:.2e} db {errs[2]:.2e}")
    assert max(errs) <= tol
    _per_layer_check(h(lam), h(dW), h(db), rl, rW, rb, tol)


def _per_layer_check(lam, dW, db, rl, rW, rb, tol=TOL):
    """The same bound layer by layer, on every layer whose reference norm is
    at least 1e-6 of the largest (adjoints per system and layer; dW and db
    per layer), so that an error confined to early layers, whose adjoints
    are orders of magnitude below the last ones, does not pass unseen."""
    el, il = per_layer_rel_err(lam, rl, layer_axis=1)
    eW, iW = per_layer_rel_err(dW, rW, layer_axis=0)
    eb, ib = per_layer_rel_err(db, rb, layer_axis=0)
    _say(f"  worst layer: adjoints {el:.2e} at (b, l) {il}, dW {eW:.2e} at l {iW[0]}, "
         f"db {eb:.2e} at l {ib[0]}")
    assert max(el, eW, eb) <= tol


def adjoint_err(lam, dz0, rl, rz):
    """Normwise error per system over the whole adjoint vector of Eq. 12,
    [dLoss/dz0, dLoss/dZ_0, ..., dLoss/dZ_{L-1}].  In a deep tanh MLP the
    adjoints of early layers decay below the float32 range (1e-200 at
    L = 1024), so they are judged against the size of the whole vector."""
    return normwise_rel_err(np.concatenate([dz0[:, None], lam], 1),
                            np.concatenate([rz[:, None], rl], 1))


@pytest.mark.parametrize("w,L,B", [(1, 1, 1), (2, 2, 3), (4, 16, 1), (3, 37, 4), (16, 100, 3),
                                   (33, 65, 2), (64, 30, 3), (128, 17, 2),
                                   (32, 2, 2), (32, 3, 2), (32, 4, 3), (32, 5, 2), (32, 9, 2),
                                   (64, 3, 2), (128, 5, 2)])
@pytest.mark.parametrize("layer,alpha", [(0, 1.0), (1, 0.1)])
def test_backward_shapes(dev, w, L, B, layer, alpha):
    _say(f"backward shapes w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=500 + w + L)
    Z32 = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"]).astype(np.float32)
    _backward_check(d, Z32, dev, layer, alpha)


# The transposed solve at the same kinds of shapes; at w = 32 also a few rows
# per chunk, less than the rows requested ahead (L = 17 and 33).
@pytest.mark.parametrize("w,L,B", [(64, 130, 40), (64, 300, 8), (128, 203, 16), (32, 130, 64),
                                   (32, 300, 40), (32, 17, 128), (32, 33, 64)])
@pytest.mark.parametrize("layer,alpha", ALL_KINDS)
def test_backward_tile_segments(dev, w, L, B, layer, alpha):
    _say(f"backward tile segments w={w} L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=1200 + w + L + layer)
    Z32 = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"]).astype(np.float32)
    _backward_check(d, Z32, dev, layer, alpha)


def test_backward_mlp_workload(dev):
    wl = synth.WORKLOADS["mlp_bwd"]
    _say(f"mlp backward B={wl.B} L={wl.L} w={wl.w}")
    d = synth.workload_inputs(wl)
    Z32 = oracle.seq_forward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"]).astype(np.float32)
    _backward_check(d, Z32, dev, wl.layer, wl.alpha)


def test_residual_forward_then_backward_workload(dev):
    """GPU forward feeds GPU backward; compared with the oracle's sequential
    forward followed by its backward."""
    wl = synth.WORKLOADS["resnet_fwd_bwd"]
    _say(f"residual fwd+bwd B={wl.B} L={wl.L} w={wl.w}")
    d = synth.workload_inputs(wl)
    res = _forward(d, dev, wl.layer, wl.alpha, wl.tol, wl.max_iter)
    assert res.status == deeppcr.OK
    lam, dz0, dW, db = deeppcr.deeppcr_mlp_backward(g(d["W"], dev), g(d["bias"], dev),
                                                    g(d["z0"], dev), res.Z, g(d["G"], dev),
                                                    layer=wl.layer, alpha=wl.alpha)
    Zref = oracle.seq_forward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"])
    rl, rz, rW, rb = oracle.seq_backward(wl.layer, wl.alpha, d["W"], d["bias"], d["z0"], Zref,
                                         d["G"])
    errs = (normwise_rel_err(h(res.Z), Zref), adjoint_err(h(lam), h(dz0), rl, rz),
            normwise_rel_err(h(dz0), rz), normwise_rel_err(h(dW), rW, axes="all"),
            normwise_rel_err(h(db), rb, axes="all"))
    _say("  errs Z %.2e adjoints %.2e dz0 %.2e dW %.2e db %.2e" % errs)
    assert max(errs) <= TOL
    _per_layer_check(h(lam), h(dW), h(db), rl, rW, rb)
    k_ref = NEWTON_COUNTS[wl.name]["solves"]
    _say(f"  gpu iters {res.iters}, oracle {k_ref}")
    assert abs(res.iters - k_ref) <= 1


# w = 64 with B >= 16 and 513 <= L <= 1024, forward (with the Newton update) and
# backward; residual layers keep the adjoints of early layers in range, so
# every layer is compared.
@pytest.mark.parametrize("L,B", [(1000, 16), (600, 20)])
def test_w64_six_level_tail_forward(dev, L, B):
    w, layer, alpha = 64, 1, 0.1
    _say(f"w=64 six-level tail forward L={L} B={B}")
    d = synth.mlp_inputs(B, L, w, seed=3100 + L)
    res = _forward(d, dev, layer, alpha)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    err = normwise_rel_err(h(res.Z), ref)
    e1, i1 = per_layer_rel_err(h(res.Z), ref, layer_axis=1)
    _say(f"  err {err:.2e}, worst layer {e1:.2e} at {i1}; gpu iters {res.iters}")
    assert err <= TOL and e1 <= TOL


@pytest.mark.parametrize("L,B,layer,alpha", [(1000, 16, 1, 0.1), (600, 20, 3, 0.2),
                                             (1024, 16, 0, 1.0)])
def test_w64_six_level_tail_backward(dev, L, B, layer, alpha):
    w = 64
    _say(f"w=64 six-level tail backward L={L} B={B} layer={layer}")
    d = synth.mlp_inputs(B, L, w, seed=3200 + L + layer)
    Z32 = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"]).astype(np.float32)
    _backward_check(d, Z32, dev, layer, alpha)


@pytest.mark.parametrize("transpose", [1, 0])
def test_pcr_solve_w64_six_level_tail(dev, transpose):
    B, L, w = 16, 1024, 64
    _say(f"pcr solve w=64 B={B} L={L} transpose={transpose}")
    d = synth.random_system(B, L, w, seed=3300 + transpose, scale=0.9)
    x = h(deeppcr.pcr_solve_block_bidiag(g(d["J"], dev), g(d["r"], dev), transpose=transpose))
    ref = oracle.seq_solve(d["J"], d["r"], bool(transpose))
    err = normwise_rel_err(x, ref)
    e1, i1 = per_layer_rel_err(x, ref, layer_axis=1)
    _say(f"  err {err:.2e}, worst row {e1:.2e} at {i1}")
    assert err <= TOL and e1 <= TOL


def test_backward_deterministic(dev):
    d = synth.mlp_inputs(6, 50, 16, seed=13)
    Z32 = oracle.seq_forward(0, 1.0, d["W"], d["bias"], d["z0"]).astype(np.float32)
    args = [g(d[k], dev) for k in ("W", "bias", "z0")] + [g(Z32, dev), g(d["G"], dev)]
    a = [h(t) for t in deeppcr.deeppcr_mlp_backward(*args)]
    b = [h(t) for t in deeppcr.deeppcr_mlp_backward(*args)]
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_workspace_too_small_is_rejected(dev):
    d = synth.random_system(1, 8, 4, seed=1)
    ws = torch.empty(16, dtype=torch.uint8, device=dev)
    with pytest.raises(deeppcr.DeepPCRError, match="workspace"):
        deeppcr.pcr_solve_block_bidiag(g(d["J"], dev), g(d["r"], dev), workspace=ws)


# ------------------------------------------------------- sequential baseline
# one wave per system (w = 2 .. 32; forward also 64), the streamed workgroup
# kernels (w = 64 backward, 128) and the generic one (33); walks shorter than
# the weight ring and walks ending in a partial trip of it
@pytest.mark.parametrize("w,L,B", [(4, 50, 3), (16, 300, 2), (33, 40, 2), (128, 20, 2),
                                   (32, 70, 2), (64, 33, 3), (32, 3, 2), (128, 3, 1),
                                   (2, 37, 2), (8, 65, 3), (8, 2, 1)])
@pytest.mark.parametrize("layer,alpha", [(0, 1.0), (3, 0.1), (4, 1.0)])
@pytest.mark.parametrize("per_layer", [False, True])
def test_sequential_passes(dev, w, L, B, layer, alpha, per_layer):
    _say(f"sequential w={w} L={L} B={B} layer={layer} per_layer={per_layer}")
    d = synth.mlp_inputs(B, L, w, seed=900 + w + L)
    t = {k: g(v, dev) for k, v in d.items()}
    Z = deeppcr.deeppcr_seq_forward(t["W"], t["bias"], t["z0"], layer=layer, alpha=alpha,
                                    launch_per_layer=per_layer)
    ref = oracle.seq_forward(layer, alpha, d["W"], d["bias"], d["z0"])
    assert normwise_rel_err(h(Z), ref) <= TOL
    Z32 = ref.astype(np.float32)
    lam, dz0 = deeppcr.deeppcr_seq_backward(t["W"], t["bias"], t["z0"], g(Z32, dev), t["G"],
                                            layer=layer, alpha=alpha, launch_per_layer=per_layer)
    rl, rz, _, _ = oracle.seq_backward(layer, alpha, d["W"], d["bias"], d["z0"], Z32, d["G"])
    assert adjoint_err(h(lam), h(dz0), rl, rz) <= TOL
