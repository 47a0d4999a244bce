"""GPU parity of the width-16 ResNet blocks where a wave takes 8 systems:
sizes on both sides of the rule, a last group that is not full, one to four
layers per block, every activation.  Against the CPU oracle.

Tolerance: a float32 product of 16 terms is within 16 2^-24 of its terms'
norm; the skips carry it through up to 260 layers, where independent errors
add as the root of their number, 16, and 64 of them are allowed for, relative
to the largest entry (as normwise_rel_err measures)."""
import numpy as np
import pytest

from oracle import resnet_oracle as R
from paper_2309_16318_amd import deeppcr, synth
from tests._util import normwise_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 64 * 16 * 2.0 ** -24

# (B, blocks, skip, activation); depths at which Newton converges from the
# usual start (a thousand blocks of one layer need more than 20 iterations)
CASES = [(128, 63, 1, R.ACT_TANH), (128, 64, 1, R.ACT_TANH), (65, 127, 2, R.ACT_SIGMOID),
         (129, 64, 3, R.ACT_RELU), (256, 65, 4, R.ACT_TANH), (257, 64, 2, R.ACT_TANH),
         (256, 64, 1, R.ACT_SIGMOID)]


@pytest.mark.parametrize("B,G,skip,act", CASES)
def test_groups(B, G, skip, act):
    print(f"resnet groups B={B} blocks={G} skip={skip} act={act}", flush=True)
    dev = torch.device("cuda:0")
    L = G * skip
    d = synth.resnet_inputs(B, L, 16, seed=5200 + B + G)
    t = {k: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(dev)
         for k, v in d.items()}
    res = deeppcr.deeppcr_resnet_forward(t["W"], t["bias"], t["z0"], skip=skip, act=act)
    assert res.status == deeppcr.OK
    ref = R.resnet_seq_forward(act, skip, d["W"], d["bias"], d["z0"])
    Z32 = ref.astype(np.float32)
    lam, dz0, dW, db = deeppcr.deeppcr_resnet_backward(
        t["W"], t["z0"], torch.from_numpy(Z32).to(dev), t["G"], skip=skip, act=act)
    rl, rz, rW, rb = R.resnet_seq_backward(act, skip, d["W"], d["bias"], d["z0"], Z32, d["G"])
    torch.cuda.synchronize()
    adj = np.concatenate([dz0.cpu().numpy()[:, None], lam.cpu().numpy()], 1)
    errs = [normwise_rel_err(res.Z.cpu().numpy(), ref),
            normwise_rel_err(adj, np.concatenate([rz[:, None], rl], 1)),
            normwise_rel_err(dW.cpu().numpy(), rW, axes="all"),
            normwise_rel_err(db.cpu().numpy(), rb, axes="all")]
    print("  errors", " ".join(f"{e:.1e}" for e in errs), flush=True)
    assert max(errs) <= TOL


@pytest.mark.parametrize("B,G", [(3, 12), (1, 40), (256, 64)])
@pytest.mark.parametrize("skip", [1, 2, 4])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_weight_that_is_no_number(B, G, skip, bad):
    """The adjoints are finite exactly where the plain backward pass has them
    finite: a NaN or infinite weight reaches the one element of its column in
    its own layer, and all of the layers before."""
    print(f"resnet {bad} weight B={B} blocks={G} skip={skip}", flush=True)
    dev = torch.device("cuda:0")
    L = G * skip
    d = synth.resnet_inputs(B, L, 16, seed=5300 + B + G)
    Z32 = R.resnet_seq_forward(R.ACT_TANH, skip, d["W"], d["bias"], d["z0"]).astype(np.float32)
    for layer in range((G // 2) * skip, (G // 2 + 1) * skip):  # every place of a block
        W = d["W"].copy()
        W[layer, 13, 2] = bad
        t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev)
             for a in (W, d["z0"], Z32, d["G"])]
        lam, dz0, _, _ = deeppcr.deeppcr_resnet_backward(*t, skip=skip, act=R.ACT_TANH)
        with np.errstate(invalid="ignore"):
            rl, rz, _, _ = R.resnet_seq_backward(R.ACT_TANH, skip, W, d["bias"], d["z0"], Z32,
                                                 d["G"])
        assert np.array_equal(np.isfinite(lam.cpu().numpy()), np.isfinite(rl)), layer
        assert np.array_equal(np.isfinite(dz0.cpu().numpy()), np.isfinite(rz)), layer
