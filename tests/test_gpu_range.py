"""The chunked MLP solve (widths 17 to 128) at the ends of the float32 range:
its products carry a value by three bf16 parts, which add up to it only in a
part of that range.  Against what IEEE arithmetic gives for the recurrence, the
same call at an ordinary scale, and the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2309_16318_amd import deeppcr, synth
from tests._util import normwise_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WIDTHS = [17, 32, 47, 64, 100, 128]


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def row_errors(got, ref, least=0.0):
    """max |got - ref| over max |ref|, per system and row, where that is at
    least `least`."""
    den = np.max(np.abs(ref), axis=-1)
    num = np.max(np.abs(got.astype(np.float64) - ref), axis=-1)
    return np.where(den >= least, num / np.where(den > 0, den, 1.0), 0.0)


class Net:
    def __init__(self, dev, w, B, L, layer, alpha=1.0, seed=0, edit=None):
        self.dev, self.layer, self.alpha = dev, layer, alpha
        self.d = synth.mlp_inputs(B, L, w, seed=seed + 31 * w + B + L)
        if edit:
            edit(self.d)
        self.Z = oracle.seq_forward(layer, alpha, self.d["W"], self.d["bias"],
                                    self.d["z0"]).astype(np.float32)

    def run(self, G):
        """[dz0; Lambda] and the weight gradient."""
        t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(self.dev)
             for a in (self.d["W"], self.d["bias"], self.d["z0"], self.Z, G)]
        lam, dz0, dW, _ = deeppcr.deeppcr_mlp_backward(*t, layer=self.layer, alpha=self.alpha)
        return torch.cat([dz0[:, None], lam], 1).cpu().numpy(), dW.cpu().numpy()

    def oracle(self, G):
        lam, dz0, _, _ = oracle.seq_backward(self.layer, self.alpha, self.d["W"], self.d["bias"],
                                             self.d["z0"], self.Z, G)
        return np.concatenate([dz0[:, None], lam], 1)


@pytest.mark.parametrize("w", WIDTHS)
@pytest.mark.parametrize("layer", [0, 1])
def test_infinite_cotangent(dev, w, layer):
    """One infinite element: infinities of the signs of its column of the first
    Jacobian, then no numbers; the other systems are untouched."""
    print(f"range: infinite w={w} layer={layer}", flush=True)
    n = Net(dev, w, 3, 40, layer, alpha=0.5)
    G = n.d["G"].copy()
    clean, _ = n.run(G)
    G[1, 5] = -np.inf
    got, _ = n.run(G)
    for b in (0, 2):
        assert np.array_equal(got[b], clean[b])
    assert np.array_equal(got[1, 40], G[1])
    first = -np.inf * n.d["W"][39, 5].astype(np.float64)  # d > 0
    if layer == 1:
        with np.errstate(invalid="ignore"):
            first = first + G[1]
    assert np.array_equal(got[1, 39], first.astype(np.float32), equal_nan=True)
    assert not np.isfinite(got[1, 38]).any()


@pytest.mark.parametrize("w", WIDTHS)
def test_largest_values(dev, w):
    """Values that round up to an infinity in bf16 but are none, at active
    units, whose slope is 1."""
    print(f"range: largest w={w}", flush=True)
    n = Net(dev, w, 3, 24, 4)
    G = (n.d["G"] * 1e36).astype(np.float32)
    for b in range(3):
        on = np.flatnonzero(n.Z[b, -1] > 0)
        G[b, on[0]] = 3.401e38
        G[b, on[-1]] = -3.395e38
    got, _ = n.run(G)
    ref = n.oracle(G)
    assert np.abs(ref[:, :-1]).max() < 3e38
    # 24 rows of at most w 2^-24 of their terms' norm each
    assert normwise_rel_err(got, ref) <= 24 * w * 2.0 ** -24


@pytest.mark.parametrize("w,B", [(17, 3), (17, 1), (32, 3), (47, 40), (64, 5), (100, 1), (128, 3)])
@pytest.mark.parametrize("layer", [0, 1])
def test_small_cotangent(dev, w, B, layer):
    """A cotangent of 2^-118: the adjoints are linear in it, and scaling by a
    power of two commutes with every rounding of a normal number.  What falls
    below 2^-126 on the way is rounded to 2^-150, in each of a row's w terms:
    2^-32 of a residual network's adjoints, over its 150 rows; 2^-27 of the
    smallest rows looked at without residuals, of which 16 are near."""
    print(f"range: small cotangent w={w} B={B} layer={layer}", flush=True)
    n = Net(dev, w, B, 150, layer, alpha=0.3)
    G = n.d["G"]
    ref, refW = n.run(G)
    got, gotW = n.run(G * np.float32(2.0 ** -118))
    tol = w * (150 * 2.0 ** -32 if layer == 1 else 16 * 2.0 ** -27)
    err = np.max(row_errors(got * 2.0 ** 118, ref.astype(np.float64), 2.0 ** -5))
    errW = np.max(np.abs(gotW * 2.0 ** 118 - refW)) / np.max(np.abs(refW))
    print(f"  err {err:.1e} dW {errW:.1e} tol {tol:.1e}", flush=True)
    assert max(err, errW) <= tol


def orthogonal_net(scales, w, B):
    """Layers a Haar orthogonal matrix times a power of two each, at the fixed
    point zero, where the slope of tanh is 1: every product of Jacobians is
    perfectly conditioned."""
    rng = np.random.default_rng(w)
    L = len(scales)
    W = np.ascontiguousarray(synth.haar_orthogonal(rng, (L,), w)).astype(np.float32)
    W *= np.exp2(scales)[:, None, None].astype(np.float32)

    def edit(d):
        d["W"], d["bias"], d["z0"] = W, np.zeros((L, w), np.float32), np.zeros((B, w), np.float32)
    return edit


def wave(first, step, half, L):
    """Exponents first, first, ... for `half` layers, then -first, ..."""
    return np.array([step * (first if (l // half) % 2 == 0 else -first) for l in range(L)], float)


WEIGHTS = {"down": wave(1, 5, 23, 322), "up": wave(-1, 5, 24, 336),
           "far": wave(-1, 24, 5, 320), "layers": np.array([-118.0, 118.0] * 3 + [0.0] * 90)}


@pytest.mark.parametrize("name", WEIGHTS)
@pytest.mark.parametrize("w,B", [(17, 1), (17, 40), (32, 2), (47, 1), (64, 3), (100, 1), (100, 20),
                                 (128, 2)])
def test_products_across_the_range(dev, w, B, name):
    """Jacobian products that sink to 2^-120, or rise to 2^120, and come back,
    over many layers or between two (weights of 2^-118 and 2^118)."""
    print(f"range: products w={w} B={B} {name}", flush=True)
    scales = WEIGHTS[name]
    n = Net(dev, w, B, len(scales), 0, edit=orthogonal_net(scales, w, B))
    got, _ = n.run(n.d["G"])
    err = np.max(row_errors(got, n.oracle(n.d["G"])))
    print(f"  err {err:.1e}", flush=True)
    # a row's sum of w terms errs by sqrt(w) 2^-24 of their norm at most; the
    # rows' errors add up without growing
    assert err <= len(scales) * np.sqrt(w) * 2.0 ** -24


@pytest.mark.parametrize("w,B", [(9, 3), (16, 2), (17, 1), (32, 2), (47, 20), (64, 3), (100, 1),
                                 (128, 2)])
@pytest.mark.parametrize("layer", [0, 4])
def test_small_states(dev, w, B, layer):
    """A network whose states are about 2^-118."""
    print(f"range: small states w={w} B={B} layer={layer}", flush=True)
    d = {}
    orthogonal_net(np.full(60, 0.25 if layer == 4 else 0.0), w, B)(d)
    z0 = np.abs(synth.mlp_inputs(B, 1, w, seed=w)["z0"]) * np.float32(2.0 ** -118)
    if layer == 4:
        d["W"] = np.abs(d["W"]) / np.sqrt(w).astype(np.float32)
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev)
         for a in (d["W"], d["bias"], z0)]
    res = deeppcr.deeppcr_mlp_forward(*t, layer=layer)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(layer, 1.0, d["W"], d["bias"], z0)
    err = np.max(row_errors(res.Z.cpu().numpy(), ref, 2.0 ** -122))
    print(f"  err {err:.1e}", flush=True)
    assert err <= 60 * np.sqrt(w) * 2.0 ** -24


@pytest.mark.parametrize("w", [9, 16] + WIDTHS)
def test_infinite_state_saturates(dev, w):
    """An infinite input, and one of 3.4e38, through the layer evaluation: the
    activation is 1 there, as of a plain sum, and the layers after it see that."""
    print(f"range: infinite state w={w}", flush=True)
    d = synth.mlp_inputs(3, 30, w, seed=w)
    z0, W = d["z0"].copy(), d["W"].copy()
    z0[1, w - 1], z0[2, 3] = np.inf, 3.4e38
    W[0, :, w - 1] = np.abs(W[0, :, w - 1]) + 0.1
    W[0, :, 3] = np.abs(W[0, :, 3]) + 0.1
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev)
         for a in (W, d["bias"], z0)]
    res = deeppcr.deeppcr_mlp_forward(*t)
    assert res.status == deeppcr.OK
    Z = res.Z.cpu().numpy()
    assert np.all(Z[1:, 0] == 1.0)
    ref = oracle.seq_forward(0, 1.0, W[1:], d["bias"][1:], np.ones((1, w), np.float32))
    assert np.max(np.abs(Z[1:, 1:] - ref)) <= 4 * w * 2.0 ** -24
