"""MLP solves of more values than 32-bit byte addresses reach (2^30): widths of
both chunked forms, in several launches.  100 different systems, repeated, all
of which must give the first ones' results; those against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2309_16318_amd import deeppcr, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("w,L", [(9, 1000), (17, 500)])
def test_beyond_32_bit_addresses(w, L):
    dev = torch.device("cuda:0")
    n = (2 ** 30 // (L * w) // 100 + 2) * 100
    B = n + n % 16  # (and no whole number of groups in the last launch)
    free = torch.cuda.mem_get_info()[0]
    need = deeppcr.workspace_bytes(deeppcr.OP_BWD, B, L, w) + 4 * 4 * B * L * w
    print(f"batches: w={w} L={L} B={B}, {need / 2 ** 30:.0f} GiB", flush=True)
    if need > 0.9 * free:
        pytest.skip(f"needs {need / 2 ** 30:.0f} GiB of device memory")
    assert B * L * w > 2 ** 30
    d = synth.mlp_inputs(100, L, w, seed=w)
    W, bias = (torch.from_numpy(d[k]).to(dev) for k in ("W", "bias"))
    z0, G = (torch.from_numpy(d[k]).to(dev).repeat(B // 100 + 1, 1)[:B].contiguous()
             for k in ("z0", "G"))
    ws = torch.empty(deeppcr.workspace_bytes(deeppcr.OP_BWD, B, L, w), dtype=torch.uint8,
                     device=dev)
    # per row at most w 2^-24 of its terms' norm; 4 rows of it add up before it fades
    tol = 4 * w * 2.0 ** -24

    def check(x, ref, of=None):
        k = B // 100
        head = x[:100 * k].view(k, 100, *x.shape[1:])
        assert all(bool((head[i] == head[0]).all()) for i in range(k))
        assert bool((x[100 * k:] == x[:B - 100 * k]).all())
        got = x[:100].cpu().numpy()
        scale = np.abs(ref if of is None else of).reshape(100, -1).max(axis=1)
        assert np.all(np.abs(got - ref).reshape(100, -1).max(axis=1) <= tol * scale)

    res = deeppcr.deeppcr_mlp_forward(W, bias, z0, layer=0, workspace=ws)
    assert res.status == deeppcr.OK
    ref = oracle.seq_forward(0, 1.0, d["W"], d["bias"], d["z0"])
    check(res.Z, ref)
    lam, dz0, dW, db = deeppcr.deeppcr_mlp_backward(W, bias, z0, res.Z, G, layer=0, workspace=ws)
    rl, rz, _, _ = oracle.seq_backward(0, 1.0, d["W"], d["bias"], d["z0"],
                                       res.Z[:100].cpu().numpy(), d["G"])
    check(lam, rl)
    check(dz0, rz, of=rl)  # (1000 layers on, it is zero)
    assert bool(torch.isfinite(dW).all()) and bool(torch.isfinite(db).all())
    del ws, res, lam, z0, G
    torch.cuda.empty_cache()
