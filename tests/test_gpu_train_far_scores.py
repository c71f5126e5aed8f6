"""A key whose attention score overflows to minus infinity takes no part in its rows' softmax, wherever it stands
in a row's list and however the list is dealt to lanes; rows whose other keys have finite scores stay finite.

One variable's key is put along the direction that every query points away from, far enough that the fp32 score
is -Inf; all other scores are exactly 0.  The forward pass and the gradients behind the attention are compared
with the float64 oracle (where that score is about -1e40).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import random_qat_params, regular_ldpc_3_6  # noqa: E402
from workloads.codes import hamming_7_4  # noqa: E402
from tests.test_gpu_train import FLIP, _dev, _rel, _to_dev  # noqa: E402


@pytest.mark.parametrize("n,d,far", [(7, 32, 6), (7, 64, 6), (7, 128, 6), (66, 32, 1), (66, 64, 30), (66, 128, 65),
                                     (1024, 32, 700)])
def test_minus_infinite_scores(n, d, far):
    import oracle.qat as Q
    import paper_2410_05911_amd as P
    H = hamming_7_4() if n == 7 else regular_ldpc_3_6(n, seed=1000 + n)
    m = H.shape[0]
    p = random_qat_params(n, m, d, 1, seed=n + d)
    # inputs: equal features (codes 127) but for token `far`, whose odd features are 0; the key map adds the even
    # features and subtracts the odd ones, times 1e20: a key of exactly 0, or of about 1e21; queries near -1e20
    p["embed"][:] = 1.0
    p["embed"][far, 1::2] = 0.0
    p["w"]["k"][:] = np.where(np.arange(d) % 2 == 0, 1e20, -1e20).astype(np.float32)[None, :, None]
    p["delta"][:, 1] = 1.0
    p["b"]["k"][:] = 0.0
    p["b"]["q"][:] = -1e20
    y = (1.0 + 0.3 * np.random.default_rng(n).standard_normal((2, n))).astype(np.float32)
    print(f"[far] n {n} d {d} token {far}", flush=True)
    loss64, _, g64 = Q.forward_backward(H, p, y, None, heads=8)
    assert np.isfinite(loss64)
    tr = P.Trainer(H, d, 1, heads=8)
    loss, g = tr.grad(_to_dev(p), _dev(y))
    torch.cuda.synchronize()
    errs = {"w_" + k: _rel(g["w"][k].cpu().numpy(), g64["w"][k]) for k in ("v", "o", "ff1", "ff2")}
    for k in ("ln1_g", "ln1_b", "ln2_g", "ln2_b", "head_w1", "head_wo", "head_bo"):
        errs[k] = _rel(g[k].cpu().numpy(), g64[k])
    print(" ".join(f"{k}={v:.1e}" for k, v in sorted(errs.items())), flush=True)
    # FLIP: a rounding decision of fp32 that falls the other way shifts the rest of its word by a code step
    assert abs(loss.item() - loss64) <= FLIP[1] * abs(loss64)
    assert all(v <= FLIP[0] for v in errs.values()), errs
    tr.close()
