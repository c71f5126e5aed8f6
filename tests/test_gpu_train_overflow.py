"""A hidden gradient that overflows to infinity, in one row of the batch: the weight gradient formed from it is what
the fp32 sum of products gives, infinite with the product's sign wherever the row's code is not zero, and NaN
only where it is (0 x Inf).  The kernels split fp32 gradients into bf16 parts; an infinity's lower parts must not
turn the whole gradient into NaN.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import random_qat_params  # noqa: E402
from workloads.codes import hamming_7_4  # noqa: E402
from tests.test_gpu_train import _dev, _to_dev  # noqa: E402


@pytest.mark.parametrize("d", [32, 64, 128])
def test_infinite_hidden_gradient(d):
    import oracle.qat as Q
    import paper_2410_05911_amd as P
    H = hamming_7_4()
    m, n = H.shape
    p = random_qat_params(n, m, d, 1, seed=d)
    # the hidden row near 1e-33, brought back by a second map of scale near 1e33, whose backward takes dR2
    # (1e8 by the head) past the largest fp32; only token 2's row has a gradient
    p["w"]["ff1"] *= np.float32(1e-33)
    p["b"]["ff1"] = (1e-33 * np.random.default_rng(d).standard_normal((1, 4 * d))).astype(np.float32)
    p["w"]["ff2"] *= np.float32(1e33)
    p["head_w1"] = (1e9 * p["head_w1"]).astype(np.float32)
    p["head_wo"][np.arange(n + m) != 2] = 0.0
    y = np.array([[0.9, -0.8, 1.1, 0.7, -1.2, 0.6, 1.0]], np.float32)
    print(f"[overflow] d {d}", flush=True)
    with np.errstate(over="ignore"):   # logits of 1e8
        _, _, g64 = Q.forward_backward(H, p, y, None, heads=8, aap_eps=0.0)
    tr = P.Trainer(H, d, 1, heads=8, aap_eps=0.0)
    loss, g = tr.grad(_to_dev(p), _dev(y))
    torch.cuda.synchronize()
    w, b = g["w"]["ff1"][0].cpu().numpy(), g["b"]["ff1"][0].cpu().numpy()
    w64, b64 = g64["w"]["ff1"][0], g64["b"]["ff1"][0]
    assert np.isfinite(loss.item())
    over = np.abs(b64) > 2 * float(np.finfo(np.float32).max)   # the row's hidden gradient in 64 bits
    assert over.sum() > d // 4 and np.array_equal(np.isinf(b[over]), np.ones(over.sum(), bool))
    assert np.array_equal(np.sign(b[over]), np.sign(b64[over]))
    code = (w64[:, over] != 0).any(1)                          # inputs whose code is not zero
    assert code.sum() > d // 2
    assert np.isinf(w[code][:, over]).all()
    assert np.array_equal(np.sign(w[code][:, over]), np.sign(w64[code][:, over]))
    tr.close()
