"""Hidden rows that are almost wholly inactive: every pre-activation of the first feed-forward map is strongly
negative but for a few that are barely positive.  Eq. 2 then divides by an alpha hundreds of times smaller
than the values that the ReLU drops, so a code formed before the ReLU (f 127 / alpha, here down to about
-10^5) leaves the range of a 16-bit code; the dropped units still have to get code 0.

Every form of the map is run: decodes against the CPU oracle, bit for bit (the fused kernel with one wavefront
a word and a word's tiles over wavefronts; the token block with a strip a wavefront and a strip a block; one
alpha per word in stages and as separate kernels), and a training step against the float64 oracle.  A
wrong code stands for up to 127 of the small alpha steps and would change the second map's output in the third
digit and its weight gradient by its whole size.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import bch_31_16, hamming_7_4, random_qat_params, random_weights, regular_ldpc_3_6  # noqa: E402
from tests.test_gpu_train import FLIP, KINDS, _dev, _rel, _to_dev  # noqa: E402


def _sleep(b, rng):
    """FF1 biases [N][d_ff]: -0.5 .. -4, one unit in sixteen at 0.004."""
    b[:] = -np.exp(rng.uniform(np.log(0.5), np.log(4.0), b.shape)).astype(np.float32)
    b[:, ::16] = 0.004


def _model(n, m, d, heads=8, **kw):
    w = random_weights(n, m, d, 2, heads, seed=n + d, **kw)
    _sleep(w.b["ff1"], np.random.default_rng(n))
    w.scale[:, 4] = 0.001 / np.sqrt(d)     # a spread of about 0.001 around the biases
    w.scale[:, 5] = 50.0                   # what is left of the hidden row counts in the residual
    return w


def _wrapped(om, y):
    """Tokens whose least code before the ReLU is below -32768, by the oracle's own intermediate values."""
    _, _, t = om.decode_taps(y)
    w = om.w
    low = 0
    for l in range(w.n_layers):
        sc = t["a1"][l][:, None] * (w.scale[l, 4] / np.float32(127.0))
        f = t["acc_ff1"][l] * sc + w.b["ff1"][l]
        ag = t["ag"][l]
        low += int(((f.min(1) * 127.0 < -32768.0 * ag) & (ag > 0)).sum())
    return low


@pytest.mark.parametrize("n,d,heads,batch,act_scale,form", [
    (7, 32, 8, 40, "token", -1),        # fused, one tile
    (31, 32, 8, 30, "token", -1),       # fused, a word's three tiles over wavefronts
    (31, 32, 8, 1500, "token", -1),     # fused, a word a wavefront
    (31, 32, 8, 30, "token", 0),        # layered, separate kernels
    (66, 64, 8, 3, "token", -1),        # token block, a strip a block
    (66, 64, 8, 1000, "token", -1),     # token block, a strip a wavefront
    (66, 128, 8, 3, "token", -1),
    (66, 128, 8, 1000, "token", -1),
    (66, 64, 8, 5, "word", -1),         # one alpha per word, in stages
    (66, 64, 8, 5, "word", 0),          # one alpha per word, separate kernels
    (66, 128, 8, 5, "word", -1),
    (66, 128, 8, 5, "word", 0),
    (31, 32, 8, 30, "word", -1),
])
def test_decode_with_inactive_hidden_rows(oracle_mod, n, d, heads, batch, act_scale, form):
    import paper_2410_05911_amd as P
    H = hamming_7_4() if n == 7 else bch_31_16() if n == 31 else regular_ldpc_3_6(n, seed=1000 + n)
    m = H.shape[0]
    print(f"[inactive] n {n} d {d} batch {batch} alpha per {act_scale} form {form}", flush=True)
    w = _model(n, m, d, heads, act_scale=act_scale)
    rng = np.random.default_rng(n + batch)
    y = (1.0 + 0.7 * rng.standard_normal((batch, n))).astype(np.float32)
    om = oracle_mod.OracleModel(H, w)
    assert _wrapped(om, y[0]) > 0
    if d == 32 and form == 0:
        dec = P.Decoder(H, w, path=P.PATH_LAYERED)
    else:
        dec = P.Decoder(H, w, layered_attention=form) if form == 0 else P.Decoder(H, w)
    bits, logits = dec.decode(_dev(y))
    torch.cuda.synchronize()
    idx = np.unique(np.linspace(0, batch - 1, 24).astype(np.int64))
    bo, fo = om.decode(y[idx], n_threads=8)
    assert int((logits.cpu().numpy()[idx] != fo).sum()) == 0
    assert (bits.cpu().numpy()[idx] == bo).all()
    dec.close()


@pytest.mark.parametrize("n,d,batch", [(7, 32, 16), (7, 64, 16), (7, 128, 16)])
def test_train_step_with_inactive_hidden_rows(n, d, batch):
    import oracle.qat as Q
    import paper_2410_05911_amd as P
    H = hamming_7_4()
    m = H.shape[0]
    print(f"[inactive] training n {n} d {d} batch {batch}", flush=True)
    p = random_qat_params(n, m, d, 2, seed=n + d)
    _sleep(p["b"]["ff1"], np.random.default_rng(n))
    p["delta"][:, 4] = 0.0015
    p["delta"][:, 5] = 50.0
    rng = np.random.default_rng(n + batch)
    y = (1.0 + 0.7 * rng.standard_normal((batch, n))).astype(np.float32)
    loss64, _, g64 = Q.forward_backward(H, p, y, None, heads=8)
    tr = P.Trainer(H, d, 2, heads=8)
    loss, g = tr.grad(_to_dev(p), _dev(y))
    torch.cuda.synchronize()
    errs = {"w_" + k: _rel(g["w"][k].cpu().numpy(), g64["w"][k]) for k in KINDS}
    for k in ("embed", "delta", "ln1_g", "ln1_b", "ln2_g", "ln2_b", "head_w1", "head_wo", "head_bo"):
        errs[k] = _rel(g[k].cpu().numpy(), g64[k])
    print(f"loss {loss.item():.6f} vs {loss64:.6f} " + " ".join(f"{k}={v:.1e}" for k, v in sorted(errs.items())), flush=True)
    # FLIP: a rounding decision of fp32 that falls the other way shifts the rest of its word by a code step
    assert abs(loss.item() - loss64) <= FLIP[1] * abs(loss64)
    assert all(v <= FLIP[0] for v in errs.values()), errs
    tr.close()
