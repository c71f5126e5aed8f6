"""The training step's row strips, tiles and row ranges at the sizes where they can go wrong: fewer rows
than a 16-token strip or a wavefront's eight, a last strip that is partly filled, several strips a
wavefront, one layer (the first is the last), more layers than a packing or Eq. 1 launch takes, a
positional table, odd lengths, words on either side of the lines between the attention's two forms.

Against the float64 oracle, normwise.  fp32 rounding alone gives a few 1e-7 (test_gpu_train.py, TIGHT);
an int8 or ternary rounding decision that falls the other way in fp32 shifts the rest of its word by
a code step, up to 1e-2 on batches of tens of words (FLIP there), and a wrong or missing row or tile
moves a gradient by its whole share, above 1 / rows of it (at most 154 rows in the first test, so above
6e-3, and in most of the twenty gradients far above; the 930 and 1536 rows of its long words are one word each,
where a wrong neighbour changes every gradient): the median gradient error has to stay below 1e-3.  The
other tests state their own bounds.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import random_qat_params, regular_ldpc_3_6  # noqa: E402
from workloads.codes import hamming_7_4  # noqa: E402
from tests.test_gpu_train import _dev, _to_dev, _rel  # noqa: E402

KINDS = ("q", "k", "v", "o", "ff1", "ff2")


@pytest.mark.parametrize("n,d,layers,batch,attention,pos", [
    (7, 32, 1, 1, "hpsa", False),      # 10 rows
    (7, 64, 1, 2, "casa", True),       # 20 rows: a strip and a quarter
    (7, 128, 9, 1, "hpsa", True),      # more layers than one launch of the packing (kTrainJobsPerLaunch / 12 = 5)
    (7, 32, 11, 1, "hpsa", True),      # and of Eq. 1 and the delta gradients (kTrainJobsPerLaunch / 6 = 10)
    (7, 128, 2, 13, "hpsa", False),    # 130 rows: two row ranges of the weight gradients
    (66, 32, 2, 1, "hpsa", False),     # 99 rows
    (66, 64, 2, 1, "casa", True),
    (102, 128, 1, 1, "hpsa", True),    # 153 rows
    (1024, 32, 1, 1, "hpsa", False),   # 1536 tokens: the attention's gathers from device memory (above 930,
    (1024, 64, 1, 1, "casa", False),   # 1024 and 1077 tokens at d_h = 4, 8 and 16)
    (1024, 128, 1, 1, "hpsa", True),
    (620, 32, 1, 1, "hpsa", False),    # 930 tokens, one word: the gathers by their measured line
])
def test_train_step_at_awkward_sizes(n, d, layers, batch, attention, pos):
    _step_against_oracle(n, d, layers, batch, attention=attention, pos=pos)


@pytest.mark.parametrize("n,d,heads,repeat", [
    (256, 32, 8, 1),     # 384 tokens at d_h = 4: in LDS in any batch
    (258, 32, 8, 1),     # 387: the gathers in small batches
    (258, 32, 8, 21),    # 126 blocks (two a word): still
    (258, 32, 8, 22),    # 132 blocks: LDS
    (258, 64, 16, 11),   # 132 blocks at d = 64: the gathers
    (620, 32, 8, 22),    # 930 tokens: the longest word in LDS at d_h = 4
    (426, 64, 8, 1),     # 639 tokens at d_h = 8: LDS
    (428, 64, 8, 1),     # 642: the gathers
    (682, 64, 8, 11),    # 1023 tokens, 132 blocks: LDS, rows in four passes
    (640, 128, 8, 1),    # 960 tokens at d_h = 16: LDS
    (642, 128, 8, 1),    # 963: the gathers
    (718, 128, 8, 6),    # 1077 tokens, 144 blocks: the longest word in LDS at d_h = 16, rows in two passes
])
def test_long_words_in_both_attention_forms(n, d, heads, repeat):
    """Either side of each line between the two forms of the attention (on 256 compute units), three words repeated to
    reach the batch: a mean over them, which the oracle takes once.  Words this long have a few codes that fp32
    decides the other way in any batch; a flip shifts its rows by at most a code step, 1 / 127 of the row's maximum,
    so the median error stays below 8e-3.  Rows left out of a last pass (5 % of the longest word's) or staged from a
    wrong token would change it by far more."""
    _step_against_oracle(n, d, 1, 3, heads=heads, repeat=repeat, median=8e-3)


@pytest.mark.parametrize("d,param_seed,word_seed", [(32, 13, 11), (64, 2, 1), (128, 17, 9)])
def test_several_strips_a_wavefront(d, param_seed, word_seed):
    """66030 rows, the last strip partly filled: 4127 strips on 256 compute units give a wavefront of every strip
    kernel (at most two blocks of eight per unit) a second and third one, and the weight gradients their largest
    number of row ranges.  Three words repeated; the seeds are ones whose rounding decisions lie farthest
    from a tie (above 6e-5 code units), so that none flips.  fp32 sums over chains of at most about 1600
    additions are within 1e-4; a strip left out or taken twice is 1 / 4127 = 2.4e-4 of every gradient."""
    errs, loss, loss64 = _errors(7, d, 2, 3, repeat=2201, param_seed=param_seed, word_seed=word_seed)
    assert abs(loss - loss64) <= 1e-4 * abs(loss64)
    assert max(errs.values()) <= 1e-4, errs


def _step_against_oracle(n, d, layers, batch, median=1e-3, **kw):
    errs, loss, loss64 = _errors(n, d, layers, batch, **kw)
    assert abs(loss - loss64) <= 1e-3 * abs(loss64)
    assert np.median(list(errs.values())) <= median and max(errs.values()) <= 5e-2, errs


def _errors(n, d, layers, batch, heads=8, attention="hpsa", pos=False, repeat=1, param_seed=None, word_seed=None):
    import oracle.qat as Q
    import paper_2410_05911_amd as P
    H = hamming_7_4() if n == 7 else regular_ldpc_3_6(n, seed=1000 + n)
    m = H.shape[0]
    print(f"[train] n {n} d {d} heads {heads} layers {layers} batch {batch} x {repeat} {attention}", flush=True)
    p = random_qat_params(n, m, d, layers, seed=n + d + layers if param_seed is None else param_seed)
    rng = np.random.default_rng(n + batch if word_seed is None else word_seed)
    if pos:
        p["pos"] = (0.5 * rng.standard_normal((n + m, d))).astype(np.float32)
    y = (1.0 + 0.7 * rng.standard_normal((batch, n))).astype(np.float32)
    loss64, _, g64 = Q.forward_backward(H, p, y, None, heads=heads, attention=attention)
    tr = P.Trainer(H, d, layers, heads=heads, attention=attention)
    loss, g = tr.grad(_to_dev(p), _dev(np.tile(y, (repeat, 1))))
    torch.cuda.synchronize()
    errs = {"w_" + k: _rel(g["w"][k].cpu().numpy(), g64["w"][k]) for k in KINDS}
    errs.update({"b_" + k: _rel(g["b"][k].cpu().numpy(), g64["b"][k]) for k in KINDS if k != "k"})
    for k in ("embed", "delta", "ln1_g", "ln1_b", "ln2_g", "ln2_b", "head_w1", "head_wo", "head_bo"):
        errs[k] = _rel(g[k].cpu().numpy(), g64[k])
    print(" ".join(f"{k}={v:.1e}" for k, v in sorted(errs.items())), flush=True)
    tr.close()
    return errs, loss.item(), loss64


def test_train_step_takes_any_workspace_alignment():
    """The step reads its workspace in 16-byte pieces; a workspace at any 4-byte boundary gives the same bits."""
    import paper_2410_05911_amd as P
    H = hamming_7_4()
    p = _to_dev(random_qat_params(7, 3, 64, 2, seed=5))
    y = _dev(1.0 + 0.7 * np.random.default_rng(5).standard_normal((4, 7)))
    tr = P.Trainer(H, 64, 2)
    loss, g = tr.grad(p, y)
    for shift in (4, 20, 128):
        tr._ws = torch.empty(tr.workspace_size(4) + shift, dtype=torch.uint8, device="cuda")[shift:]
        loss2, g2 = tr.grad(p, y)
        torch.cuda.synchronize()
        assert torch.equal(loss, loss2) and all(torch.equal(g["w"][k], g2["w"][k]) for k in KINDS)
        assert torch.equal(g["embed"], g2["embed"]) and torch.equal(g["delta"], g2["delta"])
    tr.close()
