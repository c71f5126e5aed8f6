"""Batches smaller than the card decode through other launch shapes than full ones (a word's head
groups spread over blocks, a 16-token strip or a short word's tiles over wavefronts); every shape has
to give the bits of the whole-word form, which test_gpu_parity.py pins to the oracle.

For each attention form the words of one batch too large to be spread are decoded again in the sizes
where the number of head groups per block and the token block's form change (up to 384 strips of 16
tokens on 256 compute units take a block per strip), down to a single word; results are compared bit
for bit (the order of every sum is fixed, so the tolerance is zero).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import random_weights, regular_ldpc_3_6, generator_from_parity, awgn_words  # noqa: E402


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2410_05911_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("n,d,heads,attention,hf,form,batch,sizes", [
    (128, 64, 8, "hpsa", 4, -1, 1100, (1, 5, 32, 33, 130, 200, 300, 520)),     # fp32 K and V, d_h = 8, two blocks a CU
    (66, 64, 4, "casa", 2, -1, 1100, (1, 33, 257)),                    # d_h = 16 at d = 64, 99 tokens
    (66, 128, 16, "hpsa", 6, -1, 600, (1, 40, 129)),                   # d_h = 8 at d = 128
    (256, 128, 8, "hpsa", 4, -1, 600, (1, 2, 16, 17, 37, 70, 129, 260)),       # lane pairs, codes | fp32 O
    (270, 128, 8, "casa", 2, -1, 300, (1, 50, 100)),                   # lane pairs, 405 tokens: a second row a pair
    (514, 128, 8, "hpsa", 4, -1, 300, (1, 33, 66, 130)),               # fp32 K, int16 V, 771 tokens
    (398, 64, 8, "hpsa", 4, -1, 600, (1, 70, 140)),                    # int16 K and V, d_h = 8
    (256, 128, 8, "hpsa", 4, 2, 300, (1, 40)),                         # the int16 form by request
])
def test_spread_head_groups_match_whole_words(P, n, d, heads, attention, hf, form, batch, sizes):
    H = regular_ldpc_3_6(n, seed=1000 + n)
    w = random_weights(n, n // 2, d, 3, heads, seed=n + d, first_ring_heads=hf, attention=attention, with_pos=hf == 2)
    y, _, _ = awgn_words(generator_from_parity(H), batch, (2.0, 4.0), seed=n)
    yd = torch.from_numpy(y).cuda()
    dec = P.Decoder(H, w, layered_attention=form)
    bits, logits = dec.decode(yd)
    torch.cuda.synchronize()
    assert np.isfinite(logits.cpu().numpy()).all()
    for k in sizes:
        print(f"[small] LDPC({n}) d {d} heads {heads} {attention}: {k} words", flush=True)
        at = (batch - k) // 2
        b, f = dec.decode(yd[at:at + k].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(f, logits[at:at + k]) and torch.equal(b, bits[at:at + k])
    dec.close()


@pytest.mark.parametrize("n,m,attention,sizes", [
    (7, 3, "hpsa", (1, 64, 300)),                       # one token tile: never split
    (20, 10, "hpsa", (1, 5, 257, 1537, 1536)),          # two tiles, up to six words a block
    (31, 15, "casa", (1, 255, 256, 257, 513, 1024, 1025)),   # three tiles, up to four words a block
    (40, 20, "hpsa", (1, 256, 700, 768, 769)),          # four tiles, up to three words a block
])
def test_fused_word_over_wavefronts_matches_one_wavefront(P, n, m, attention, sizes):
    rng = np.random.default_rng(n)
    H = (rng.random((m, n)) < 0.3).astype(np.uint8)
    H[np.arange(n) % m, np.arange(n)] = 1               # no empty row or column
    w = random_weights(n, m, 32, 3, seed=n, attention=attention, with_pos=m == 20)
    batch = 3500
    yd = torch.from_numpy((1.0 + 0.6 * rng.standard_normal((batch, n))).astype(np.float32)).cuda()
    dec = P.Decoder(H, w, path=P.PATH_FUSED)
    bits, logits = dec.decode(yd)
    torch.cuda.synchronize()
    assert np.isfinite(logits.cpu().numpy()).all()
    for k in sizes:
        print(f"[small] fused n {n} m {m} {attention}: {k} words", flush=True)
        b, f = dec.decode(yd[batch - k:].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(f, logits[batch - k:]) and torch.equal(b, bits[batch - k:])
    dec.close()


@pytest.mark.parametrize("n,d,heads,attention,hf,sizes", [
    (66, 64, 8, "hpsa", 4, (1, 3, 700)),        # 99 tokens: strips straddle words
    (66, 64, 4, "casa", 2, (5,)),               # d_h = 16 at d = 64, positional table
    (128, 64, 8, "hpsa", 4, (1, 520)),
    (256, 128, 8, "casa", 2, (1, 40, 300)),     # lane pairs
    (514, 128, 8, "hpsa", 4, (1, 20)),          # fp32 K, int16 V, 771 tokens
    (398, 64, 8, "hpsa", 6, (1, 60)),           # int16 K and V
])
def test_word_scale_stages_match_separate_kernels(P, n, d, heads, attention, hf, sizes):
    """One alpha per word: the fused attention with the maps in stages between the word maxima, against the
    separate kernels (pinned to the oracle below and by test_gpu_boundary.py), bit for bit."""
    H = regular_ldpc_3_6(n, seed=1000 + n)
    w = random_weights(n, n // 2, d, 2, heads, seed=n + d, first_ring_heads=hf, attention=attention, act_scale="word",
                       with_pos=hf == 2)
    y, _, _ = awgn_words(generator_from_parity(H), max(sizes), (2.0, 4.0), seed=n)
    yd = torch.from_numpy(y).cuda()
    staged, separate = P.Decoder(H, w), P.Decoder(H, w, layered_attention=P.LAYERED_ATTN_UNFUSED)
    bits, logits = separate.decode(yd)
    torch.cuda.synchronize()
    assert np.isfinite(logits.cpu().numpy()).all()
    for k in sizes:
        print(f"[word] LDPC({n}) d {d} {attention}: {k} words", flush=True)
        b, f = staged.decode(yd[:k].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(f, logits[:k]) and torch.equal(b, bits[:k])
    b, f = staged.decode_static(yd)
    torch.cuda.synchronize()
    assert torch.equal(f, logits) and torch.equal(b, bits)
    staged.close()
    separate.close()


@pytest.mark.parametrize("n,d,heads,attention,hf,form", [
    (66, 64, 4, "casa", 2, -1),        # fp32 K and V, d_h = 16 at d = 64
    (128, 128, 16, "hpsa", 6, -1),     # d_h = 8 at d = 128
    (256, 128, 8, "hpsa", 4, -1),      # lane pairs
    (514, 128, 8, "casa", 2, -1),      # fp32 K, int16 V, 771 tokens
    (398, 64, 8, "hpsa", 4, -1),       # int16 K and V
    (256, 128, 8, "hpsa", 4, 0),       # the separate kernels
    (514, 128, 8, "casa", 2, 0),
])
def test_word_scale_against_oracle(P, oracle_mod, n, d, heads, attention, hf, form):
    """One alpha per word at the widths and lengths of every attention form, staged (AUTO) and as separate kernels:
    bits and logits of a few words equal the oracle's.  Both are reported as UNFUSED; the staged form is told
    by its workspace of less than four fp32 rows of d a token, where the separate kernels hold Q, K, V and the
    hidden row besides."""
    H = regular_ldpc_3_6(n, seed=1000 + n)
    w = random_weights(n, n // 2, d, 2, heads, seed=n + d, first_ring_heads=hf, attention=attention, act_scale="word",
                       with_pos=hf == 2)
    y, _, _ = awgn_words(generator_from_parity(H), 5, (2.0, 4.0), seed=n)
    print(f"[word] LDPC({n}) d {d} {attention} form {form} against the oracle", flush=True)
    dec = P.Decoder(H, w, layered_attention=form)
    rows = 5 * dec.L
    assert (dec.workspace_size(5) < 4 * rows * 4 * d) == (form == -1)
    bits, logits = dec.decode(torch.from_numpy(y).cuda())
    torch.cuda.synchronize()
    bo, fo = oracle_mod.OracleModel(H, w).decode(y, n_threads=5)
    assert np.array_equal(logits.cpu().numpy(), fo) and np.array_equal(bits.cpu().numpy(), bo)
    dec.close()
