"""The work that a user of this framework has it do, as cases to be measured.

A case is one decode of a batch of received words (Decoder.decode: fused kernel for short codes,
layered kernels otherwise, and the separate kernels of the one-scale-per-word mode) or one
quantisation-aware training step (Trainer.grad: loss and every gradient).  The codes and model
sizes are those of workloads/configs.py; batches run from a single word (a receiver that waits for
its answer) to the configured batches of a throughput decoder.  Parity-check matrices belong to the
code and are fixed; weights and channel words come from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2410_05911_amd as aecct
from workloads import bch_31_16, generator_from_parity, hamming_7_4, random_qat_params, random_weights, regular_ldpc_3_6

KINDS = ("q", "k", "v", "o", "ff1", "ff2")
EBN0 = {"hamming": (4.0, 5.0, 6.0), "bch": (4.0, 5.0, 6.0, 7.0), "ldpc": (2.0, 3.0, 4.0, 5.0)}


def _decode(name, code, n, d, layers, batch, **options):
    return {"name": name, "do": "decode", "code": code, "n": n, "d": d, "layers": layers, "batch": batch,
            "attention": "hpsa", "first_ring_heads": 4, "act_scale": "token", "pos": False, **options}


def _train(name, code, n, d, layers, batch, **options):
    return {"name": name, "do": "train", "code": code, "n": n, "d": d, "layers": layers, "batch": batch,
            "attention": "hpsa", "first_ring_heads": 4, "zero_codeword": True, "pos": False, **options}


def listed():
    return [
        # a control channel's short code, a few words at a time: nothing but latency
        _decode("decode_hamming7_4_b64", "hamming", 7, 32, 2, 64),
        # the benchmark's workload: the short BCH code at the batch of a throughput decoder
        _decode("decode_bch31_16_b65536", "bch", 31, 32, 6, 65536),
        # the ECCT mask on every head (the comparison model), an odd batch
        _decode("decode_bch31_16_casa_b3001", "bch", 31, 32, 6, 3001, attention="casa"),
        # one received word of a medium code: the receiver waits for this answer
        _decode("decode_ldpc128_64_b1", "ldpc", 128, 64, 6, 1),
        # the medium code in bulk
        _decode("decode_ldpc128_64_b8192", "ldpc", 128, 64, 6, 8192),
        # a handful of words of the large model, fewer than the card has compute units
        _decode("decode_ldpc256_128_b37", "ldpc", 256, 128, 10, 37),
        # the large model in bulk
        _decode("decode_ldpc256_128_b4096", "ldpc", 256, 128, 10, 4096),
        # the longest code, with a positional table
        _decode("decode_ldpc1024_512_b1024", "ldpc", 1024, 128, 10, 1024, pos=True),
        # one activation scale per word, the literal reading of the paper's Eq. 2
        _decode("decode_ldpc128_64_word_b1024", "ldpc", 128, 64, 6, 1024, act_scale="word"),
        # training steps: the short code at the paper's batch of 128 words, the medium code on random
        # codewords with an odd batch, the large model at a batch that a card of this size takes
        _train("train_bch31_16_b128", "bch", 31, 32, 6, 128),
        _train("train_ldpc128_64_b125", "ldpc", 128, 64, 6, 125, zero_codeword=False),
        _train("train_ldpc256_128_b256", "ldpc", 256, 128, 10, 256),
    ]


# what a second does, roughly, on the path that a case takes: bounds the drawn sizes
_RATE = {"fused": 200e12, "layered": 400e12, "word": 40e12, "train": 45e12}


def _linear_flops(n, m, d, layers):
    """The six ternary maps of one word, every layer: two operations a multiply-accumulate."""
    return 2.0 * 12 * d * d * (n + m) * layers


def draw(rng):
    train = rng.random() < 0.3
    code = rng.choice(("hamming", "bch", "bch", "ldpc", "ldpc", "ldpc", "ldpc", "ldpc"))
    if train and code == "hamming":   # a training step of a toy code has too few roundings to compare
        code = "bch"
    if code == "hamming":
        n, m, d = 7, 3, 32
    elif code == "bch":
        n, m, d = 31, 15, 32
    else:   # (3, 6)-regular, any even length from 64 to 1024 (400 where it is trained)
        n = 2 * round(math.exp(rng.uniform(math.log(32), math.log(200 if train else 512))))
        m = n // 2
        d = 64 if n <= 160 else 128
        if n <= 320 and rng.random() < 0.25:
            d = 192 - d   # the other width
    layers = rng.choice((2, 4, 6)) if d == 32 else rng.choice((4, 6, 8, 10))
    attention = "casa" if rng.random() < 0.2 else "hpsa"
    case = {"do": "train" if train else "decode", "code": code, "n": n, "d": d, "layers": layers, "attention": attention,
            "first_ring_heads": 4 if rng.random() < 0.7 else rng.choice((2, 6)), "pos": rng.random() < 0.25}
    word = not train and rng.random() < 0.12
    per = _linear_flops(n, m, d, layers) * (3 if train else 1)
    rate = _RATE["train" if train else "word" if word else "fused" if d == 32 else "layered"]
    most = max(1, int((0.018 if train else 0.009) * rate / per))   # about 18 ms, 9 ms
    if train:
        case["zero_codeword"] = rng.random() < 0.5
        # below a hundred words a handful of roundings decides how far two correct steps are apart
        low, most = (100, 512) if code == "bch" else (128, max(136, min(most, 320)))
    else:
        case["act_scale"] = "word" if word else "token"
        low, most = 1, min(most, 65536)
    case["batch"] = max(1, min(most, round(math.exp(rng.uniform(math.log(low), math.log(most))))))
    return case


_CODES: dict = {}


def _code(case):
    """(H, G) of the case's code; building an LDPC graph takes longer than a decode."""
    key = case["code"], case["n"]
    if key not in _CODES:
        H = hamming_7_4() if key[0] == "hamming" else bch_31_16() if key[0] == "bch" else regular_ldpc_3_6(key[1], seed=1000 + key[1])
        _CODES[key] = H, generator_from_parity(H)
    return _CODES[key]


def _words(case, seed):
    """Channel words y = x_s + noise of random codewords, the SNR drawn per word, and the sent +-1 words."""
    _, G = _code(case)
    k, n = G.shape
    B = case["batch"]
    rng = np.random.default_rng(seed)
    msg = torch.from_numpy(rng.integers(0, 2, (B, k)).astype(np.float32)).cuda()
    xs = 1.0 - 2.0 * ((msg @ torch.from_numpy(G.astype(np.float32)).cuda()) % 2.0)
    levels = (3.0, 4.0, 5.0, 6.0, 7.0) if case["do"] == "train" else EBN0[case["code"]]
    ebn0 = rng.choice(np.asarray(levels), B)
    sigma = 1.0 / np.sqrt(2.0 * k / n * 10.0 ** (ebn0 / 10.0))
    noise = (rng.standard_normal((B, n), dtype=np.float32) * sigma[:, None].astype(np.float32)).astype(np.float32)
    return (xs + torch.from_numpy(noise).cuda()).contiguous(), xs.contiguous()


def _model(case, seed):
    H, _ = _code(case)
    m, n = H.shape
    return random_weights(n, m, case["d"], case["layers"], seed=seed, with_pos=case["pos"],
                          first_ring_heads=case["first_ring_heads"], attention=case["attention"], act_scale=case["act_scale"])


def _qat(case, seed):
    H, _ = _code(case)
    m, n = H.shape
    p = random_qat_params(n, m, case["d"], case["layers"], seed=seed)
    p["head_b1"] = np.array([p["head_b1"]], np.float32)
    if case["pos"]:
        p["pos"] = (0.5 * np.random.default_rng(seed).standard_normal((n + m, case["d"]))).astype(np.float32)
    return p


def _cuda(p, dtype=torch.float32):
    if isinstance(p, dict):
        return {k: _cuda(v, dtype) for k, v in p.items()}
    return None if p is None else torch.from_numpy(p).to("cuda", dtype)


def _train_words(case, seed):
    y, xs = _words(case, seed)
    # the paper trains on the all-zero codeword: the same noise with the sent word divided out
    return ((y * xs).contiguous(), None) if case["zero_codeword"] else (y, xs)


def prepare(case, seed):
    H, _ = _code(case)
    if case["do"] == "decode":
        y, _ = _words(case, seed)
        return {"decoder": aecct.Decoder(H, _model(case, seed)), "y": y}
    y, xs = _train_words(case, seed)
    trainer = aecct.Trainer(H, case["d"], case["layers"], first_ring_heads=case["first_ring_heads"],
                            attention=case["attention"])
    return {"trainer": trainer, "params": _cuda(_qat(case, seed)), "y": y, "xs": xs}


def run(state):
    if "decoder" in state:
        bits, logits = state["decoder"].decode(state["y"])
        return {"bits": bits, "logits": logits}
    loss, grads = state["trainer"].grad(state["params"], state["y"], state["xs"])
    # The key bias has no gradient (softmax ignores a constant added to a row's scores): what comes
    # back there is rounding noise around zero and not returned.
    return {"loss": loss, **{k: v for k, v in grads.items() if k != "b"},
            "b": {k: v for k, v in grads["b"].items() if k != "k"}}


def work(case):
    H, _ = _code(case)
    m, n = H.shape
    L, d, N, B = n + m, case["d"], case["layers"], case["batch"]
    adj = np.zeros((L, L), bool)
    adj[:n, n:] = H.T > 0
    adj[n:, :n] = H > 0
    first = int(adj.sum())
    a = adj.astype(np.float32)
    second = int(((a @ a) > 0).sum())
    hf = case["first_ring_heads"]
    pairs = 8 * (first + second) if case["attention"] == "casa" else hf * first + (8 - hf) * second
    # a pair: the dot product and the weighted value, d_h multiply-accumulates each
    flops = B * (_linear_flops(n, m, d, N) + N * pairs * 4 * (d // 8) + 2 * (L * d + L * n))
    if case["do"] == "decode":
        # y in, bits and logits out; ternary weights at two bits an entry, the rest as fp32
        params = N * (12 * d * d / 4 + 4 * (13 * d)) + 4 * (L * d * (2 if case["pos"] else 1) + L * n)
        return {"bytes": B * n * (4 + 1 + 4) + params, "flops": flops}
    # forward, input gradients and weight gradients; parameters in, gradients out, fp32
    params = 4 * (N * (12 * d * d + 13 * d + 6) + L * d + L * n + n + d + 1)
    return {"bytes": B * n * 4 * (1 if case["zero_codeword"] else 2) + 2 * params, "flops": 3 * flops}


def tolerance(case):
    # A decode's order of evaluation is fixed: its bits and logits are the same in every kernel.
    # A training step takes its int8 and ternary rounding decisions in fp32; one that falls on the
    # other side shifts the rest of its word by a code step.  Gradients seen against 64 bits: up to
    # 3e-3 on the BCH code, up to 1.6e-2 on LDPC codes (batches of 100 to 128), single entries more.
    if case["do"] == "decode":
        return "exact"
    return {"rel": 0.012, "max": 0.5} if case["code"] == "bch" else {"rel": 0.03, "max": 0.99}


# ---- the same in 64 bits, plain torch ---------------------------------------------------------

def _masks(H, attention, hf):
    m, n = H.shape
    L = n + m
    adj = torch.zeros(L, L, dtype=torch.float64, device="cuda")
    h = torch.from_numpy(H.astype(np.float64)).cuda()
    adj[:n, n:] = h.t()
    adj[n:, :n] = h
    one, two = adj > 0, (adj @ adj) > 0
    return [one | two] * 8 if attention == "casa" else [one if i < hf else two for i in range(8)]


def _quant(x, word):
    """Eq. 2: absmax codes of each token's row (or of the whole word) as the values they stand for,
    the rounding passing gradients straight through."""
    a = x.detach().abs().amax((1, 2) if word else 2, keepdim=True)
    q = torch.where(a == 0, torch.zeros_like(x), torch.round(x.detach() * (127.0 / torch.where(a == 0, 1.0, a))) * a / 127.0)
    return x + (q - x).detach()


def _forward(y, H, embed, pos, maps, ln, head, masks, word):
    """Logits of the words y; maps[l][kind] = (scaled ternary matrix, bias)."""
    syn = ((y < 0).double() @ H.t()) % 2.0
    t = torch.cat([y.abs(), 1.0 - 2.0 * syn], 1)
    X = t[:, :, None] * embed + (0.0 if pos is None else pos)
    B, L, d = X.shape
    dh = d // 8

    def norm(r, g, b):
        e = r - r.mean(-1, keepdim=True)
        return e / torch.sqrt((e * e).mean(-1, keepdim=True) + 1e-5) * g + b

    for l, layer in enumerate(maps):
        lin = lambda x, kind: x @ layer[kind][0] + layer[kind][1]  # noqa: E731
        Xh = _quant(X, word)
        Q, K, V = (lin(Xh, k) for k in ("q", "k", "v"))
        out = []
        for h in range(8):
            c = slice(h * dh, (h + 1) * dh)
            s = Q[..., c].contiguous() @ K[..., c].transpose(1, 2).contiguous() / math.sqrt(dh)
            p = torch.softmax(s.masked_fill(~masks[h], -math.inf), -1)
            out.append(p @ V[..., c].contiguous())
        X1 = norm(X + lin(_quant(torch.cat(out, -1), word), "o"), ln["ln1_g"][l], ln["ln1_b"][l])
        G = _quant(torch.relu(lin(_quant(X1, word), "ff1")), word)
        X = norm(X1 + lin(G, "ff2"), ln["ln2_g"][l], ln["ln2_b"][l])
    z = X @ head["w1"] + head["b1"]
    return z @ head["wo"] + head["bo"]


def exact(case, seed):
    H, _ = _code(case)
    Hd = torch.from_numpy(H.astype(np.float64)).cuda()
    L, B = sum(H.shape), case["batch"]
    masks = _masks(H, case["attention"], case["first_ring_heads"])
    f64 = torch.float64
    if case["do"] == "decode":
        y, _ = _words(case, seed)
        w = _model(case, seed)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float64)).cuda()  # noqa: E731
        maps = [{k: (dev(w.w[k][l]) * float(w.scale[l, i]), dev(w.b[k][l])) for i, k in enumerate(KINDS)} for l in range(w.n_layers)]
        ln = {k: dev(getattr(w, k)) for k in ("ln1_g", "ln1_b", "ln2_g", "ln2_b")}
        head = {"w1": dev(w.head_w1), "b1": float(w.head_b1), "wo": dev(w.head_wo), "bo": dev(w.head_bo)}
        pos = None if w.pos is None else dev(w.pos)
        step = max(1, int(2e9 / (8 * L * (L + 16 * case["d"]))))
        got = [_forward(y[i:i + step].to(f64), Hd, dev(w.embed), pos, maps, ln, head, masks, case["act_scale"] == "word")
               for i in range(0, B, step)]
        return {"bits": None, "logits": torch.cat(got)}
    y, xs = _train_words(case, seed)
    p = _cuda(_qat(case, seed), f64)
    leaves = {k: v.requires_grad_() for k, v in p.items() if k not in ("w", "b", "pos")}
    for group in ("w", "b"):
        leaves.update({(group, k): p[group][k].requires_grad_() for k in KINDS})
    maps = []
    for l in range(case["layers"]):
        layer = {}
        for i, k in enumerate(KINDS):   # Eq. 1 on the latent matrix, the rounding passing gradients through
            W = p["w"][k][l]
            s = torch.quantile(W.detach().abs().flatten(), 0.5) * p["delta"][l, i]
            u = W / (s + 1e-8)
            T = u + (torch.round(u).clamp(-1, 1) - u).detach()
            layer[k] = T * s, p["b"][k][l]
        maps.append(layer)
    head = {"w1": p["head_w1"], "b1": p["head_b1"], "wo": p["head_wo"], "bo": p["head_bo"]}
    sent = torch.ones_like(y) if xs is None else xs
    target = (y * sent < 0).to(f64)
    step = max(1, int(1.5e9 / (8 * L * (L + 8 * case["d"]))))
    total = {k: torch.zeros_like(v) for k, v in leaves.items()}
    for i in range(0, B, step):
        f = _forward(y[i:i + step].to(f64), Hd, p["embed"], p["pos"], maps, p, head, masks, False)
        loss = torch.nn.functional.binary_cross_entropy_with_logits(-f, target[i:i + step], reduction="sum") / (B * H.shape[1])
        for k, g in zip(leaves, torch.autograd.grad(loss, list(leaves.values()), retain_graph=i + step < B)):
            total[k] += g
    # The loss and the head's scalar bias gradient are single numbers, off by chance and not by precision
    # (each rounding decision of the int8 codes that falls on the other side moves them): no value here.
    return {"loss": None, "head_b1": None, "w": {k: total["w", k] for k in KINDS},
            "b": {k: total["b", k] for k in KINDS if k != "k"},
            **{k: total[k] for k in leaves if isinstance(k, str) and k != "head_b1"}}
