"""Performance cases: the work that users of this framework have it do, through its public entry points.

Three kinds of call:

* "request": one decoding request at batch 1.  A context is made for the request (P.Engine: a context serves one prompt),
  the prompt is prefilled, draft / verify / accept cycles run until `gen` tokens are out, the context is closed.  The
  weights are what a serving program keeps; prompts differ.  Outputs: the tokens, and the target's logits behind each token
  of the last cycle (one row per token; the other rows of the verified tree belong to candidates that the draft proposed
  and the target did not take, and which those are may hang on a near tie).
* "hca": the attention of one training step of the draft layer (harmonized context alignment), j = `streams`.
* "loss": the Top-K distillation loss of a batch of positions through the LM head.

Sizes are those of the benchmark configurations (workload.CONFIGS), with fewer layers where a full model would only repeat
the same layer more often, and of the tests.
"""
import math

import numpy as np
import torch

import paper_2408_15766_amd as P
import workload as wl

# (parent, rank) of the 26-node static tree that the benchmark offers: 4/8/8/4/1 nodes per depth
TREE26 = ([-1, 0, 0, 0, 0, 1, 1, 1, 2, 2, 3, 3, 4, 5, 5, 5, 6, 6, 8, 8, 10, 13, 13, 14, 16, 21],
          [0, 0, 1, 2, 3, 0, 1, 2, 0, 1, 0, 1, 0, 0, 1, 2, 0, 1, 0, 1, 0, 0, 1, 0, 0, 0])


def _request(model, layers, prompt, gen, depth, topk, total, temperature, static=""):
    return {"kind": "request", "model": model, "layers": layers, "prompt": prompt, "gen": gen, "depth": depth, "topk": topk,
            "total": total, "temperature": temperature, "static": static}


def _hca(streams, batch, seq, hq, hkv, hd):
    return {"kind": "hca", "streams": streams, "batch": batch, "seq": seq, "hq": hq, "hkv": hkv, "hd": hd}


def _loss(dtype, rows, d, vocab, k):
    return {"kind": "loss", "dtype": dtype, "rows": rows, "d": d, "vocab": vocab, "k": k}


def listed():
    return [
        # the smallest request: a two-layer fp32 model whose launches cost more than their work (functional tests, debugging)
        dict(_request("tiny", 2, 32, 64, 3, 4, 16, 0.0), name="tiny-fp32"),
        # the headline: a chat turn on the full 7B model, 60-node dynamic tree, greedy
        dict(_request("llama2-7b", 32, 512, 64, 6, 10, 60, 0.0), name="7b-tree"),
        # plain decoding (what speculation is compared with), short prompt of odd length
        dict(_request("llama2-7b", 32, 77, 16, 1, 1, 1, 0.0), name="7b-plain"),
        # sampling at T = 1 on the 13B widths (depth shortened)
        dict(_request("llama2-13b", 10, 512, 48, 6, 10, 60, 1.0), name="13b-sampled"),
        # a long document: 4096-token prompt, grouped heads, large vocabulary (depth shortened)
        dict(_request("llama3-8b", 16, 4096, 32, 6, 10, 60, 0.0), name="8b-long-prompt"),
        # the largest widths, prompt of 1024 (depth shortened: the full model does not fit the card three times)
        dict(_request("llama3-70b", 8, 1024, 32, 6, 10, 60, 0.0), name="70b-widths"),
        # a static tree with sampled children (the ratio rule), prompt length ragged against every tile
        dict(_request("llama3-8b", 8, 1333, 24, 5, 8, 26, 1.0, "tree26"), name="8b-static-tree"),
        # training attention at the paper's launch: batch 2 x 2048, three aligning steps, 7B draft layer
        dict(_hca(3, 2, 2048, 32, 32, 128), name="hca-7b"),
        # the same step with grouped heads and a short ragged batch: a launch that does not fill the chip
        dict(_hca(2, 1, 333, 16, 4, 64), name="hca-short"),
        # distillation loss of one training batch at the 7B vocabulary, the paper's K
        dict(_loss("bf16", 4096, 4096, 32000, 10), name="loss-7b"),
        # the largest K of the paper's ablation, LLaMA3 vocabulary, a ragged number of positions
        dict(_loss("bf16", 700, 4096, 128256, 100), name="loss-k100"),
        # a small fp32 loss (unit tests of a trainer)
        dict(_loss("fp32", 129, 512, 9000, 16), name="loss-fp32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["request", "request", "request", "hca", "loss"])
    if kind == "request":
        model = rng.choice(["tiny", "llama2-7b", "llama2-13b", "llama3-8b", "llama3-70b"])
        layers = 2 if model == "tiny" else rng.randint(1, {"llama2-7b": 12, "llama2-13b": 8, "llama3-8b": 10, "llama3-70b": 4}[model])
        prompt = _log_int(rng, 1, 900 if model == "tiny" else 1024 if model == "llama3-70b" else 4096)
        gen = _log_int(rng, 2, 48)
        temperature = float(rng.choice([0, 0, 1]))
        form = rng.choice(["dynamic", "dynamic", "dynamic", "plain", "tree26", "chain"])
        if form == "plain":
            return _request(model, layers, prompt, gen, 1, 1, 1, temperature)
        if form == "tree26":
            return _request(model, layers, prompt, gen, 5, 8, 26, temperature, "tree26")
        if form == "chain":
            n = rng.randint(1, 8)
            return _request(model, layers, prompt, gen, n, 1, n + 1, temperature, "chain%d" % n)
        depth, topk = rng.randint(2, 10), rng.randint(2, 16)
        total = min(_log_int(rng, 8, 128), 1 + topk + (depth - 1) * topk * topk)
        return _request(model, layers, prompt, gen, depth, topk, max(total, depth + 1), temperature)
    if kind == "hca":
        hkv = rng.choice([1, 2, 4, 8, 32])
        hq = hkv * (1 if hkv == 32 else rng.choice([1, 2, 4, 8]))
        return _hca(rng.randint(1, 8), rng.randint(1, 3), _log_int(rng, 16, 2048), hq, hkv, rng.choice([64, 128, 128]))
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    vocab = rng.choice([1000, 9000, 32000, 32000, 128256])
    d = 8 * _log_int(rng, 32, 640)
    rows = _log_int(rng, 1, 4096)
    if dtype == "fp32":                                        # fp32 is for small models
        d, rows, vocab = min(d, 1024), min(rows, 700), min(vocab, 32000)
    rows = max(1, min(rows, int(4.0e11 / (d * vocab))))        # no dearer than the listed ones
    return _loss(dtype, rows, d, vocab, min(_log_int(rng, 1, 128), 4096 // ((vocab + 4095) // 4096)))


def _shape(case):
    return wl.BY_NAME[case["model"]].with_(n_layers=case["layers"], prompt_len=case["prompt"], gen_tokens=case["gen"],
                                           tree_depth=case["depth"], tree_topk=case["topk"], tree_total=case["total"],
                                           temperature=case["temperature"])


def _weights(shape, gen):
    """Random weights of the shape whose next-token distribution is peaked, as a trained model's is, and whose draft agrees with
    the target: the LM head row of a token carries the embedding of its predecessor in a random cycle through the
    vocabulary, the draft's fc passes the token's embedding on, and the output projections are scaled (down with the depth,
    the usual initialisation, and with the width) so that all layers together add about half of the embedding's size to
    the residual stream.  The tokens are then a function of the prompt and not of rounding."""
    dt = torch.bfloat16 if shape.dtype == "bf16" else torch.float32
    d, v = shape.d_model, shape.vocab

    def normal(dims, std):
        return torch.empty(dims, dtype=dt, device="cuda").normal_(0.0, std, generator=gen)
    embed = normal((v, d), 1.0)
    cycle = torch.randperm(v, device="cuda", generator=gen)
    head = normal((v, d), 0.02)
    head[cycle] += embed[cycle.roll(1)] * (40.0 / d)
    gate = 0.02 * math.sqrt(d)                                 # spread of the gate and up sums; their SwiGLU's is about 0.6 of its square
    down_std = 0.5 / (0.6 * gate * gate * math.sqrt(shape.d_ffn))
    for name, dims, kind in wl.tensor_specs(shape):
        if name == "embed":
            yield name, embed
        elif name == "lm_head":
            yield name, head
        elif kind == "ones":
            yield name, torch.ones(dims, dtype=dt, device="cuda")
        elif name == "draft.fc":
            fc = normal(dims, 0.01)
            fc[:, d:].diagonal().add_(2.0)
            yield name, fc
        elif name.endswith(".w_down"):
            yield name, normal(dims, down_std / (math.sqrt(shape.n_layers) if name.startswith("layers.") else 1.0))
        elif name.endswith(".wo"):
            yield name, normal(dims, 0.01 / math.sqrt(2 * shape.n_layers))
        else:
            yield name, normal(dims, 0.02)


def _normal(dims, dt, gen, std=1.0):
    return torch.empty(dims, dtype=dt, device="cuda").normal_(0.0, std, generator=gen)


def _loss_inputs(case, dt, gen):
    rows, d = case["rows"], case["d"]
    ft = _normal((rows, d), dt, gen)
    fd = ft + _normal((rows, d), dt, gen, 0.5)                 # a draft's estimate of the feature
    return ft, fd, _normal((case["vocab"], d), dt, gen, 3.0 / math.sqrt(d))


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "request":
        shape = _shape(case)
        weights = P.pack_weights(_weights(shape, gen))
        prompt = torch.randint(0, shape.vocab, (case["prompt"],), generator=gen, device="cuda").cpu().numpy().astype(np.int32)
        static = None
        if case["static"] == "tree26":
            static = TREE26
        elif case["static"]:
            n = int(case["static"][5:])
            static = ([-1] + list(range(n)), [0] * (n + 1))
        return {"kind": "request", "shape": shape, "weights": weights, "prompt": prompt, "gen": case["gen"], "static": static,
                "seed": seed & 0xFFFF}

    def normal(dims, dt, std=1.0):
        return _normal(dims, dt, gen, std)
    if case["kind"] == "hca":
        q = normal((case["batch"], case["seq"], case["hq"], case["hd"]), torch.bfloat16)
        kv = (case["batch"], case["seq"], case["hkv"], case["hd"])
        k0, v0 = normal(kv, torch.bfloat16), normal(kv, torch.bfloat16)
        # the draft's streams sit near the target's, the further the more steps it has run on its own features
        ks = [k0] + [k0 + normal(kv, torch.bfloat16, 0.3 * m) for m in range(1, case["streams"])]
        vs = [v0] + [v0 + normal(kv, torch.bfloat16, 0.3 * m) for m in range(1, case["streams"])]
        return {"kind": "hca", "q": q, "ks": ks, "vs": vs}
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    ft, fd, head = _loss_inputs(case, dt, gen)
    head = P.spec_pack_weight(head)
    scratch = torch.empty(P.spec_topk_loss_scratch_bytes(case["rows"], case["vocab"], case["k"]), dtype=torch.uint8, device="cuda")
    return {"kind": "loss", "ft": ft, "fd": fd, "head": head, "k": case["k"], "scratch": scratch}


def _emitted_rows(tree, tokens):
    """Rows of the verified tree whose logits the emitted tokens were taken from: the root, then each accepted node."""
    rows, cur = [0], 0
    for tok in tokens[:-1]:
        cur = next(j for j in range(cur + 1, tree.n_nodes) if tree.parent[j] == cur and tree.token[j] == tok)
        rows.append(cur)
    return rows


def run(state):
    if state["kind"] == "hca":
        return P.spec_hca_attention(state["q"], state["ks"], state["vs"])
    if state["kind"] == "loss":
        return P.spec_topk_loss(state["ft"], state["fd"], state["head"], state["k"], state["scratch"])
    eng = P.Engine(state["shape"], state["weights"], seed=state["seed"])
    if state["static"] is not None:
        eng.set_static_tree(*state["static"], sampled=state["shape"].temperature > 0)
    tokens = [eng.prefill(state["prompt"])]
    emitted, tree = [], None
    while len(tokens) < state["gen"]:
        tree = eng.draft_tree()
        eng.verify(tree)
        emitted = eng.accept(tree)
        tokens += emitted
    logits = eng.logits(tree.n_nodes)[_emitted_rows(tree, emitted)]
    eng.close()
    return {"tokens": np.array(tokens, dtype=np.int32), "logits": logits}


def work(case):
    if case["kind"] == "hca":
        pairs = case["batch"] * case["hq"] * case["seq"] * (case["seq"] + 1) / 2
        io = case["batch"] * case["seq"] * case["hd"] * 2.0 * (2 * case["hq"] + 2 * case["hkv"] * case["streams"])
        return {"bytes": io, "flops": 4.0 * case["hd"] * pairs}
    if case["kind"] == "loss":
        esz = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": esz * (2.0 * case["rows"] + case["vocab"]) * case["d"] + 8.0 * case["rows"],
                "flops": 4.0 * case["rows"] * case["vocab"] * case["d"]}
    sh = _shape(case)
    by = wl.algorithmic_bytes(sh)
    esz = 2 if sh.dtype == "bf16" else 4
    plain = case["total"] == 1
    # drafts follow the target: every cycle emits the longest path of the tree
    depth = 0 if plain else int(case["static"][5:]) if case["static"].startswith("chain") else case["depth"]
    cycles = -(-(case["gen"] - 1) // (depth + 1))
    kv = by["kv_bytes_per_token"]
    n = case["prompt"]
    draft_layer = by["layer"] + by["draft_fc"]
    # prefill: every weight once, the cache written once; a cycle: verify weights, cache read and tree rows written, the draft
    # passes (their head is the target's)
    nbytes = by["verify_weights"] + n * kv + (0 if plain else draft_layer)
    nbytes += cycles * (by["verify_weights"] + (n + case["total"]) * kv + (0 if plain else depth * by["draft_forward"]))
    layer_par, head_par = by["layer"] / esz, by["lm_head"] / esz
    attn = 4.0 * sh.d_q                                         # per (query, key) pair and layer
    rows = [1] + [case["topk"]] * (depth - 1) if depth else []
    flops = 2.0 * n * sh.n_layers * layer_par + 2.0 * head_par + sh.n_layers * attn * n * (n + 1) / 2
    flops += 0 if plain else 2.0 * n * draft_layer / esz + attn * n * (n + 1) / 2
    flops += cycles * (case["total"] * (2.0 * (sh.n_layers * layer_par + head_par) + sh.n_layers * attn * n)
                       + sum(rows) * (2.0 * (draft_layer / esz + head_par) + attn * n))
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    """About four times what was measured against the same call in fp64 (hca, loss) or in fp32 storage (bf16 requests)."""
    if case["kind"] == "hca":
        return {"rel": 0.008, "max": 0.09}                     # measured 0.0021, 0.022: probabilities and output rounded to bf16
    if case["kind"] == "loss":
        # measured 1.3e-6, 4e-6; a position whose K-th and (K+1)-th target logits are equal in fp32 but not in fp64 may take
        # either, which moves that position's loss by up to about a hundredth
        return {"rel": 1e-4, "max": 2e-2}
    if wl.BY_NAME[case["model"]].dtype == "bf16":
        return {"rel": 0.015, "max": 0.07}                     # measured 0.003 .. 0.004, 0.012 .. 0.018
    return {"rel": 2e-5, "max": 2e-4}


def _exact_request(case, seed):
    """The greedy target model over prompt and answer in 64 bits, one causal forward.  The answer is found by guess and
    correction: the guess walks the cycle that the weights were made around, a wrong token is replaced from the forward's
    logits.  As in work(), every cycle is taken to emit the tree's longest path (otherwise the outputs have other sizes)."""
    shape = _shape(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = dict(_weights(shape, gen))
    prompt = torch.randint(0, shape.vocab, (case["prompt"],), generator=gen, device="cuda")
    gen.manual_seed(seed)                                      # the draws of _weights up to the cycle
    torch.empty_like(w["embed"]).normal_(0.0, 1.0, generator=gen)
    cycle = torch.randperm(shape.vocab, device="cuda", generator=gen)
    after = torch.empty_like(cycle)
    after[cycle.roll(1)] = cycle
    step = 1 if case["total"] == 1 else 1 + (int(case["static"][5:]) if case["static"].startswith("chain") else case["depth"])
    count = 1 + -(-(case["gen"] - 1) // step) * step
    answer = [after[prompt[-1]]]
    while len(answer) < count:
        answer.append(after[answer[-1]])
    answer = torch.stack(answer)
    n, hq, hkv, hd = case["prompt"], shape.n_q_heads, shape.n_kv_heads, shape.head_dim

    def norm(h, weight):
        return h / torch.sqrt((h * h).mean(-1, keepdim=True) + shape.rms_eps) * weight.double()

    def linear(x, name):
        return x @ w[name].double().t()

    def turn(x, angle):
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        c, s = torch.cos(angle)[:, None], torch.sin(angle)[:, None]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    def forward(tokens):
        t = tokens.numel()
        angle = torch.arange(t, device="cuda").double()[:, None] * shape.rope_theta ** (
            -2.0 * torch.arange(hd // 2, device="cuda").double() / hd)
        hidden = torch.ones(t, t, dtype=torch.bool, device="cuda").triu(1)
        h = w["embed"][tokens].double()
        for l in range(shape.n_layers):
            p = "layers.%d." % l
            a = norm(h, w[p + "attn_norm"])
            q = turn(linear(a, p + "wq").view(t, hq, hd), angle)
            k = turn(linear(a, p + "wk").view(t, hkv, hd), angle)
            v = linear(a, p + "wv").view(t, hkv, hd)
            o = torch.empty(t, hq, hd, dtype=torch.float64, device="cuda")
            for i in range(hq):
                kv = i * hkv // hq
                score = (q[:, i] @ k[:, kv].t()).mul_(hd ** -0.5).masked_fill_(hidden, -math.inf)
                o[:, i] = torch.softmax(score, -1) @ v[:, kv]
            h = h + linear(o.view(t, hq * hd), p + "wo")
            b = norm(h, w[p + "ffn_norm"])
            h = h + linear(torch.nn.functional.silu(linear(b, p + "w_gate")) * linear(b, p + "w_up"), p + "w_down")
        return linear(norm(h[n - 1:], w["final_norm"]), "lm_head")
    for _ in range(4):
        logits = forward(torch.cat([prompt, answer[:-1]]))
        found = logits.argmax(-1)
        if bool((found == answer).all()):
            return {"tokens": answer.cpu().numpy().astype(np.int32), "logits": logits[count - step:].cpu().numpy()}
        answer = found
    return None


def _exact_hca(s):
    q, j = s["q"].double(), len(s["ks"])
    batch, t, hq, hd = q.shape
    ks, vs = [k.double() for k in s["ks"]], [v.double() for v in s["vs"]]
    off = torch.arange(t, device="cuda")[:, None] - torch.arange(t, device="cuda")[None]
    out = torch.empty_like(q)
    for b in range(batch):
        for i in range(hq):
            kv = i * ks[0].shape[2] // hq
            # the key of position t - o is stream j-1-o's for o <= j-2, stream 0's beyond
            score = q[b, :, i] @ ks[0][b, :, kv].t()
            for o in range(j - 1):
                score = torch.where(off == o, q[b, :, i] @ ks[j - 1 - o][b, :, kv].t(), score)
            p = torch.softmax((score * hd ** -0.5).masked_fill_(off < 0, -math.inf), -1)
            got = p.masked_fill(off < j - 1, 0.0) @ vs[0][b, :, kv]
            for o in range(j - 1):
                got += torch.where(off == o, p, 0.0) @ vs[j - 1 - o][b, :, kv]
            out[b, :, i] = got
    return out


def _exact_loss(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    ft, fd, head = _loss_inputs(case, dt, gen)
    topk, ce = [], []
    for r in range(0, case["rows"], 256):
        zq, zp = ft[r:r + 256].double() @ head.double().t(), fd[r:r + 256].double() @ head.double().t()
        q, logp = torch.softmax(zq, -1), torch.log_softmax(zp, -1)
        best = zq.topk(case["k"], -1).indices
        topk.append(-(q.gather(1, best) * logp.gather(1, best)).sum(-1))
        ce.append(-(q * logp).sum(-1))
    topk, ce = torch.cat(topk), torch.cat(ce)
    return topk, ce, torch.stack([topk.sum(), ce.sum()])


def exact(case, seed):
    """What run() returns, in 64 bits by plain torch; sampled requests have no such value."""
    if case["kind"] == "hca":
        return _exact_hca(prepare(case, seed))
    if case["kind"] == "loss":
        return _exact_loss(case, seed)
    return _exact_request(case, seed) if case["temperature"] == 0 else None
