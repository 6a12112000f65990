"""What is timed: the serving step as an engine's user runs it, through `paper_2507_17769_amd.runner.Engine`.

A user of this library feeds it one iteration after another: a list of records (request id, new tokens, KV length,
page table) and the activations or token ids that go with them, and reads the hidden states, the logits or a
request's keys and values back.  The cases cover the range of such iterations: the smallest call, single-token and
decode-only steps, mixed steps on either side of every token count at which the library changes its kernels, prefill
steps with one and several requests, long cached prefixes, the step without allocations, and the hand-off of a
prefilled request to another instance.  Model shapes are the repository's ("tiny", "8b", "70b"); lengths follow its
benchmark configurations and latency grid.  The host-only calls (admission, chunk planning, the cluster simulator)
run no device code and are not among them.

A case is a dict of plain values:
  kind      "step" (hidden states in and out), "static" (the step that allocates nothing), "model" (token ids in,
            logits and final hidden states out), "handoff" (one request's KV read on one instance, written to another
            and continued there by one decode step)
  model, layers
  chunk, chunk_prefix, n_chunks   prefill requests: `n_chunks` of them share `chunk` new tokens, cut at uneven places,
                                  each behind `chunk_prefix` cached tokens
  decodes, kv, kv_lo, kv_hi       decode requests and their KV length after the step: "uniform" in [kv_lo, kv_hi], or
                                  "lognormal" with median `kv`, sigma 0.8, clipped to [kv_lo, kv_hi]
  lengths   seed of the lengths, so that a case always means the same batch
The stacks are cut to a few layers (every layer has weights and a KV slot of its own, several times the last-level
cache together), except for the single-token model step, whose 32 layers are what its latency consists of.
"""
import functools
import random

import numpy as np
import torch

from paper_2507_17769_amd import workloads as W
from paper_2507_17769_amd.runner import Engine

VOCAB = 128256   # the benchmark's full-model vocabulary (a multiple of 64)


def _case(kind, model, layers, chunk=0, chunk_prefix=0, n_chunks=1, decodes=0, kv="lognormal", median=1024, kv_lo=16, kv_hi=8192,
          lengths=0, name=None):
    c = dict(kind=kind, model=model, layers=layers, chunk=chunk, chunk_prefix=chunk_prefix, n_chunks=n_chunks, decodes=decodes, kv=kv,
             median=median, kv_lo=kv_lo, kv_hi=kv_hi, lengths=lengths)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one layer of the tiny shape, a 64-token chunk and four decodes; launches and host time are all of it
        _case("step", "tiny", 1, chunk=64, chunk_prefix=64, decodes=4, kv="uniform", kv_lo=17, kv_hi=128, name="tiny_mixed"),
        # the engine's minimal per-token latency: one request, token in, next token out, whole 8B-shaped model
        _case("model", "8b", 32, decodes=1, kv="uniform", kv_lo=1024, kv_hi=1024, name="model_1_decode"),
        # a decode instance of a disaggregated deployment at an ordinary load
        _case("step", "8b", 4, decodes=64, kv="uniform", kv_lo=512, kv_hi=4096, name="decode_64"),
        # the same at a high load: as many decode tokens as the latency grid has
        _case("step", "8b", 4, decodes=256, name="decode_256"),
        # a serving loop that may not allocate; an odd batch just past the sizes with a row tile of their own
        _case("static", "8b", 4, decodes=97, median=512, kv_hi=4096, name="static_decode_97"),
        # a co-located instance under a tight token budget: small chunk, few decodes
        _case("step", "8b", 4, chunk=128, chunk_prefix=1500, decodes=16, name="chunk_128_decode_16"),
        # a ragged small prefill: three requests share 250 new tokens, next to a few decodes
        _case("step", "8b", 4, chunk=250, chunk_prefix=333, n_chunks=3, decodes=21, name="ragged_250_decode_21"),
        # the ordinary mixed step of a co-located instance
        _case("step", "8b", 4, chunk=512, chunk_prefix=2048, decodes=128, name="mixed_512_128"),
        # a prefill instance at its full budget, several prompts from position 0 (their lengths uneven)
        _case("step", "8b", 4, chunk=2048, n_chunks=3, name="prefill_2048"),
        # the last chunk of a long prompt
        _case("step", "8b", 4, chunk=2048, chunk_prefix=8192, name="chunk_2048_at_8192"),
        # the large shape: a mixed step at its full load
        _case("step", "70b", 2, chunk=1024, chunk_prefix=4096, decodes=256, median=2048, kv_hi=16384, name="mixed_70b"),
        # prefill instance -> decode instance: 2047 cached tokens of four layers move, one token is decoded behind them
        _case("handoff", "8b", 4, decodes=1, kv="uniform", kv_lo=2048, kv_hi=2048, name="handoff_2048"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng: random.Random):
    """One more iteration of the same kinds: token counts, prefixes and KV lengths spread over their logarithm."""
    lengths = rng.randrange(1, 1 << 20)
    family = rng.choice(["decode", "decode", "mixed", "mixed", "prefill", "static", "model", "handoff", "large", "tiny"])
    if family == "decode":
        return _case("step", "8b", 4, decodes=_log_uniform(rng, 2, 300), median=_log_uniform(rng, 128, 2048), lengths=lengths)
    if family == "mixed":
        return _case("step", "8b", 4, chunk=_log_uniform(rng, 17, 1600), chunk_prefix=_log_uniform(rng, 1, 4096) - 1, n_chunks=rng.randint(1, 3),
                     decodes=_log_uniform(rng, 1, 256), median=_log_uniform(rng, 128, 2048), lengths=lengths)
    if family == "prefill":
        return _case("step", "8b", 4, chunk=_log_uniform(rng, 32, 2048), chunk_prefix=_log_uniform(rng, 1, 8192) - 1, n_chunks=rng.randint(1, 4), lengths=lengths)
    if family == "static":
        return _case("static", "8b", 4, decodes=_log_uniform(rng, 1, 128), median=_log_uniform(rng, 64, 512), kv_hi=4096, lengths=lengths)
    if family == "model":
        return _case("model", "8b", 4, chunk=rng.choice([0, _log_uniform(rng, 32, 512)]), chunk_prefix=_log_uniform(rng, 1, 2048) - 1,
                     decodes=_log_uniform(rng, 1, 64), median=_log_uniform(rng, 128, 2048), lengths=lengths)
    if family == "handoff":
        n = _log_uniform(rng, 32, 8192)
        return _case("handoff", "8b", 4, decodes=1, kv="uniform", kv_lo=n, kv_hi=n, lengths=lengths)
    if family == "large":
        return _case("step", "70b", 2, chunk=rng.choice([0, _log_uniform(rng, 64, 1024)]), chunk_prefix=_log_uniform(rng, 1, 4096) - 1,
                     decodes=_log_uniform(rng, 8, 256), median=_log_uniform(rng, 256, 2048), kv_hi=8192, lengths=lengths)
    return _case("step", "tiny", 1, chunk=rng.choice([0, _log_uniform(rng, 5, 300)]), chunk_prefix=_log_uniform(rng, 1, 300) - 1,
                 decodes=_log_uniform(rng, 1, 40), kv="uniform", kv_lo=1, kv_hi=_log_uniform(rng, 17, 600), lengths=lengths)


@functools.lru_cache(maxsize=64)
def _lengths_of(chunk, chunk_prefix, n_chunks, decodes, kv, median, kv_lo, kv_hi, lengths):
    rng = np.random.Generator(np.random.PCG64([int(lengths), 86311, chunk, decodes]))
    spec = []
    if chunk > 0:
        # uneven pieces: every request gets at least one token
        cuts = np.sort(rng.choice(np.arange(1, chunk), size=n_chunks - 1, replace=False)) if n_chunks > 1 else np.zeros(0, dtype=np.int64)
        edges = [0] + [int(c) for c in cuts] + [chunk]
        spec += [(b - a, chunk_prefix + b - a) for a, b in zip(edges, edges[1:])]
    if kv == "uniform":
        spec += [(1, int(n)) for n in rng.integers(kv_lo, kv_hi, size=decodes, endpoint=True)]
    else:
        spec += [(1, int(n)) for n in W.lognormal_lengths(rng, decodes, median, 0.8, kv_lo, kv_hi)]
    return tuple(spec)


def _spec(case):
    """[(new tokens, KV length after the step)], prefill requests first."""
    return _lengths_of(*(case[k] for k in ("chunk", "chunk_prefix", "n_chunks", "decodes", "kv", "median", "kv_lo", "kv_hi", "lengths")))


def _layer_weights(m, n_layers, gen, device):
    """The weight matrices of one layer after another, drawn into the same buffers (the gains are ones)."""
    H, F, d = m["hidden"], m["ffn"], m["head_dim"]
    shapes = {"w_qkv": (H, (m["n_q"] + 2 * m["n_kv"]) * d), "w_o": (m["n_q"] * d, H), "w_gate": (H, F), "w_up": (H, F), "w_down": (F, H)}
    w = {k: torch.empty(s, dtype=torch.bfloat16, device=device) for k, s in shapes.items()}
    for _ in range(n_layers):
        for t in w.values():
            t.normal_(0.0, W.WEIGHT_STD, generator=gen)
        yield w


def _layer_prefixes(m, n_layers, prefixes, gen, device):
    """N(0, 1) keys and values of one layer after another; request i's are the rows from 16 i on."""
    rows = max(prefixes) + 16 * len(prefixes)
    k = torch.empty((rows, m["n_kv"], m["head_dim"]), dtype=torch.bfloat16, device=device)
    v = torch.empty_like(k)
    for _ in range(n_layers):
        k.normal_(generator=gen)
        v.normal_(generator=gen)
        yield k, v


def _head(m, gen, device):
    emb = torch.empty((VOCAB, m["hidden"]), dtype=torch.bfloat16, device=device).normal_(generator=gen)
    w_out = torch.empty((m["hidden"], VOCAB), dtype=torch.bfloat16, device=device).normal_(0.0, W.WEIGHT_STD, generator=gen)
    return emb, w_out


def _generator(seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(int(seed) * 1000003 + 17)
    return gen


def _load_layers(eng, n_layers, gen):
    one = torch.ones(eng.model["hidden"], dtype=torch.bfloat16, device=eng.device)
    for layer, w in enumerate(_layer_weights(eng.model, n_layers, gen, eng.device)):
        eng.ctx.init_layer(layer, g_attn=one.data_ptr(), g_ffn=one.data_ptr(), **{k: t.data_ptr() for k, t in w.items()})
    eng.ctx.sync()


def _load_prefixes(eng, n_layers, batch, gen):
    for layer, (k, v) in enumerate(_layer_prefixes(eng.model, n_layers, [s.prefix for s in batch], gen, eng.device)):
        step = k[0].numel() * k.element_size()
        for i, s in enumerate(batch):
            if s.prefix > 0:
                eng.ctx.kv_write(layer, s.pages, 0, s.prefix, k.data_ptr() + 16 * i * step, v.data_ptr() + 16 * i * step)
    eng.ctx.sync()


def prepare(case, seed):
    spec = _spec(case)
    gen = _generator(seed)
    layers, n_pages = case["layers"], [(kv + W.PAGE - 1) // W.PAGE for _, kv in spec]
    n_pool = sum(n_pages) + max(3, sum(n_pages) // 8)
    longest = max(kv for _, kv in spec) + W.PAGE
    perm = np.random.Generator(np.random.PCG64([int(seed), 715827883])).permutation(n_pool).astype(np.int32)
    batch, at = [], 0
    for i, ((n, kv), p) in enumerate(zip(spec, n_pages)):
        batch.append(W.SeqSpec(req_id=1000 + i, n_new=n, kv_len=kv, pages=perm[at:at + p].copy()))
        at += p
    eng = Engine(case["model"], n_pool, layers, layers, max_position=longest)
    _load_layers(eng, layers, gen)
    _load_prefixes(eng, layers, batch, gen)
    st = {"kind": case["kind"], "eng": eng, "batch": batch, "layers": layers}
    H, T = eng.model["hidden"], sum(n for n, _ in spec)
    if case["kind"] == "model":
        emb, w_out = _head(eng.model, gen, eng.device)
        g = torch.ones(H, dtype=torch.bfloat16, device=eng.device)
        eng.ctx.init_head(emb.data_ptr(), g.data_ptr(), w_out.data_ptr(), VOCAB)
        eng.ctx.sync()
        eng.vocab = VOCAB
        st["ids"] = W.token_ids(VOCAB, T, seed)
    else:
        st["x"] = torch.empty((T, H), dtype=torch.bfloat16, device=eng.device).normal_(generator=gen).view(torch.int16)
    if case["kind"] == "handoff":
        # the second instance: the same weights, an empty pool with pages of its own
        gen = _generator(seed)
        other = Engine(case["model"], n_pool, layers, layers, max_position=longest)
        _load_layers(other, layers, gen)
        st["other"] = other
        st["other_pages"] = perm[::-1][:n_pages[0]].copy()
    return st


def run(state):
    eng, kind = state["eng"], state["kind"]
    if kind == "step":
        out, _ = eng.step(state["batch"], state["x"])
        return out.view(torch.bfloat16)
    if kind == "static":
        out = torch.empty_like(state["x"])
        eng.ctx.step_static(state["batch"], state["x"].data_ptr(), out.data_ptr())
        return out.view(torch.bfloat16)
    if kind == "model":
        # The next token is the first maximum of a row of logits; the tokens themselves are not compared, since logits that
        # lie within rounding of each other are common.  The logit each token was picked for is.
        r = eng.step_tokens(state["batch"], state["ids"], want_logits=True, want_hidden=True)
        return {"logits": r["logits"], "hidden": r["hidden"], "picked": torch.gather(r["logits"], 1, r["next"].long()[:, None])}
    seq, other = state["batch"][0], state["other"]
    m, n = eng.model, seq.prefix
    k = torch.empty((state["layers"], n, m["n_kv"], m["head_dim"]), dtype=torch.bfloat16, device=eng.device)
    v = torch.empty_like(k)
    for layer in range(state["layers"]):
        eng.ctx.kv_read(layer, seq.pages, 0, n, k[layer].data_ptr(), v[layer].data_ptr())
        other.ctx.kv_write(layer, state["other_pages"], 0, n, k[layer].data_ptr(), v[layer].data_ptr())
    out, _ = other.step([W.SeqSpec(seq.req_id, seq.n_new, seq.kv_len, state["other_pages"])], state["x"])
    return {"k": k, "v": v, "x": out.view(torch.bfloat16)}


def work(case):
    """Each layer's weights and the attended keys and values read once, the new ones and the results written once; two
    operations per weight and token, four per attended key, query head and dimension."""
    m = W.MODELS[case["model"]]
    spec = _spec(case)
    H, F, d, nq, nkv, L = m["hidden"], m["ffn"], m["head_dim"], m["n_q"], m["n_kv"], case["layers"]
    T = sum(n for n, _ in spec)
    params = H * (nq + 2 * nkv) * d + nq * d * H + 3 * H * F
    kv_row = 2 * nkv * d * 2
    pairs = sum(n * (kv - n) + n * (n + 1) // 2 for n, kv in spec)
    flops = L * (2 * params * T + 4 * nq * d * pairs)
    nbytes = L * (2 * params + kv_row * (sum(kv - n for n, kv in spec) + T)) + 4 * T * H
    if case["kind"] == "model":
        flops += 2 * H * VOCAB * len(spec)
        nbytes += 2 * H * VOCAB + 4 * VOCAB * len(spec) + 2 * T * H
    if case["kind"] == "handoff":
        nbytes += L * 4 * kv_row * (spec[0][1] - spec[0][0])   # cache -> rows -> cache: two reads, two writes
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what two orders of summation differ by (K splits, tile edges and attention cuts forced to other values
    through the library's options), up to the comparison's own limit.  Seen over one to four layers, every T: rel
    0.0051-0.0066, max 0.018-0.037 of bf16 hidden states; over 32 layers: rel 0.015, max 0.07 of the logits; the tiny
    shape, whose K loops are too short to be cut, gave the same bits and gets a bf16 rounding flip per value."""
    if case["layers"] > 8:
        return {"rel": 0.03, "max": 0.3}
    if case["model"] == "tiny":
        return {"rel": 0.008, "max": 0.04}
    return {"rel": 0.025, "max": 0.15}


def _exact_layer(m, spec, w, k_pre, v_pre, x):
    """One layer of plain torch in 64 bits: pre-norm attention over each request's own prefix, SwiGLU; x is [T][hidden]."""
    d, nq, nkv = m["head_dim"], m["n_q"], m["n_kv"]
    half, dev = d // 2, x.device
    norm = lambda t: t * torch.rsqrt(t.square().mean(-1, keepdim=True) + W.RMS_EPS)
    pos = torch.cat([torch.arange(kv - n, kv, device=dev) for n, kv in spec]).double()
    theta = float(m["rope_base"]) ** (-2.0 * torch.arange(half, device=dev).double() / d)
    cos, sin = (pos[:, None] * theta).cos()[:, None], (pos[:, None] * theta).sin()[:, None]

    def rotate(t):
        lo, hi = t[..., :half], t[..., half:]
        return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)

    q, k, v = (norm(x) @ w["w_qkv"].double()).view(len(x), -1, d).split([nq, nkv, nkv], 1)
    q, k, out, at = rotate(q), rotate(k), torch.empty_like(q), 0
    for i, (n, kv) in enumerate(spec):
        pre = kv - n
        keys = torch.cat([k_pre[16 * i:16 * i + pre].double(), k[at:at + n]])
        values = torch.cat([v_pre[16 * i:16 * i + pre].double(), v[at:at + n]])
        allowed = torch.arange(kv, device=dev)[None] <= torch.arange(pre, kv, device=dev)[:, None]
        for h in range(nq):
            g = h // (nq // nkv)
            s = (q[at:at + n, h] @ keys[:, g].T / d ** 0.5).masked_fill_(~allowed, -float("inf"))
            out[at:at + n, h] = torch.softmax(s, -1) @ values[:, g]
        at += n
    x = x + out.reshape(len(x), nq * d) @ w["w_o"].double()
    y = norm(x)
    return x + (torch.nn.functional.silu(y @ w["w_gate"].double()) * (y @ w["w_up"].double())) @ w["w_down"].double()


def exact(case, seed):
    """The same inputs through plain torch in 64 bits, nothing rounded on the way.  The value of `picked` is left out: which
    of two logits that lie within rounding of each other it is taken at has no one answer."""
    m, spec, layers, dev = W.MODELS[case["model"]], _spec(case), case["layers"], torch.device("cuda:0")
    T = sum(n for n, _ in spec)
    gen = _generator(seed)
    for _ in _layer_weights(m, layers, gen, dev):   # only for the draws: the weights come again below
        pass
    cached = [(k.clone(), v.clone()) for k, v in _layer_prefixes(m, layers, [kv - n for n, kv in spec], gen, dev)]
    if case["kind"] == "model":
        emb, w_out = _head(m, gen, dev)
        x = emb[torch.from_numpy(np.asarray(W.token_ids(VOCAB, T, seed))).long().to(dev)].double()
    else:
        x = torch.empty((T, m["hidden"]), dtype=torch.bfloat16, device=dev).normal_(generator=gen).double()
    for w, (k, v) in zip(_layer_weights(m, layers, _generator(seed), dev), cached):
        x = _exact_layer(m, spec, w, k, v, x)
    if case["kind"] == "model":
        last = x[np.cumsum([n for n, _ in spec]) - 1]
        logits = (last * torch.rsqrt(last.square().mean(-1, keepdim=True) + W.RMS_EPS)) @ w_out.double()
        return {"logits": logits, "hidden": x, "picked": None}
    if case["kind"] == "handoff":
        n = spec[0][1] - spec[0][0]
        return {"k": torch.stack([k[:n] for k, _ in cached]).double(), "v": torch.stack([v[:n] for _, v in cached]).double(), "x": x}
    return x
