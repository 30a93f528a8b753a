"""The calls this framework is used for, as cases that can be timed and compared.

Each case is one call of the public entry points of ``paper_2408_07802_amd.kraken`` on a
model of a given shape: a prefill of packed prompts (with or without filling a KV cache),
a decode step over a KV cache, or the whole model from token ids to logits.  Most cases
are one layer of an architecture (a layer is the unit every larger model repeats); three
are whole models.  Values follow the repository's synthetic recipe: hidden rows ~ N(0, 1),
weights ~ N(0, 0.02), biases and LayerNorm parameters spread around their usual values.
"""

import math

import numpy as np
import torch

from paper_2408_07802_amd import kraken

DEVICE = "cuda"
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
NAMES = ("ln1_g", "ln1_b", "Wqkv", "bqkv", "Wo", "bo", "ln2_g", "ln2_b", "W1", "b1", "W2", "b2")


def case(call, lens, n_sub, d, heads, ff, storage="bf16", compute="f16", arch="kraken", layers=1,
         head_dim=0, kv_heads=0, vocab=0, **more):
    """A case.  lens: the prompts' lengths of a prefill, the cached tokens of each sequence
    of a decode step (a text, one number per sequence)."""
    return dict(call=call, lens=",".join(str(v) for v in lens), n_sub=n_sub, d=d, heads=heads,
                head_dim=head_dim or d // heads, kv_heads=kv_heads or heads, ff=ff,
                storage=storage, compute=compute, arch=arch, layers=layers, vocab=vocab, **more)


def listed():
    return [
        # the smallest whole model: bound by the number and latency of its launches
        case("prefill", [64], 2, 128, 4, 512, storage="f32", compute="f32", layers=2,
             name="prefill_f32_d128_s64"),
        # one prompt of 2048 tokens on a small Kraken layer with heads of 64
        case("prefill", [2048], 4, 768, 12, 3072, name="prefill_d768_s2048"),
        # eight prompts of very different lengths in one packed batch, heads of 64
        case("prefill", [2755, 1653, 3903, 817, 2210, 3377, 512, 2001], 4, 1280, 20, 5120,
             name="prefill_d1280_ragged8"),
        # the benchmark's layer: one 8192-token prompt, 8 sub-layers of width 2048
        case("prefill", [8192], 8, 2048, 16, 8192, name="prefill_d2048_s8192"),
        # a short prompt on the 4-way layer of the 65B engine: every weight used 128 times
        case("prefill", [128], 4, 4992, 39, 9984, storage="f16", name="prefill_d4992_s128"),
        # a handful of chat-sized prompts entering the KV cache, bf16 operands
        case("prefill_kv", [301, 97, 411, 36, 188], 4, 1024, 16, 4096, compute="bf16",
             name="prefill_kv_d1024_chat5_bf16"),
        # the parallel attention + FFN layer of the 6.7B engine on one 700-token prompt
        case("prefill", [700], 1, 4096, 32, 16384, storage="f16", arch="parallel",
             name="prefill_parallel_d4096_s700"),
        # time to first token of the whole 4-way 1.3B engine: width 1248, heads of 104, both
        # stored padded
        case("tokens", [128], 4, 1248, 12, 2496, storage="f16", layers=24, vocab=51200,
             name="tokens_kraken4_1b3_s128"),
        # a decode step of one long conversation on the benchmark's layer
        case("decode", [8191], 8, 2048, 16, 8192, name="decode_d2048_b1_ctx8191"),
        # a decode step of eight conversations of different lengths, grouped-query attention
        case("decode", [8000, 513, 4097, 2046, 7163, 1200, 5555, 3071], 8, 2048, 16, 8192,
             kv_heads=4, name="decode_gqa4_d2048_b8"),
        # a decode step of a large serving batch on a small layer, bf16 operands
        case("decode", [37 + (53 * b) % 900 for b in range(128)], 4, 1024, 16, 4096,
             compute="bf16", name="decode_d1024_b128_bf16"),
        # a decode step of the whole GPT-like 1.3B engine, one sequence: 24 layers of small
        # launches
        case("decode", [1023], 1, 2048, 16, 8192, storage="f16", arch="gpt", layers=24,
             name="decode_gpt_1b3_b1"),
    ]


# ------------------------------------------------------------------------------ drawn cases

def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more case: any call, architecture, type, width, head size, batch and length of the
    ranges above, no larger than the benchmark's layer."""
    while True:
        arch = rng.choice(["kraken", "kraken", "kraken", "gpt", "parallel"])
        n_sub = rng.choice([2, 4, 8]) if arch == "kraken" else 1
        call = rng.choice(["prefill", "prefill", "prefill_kv", "decode", "decode", "tokens"])
        storage, compute = rng.choice([("bf16", "f16"), ("bf16", "f16"), ("f16", "f16"),
                                       ("bf16", "bf16"), ("f32", "f32")])
        head_dim = rng.choice([32, 64, 64, 96, 104, 128, 128])
        heads = _log_int(rng, 2, 32)
        if head_dim == 32:
            heads += heads % 2
        d = heads * head_dim
        if rng.random() < 0.2:
            d += 4 * rng.randint(1, 8)               # a width that is not heads x head size
        group = rng.choice([1, 1, 2, 4])
        kv_heads = heads // group if heads % group == 0 else heads
        if (kv_heads * (32 if head_dim == 32 else 64)) % 64:
            kv_heads = heads
        ff = d * rng.choice([2, 4, 4])
        layers = rng.choice([1, 1, 2])
        if call == "decode":
            seqs = _log_int(rng, 1, 256)
            top = _log_int(rng, 1, 16384)
            lens = [rng.randint(0, top) for _ in range(seqs)]
        else:
            seqs = _log_int(rng, 1, 16)
            total = _log_int(rng, max(seqs, 5), 8192)
            cuts = sorted(rng.sample(range(1, total), seqs - 1))
            lens = [b - a for a, b in zip([0] + cuts, cuts + [total])]
        vocab = _log_int(rng, 1000, 51200) if call == "tokens" else 0
        c = case(call, lens, n_sub, d, heads, ff, storage, compute, arch, layers, head_dim,
                 kv_heads, vocab)
        if 128 <= d <= 5000 and cost(c) <= cost(listed()[3]) and cache_bytes(c) <= 1 << 30 \
                and weight_elems(c) <= 900e6:
            return c


# ------------------------------------------------------------------------------ sizes

def lens_of(c):
    return [int(v) for v in c["lens"].split(",")]


def rows_of(c):
    """Token rows of the call."""
    lens = lens_of(c)
    return len(lens) if c["call"] == "decode" else sum(lens)


def capacity_of(c):
    """Positions per slot of the case's KV cache."""
    return max(lens_of(c)) + 1


def widths(c):
    return c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]


def sub_elems(c):
    """Weight matrix elements of one sub-layer."""
    dq, dkv = widths(c)
    return c["d"] * (2 * dq + 2 * dkv + 2 * c["ff"])


def weight_elems(c):
    n = c["layers"] * c["n_sub"] * sub_elems(c) + c["vocab"] * c["d"]
    return n + (c["n_sub"] * c["d"] ** 2 if c["arch"] == "kraken" else 0)


def operand_bytes(c):
    return TORCH[c["compute"]].itemsize


def cache_bytes(c):
    if c["call"] not in ("decode", "prefill_kv"):
        return 0
    hd = 32 if c["head_dim"] <= 32 else 64 if c["head_dim"] <= 64 else 128
    return (c["layers"] * c["n_sub"] * 2 * len(lens_of(c)) * c["kv_heads"] * capacity_of(c) * hd *
            operand_bytes(c))


def cost(c):
    """A bound of the call's time that orders cases (fp32 matrix products run 16 times
    slower than 16-bit ones)."""
    w = work(c)
    return max(w["bytes"] / 4e12, w["flops"] * (16 if c["compute"] == "f32" else 1) / 1e15)


def work(c):
    T, d, lens = rows_of(c), c["d"], lens_of(c)
    dq, dkv = widths(c)
    es, ss = operand_bytes(c), TORCH[c["storage"]].itemsize
    LN = c["layers"] * c["n_sub"]
    flops = 2.0 * LN * T * sub_elems(c)
    nbytes = float(weight_elems(c) * es)
    if c["arch"] == "kraken":
        flops += 2.0 * T * c["n_sub"] * d * d
    if c["call"] == "decode":
        flops += LN * 4.0 * dq * sum(n + 1 for n in lens)
        nbytes += LN * 2.0 * dkv * es * (sum(lens) + T)           # cached rows in, new ones out
    else:
        flops += LN * 4.0 * dq * sum(n * (n + 1) / 2.0 for n in lens)
        if c["call"] == "prefill_kv":
            nbytes += LN * 2.0 * dkv * es * T
    if c["call"] == "tokens":
        flops += 2.0 * len(lens) * d * c["vocab"]
        nbytes += 4.0 * T + 4.0 * len(lens) * c["vocab"]
    else:
        nbytes += T * d * (ss + 4.0)
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------------------ inputs

def _config(c):
    T = rows_of(c)
    return kraken.Config(
        n_sub=c["n_sub"], n_layers=c["layers"], d_model=c["d"], n_heads=c["heads"],
        d_ff=c["ff"], max_tokens=max(T, 2048) if c["call"] == "decode" else T,
        dtype=c["storage"], compute=c["compute"], arch=c["arch"], head_dim=c["head_dim"],
        n_kv_heads=c["kv_heads"], vocab=c["vocab"],
        max_positions=max(lens_of(c)) if c["vocab"] else 0)


def _inputs(c, seed):
    """Weights, embeddings and call inputs of a case, from the seed alone."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    st = TORCH[c["storage"]]
    d, ff = c["d"], c["ff"]
    dq, dkv = widths(c)

    def normal(shape, std, mean=0.0, dtype=st):
        return torch.empty(shape, dtype=dtype, device=DEVICE).normal_(mean, std, generator=g)

    def sub_layer():
        shapes = {"Wqkv": (d, dq + 2 * dkv), "bqkv": (dq + 2 * dkv,), "Wo": (dq, d), "bo": (d,),
                  "W1": (d, ff), "b1": (ff,), "W2": (ff, d), "b2": (d,)}
        p = {}
        for name in NAMES:
            if name in shapes:
                p[name] = normal(shapes[name], 0.02)
            elif c["arch"] != "parallel" or not name.startswith("ln2"):
                p[name] = normal((d,), 0.1, 1.0) if name.endswith("_g") else normal((d,), 0.02)
        return p

    x = {"layers": [[sub_layer() for _ in range(c["n_sub"])] for _ in range(c["layers"])],
         "w_concat": normal((c["n_sub"] * d, d), 0.02) if c["arch"] == "kraken" else None,
         "embeddings": None}
    lens = lens_of(c)
    if c["vocab"]:
        x["embeddings"] = {"tok_emb": normal((c["vocab"], d), 0.02),
                           "pos_emb": normal((max(lens), d), 0.02),
                           "lnf_g": normal((d,), 0.1, 1.0), "lnf_b": normal((d,), 0.02)}
    if c["call"] == "tokens":
        rng = np.random.default_rng(seed)
        x["ids"] = rng.integers(0, c["vocab"], size=sum(lens)).astype(np.int32)
    else:
        x["hidden"] = normal((rows_of(c), d), 1.0)
    if cache_bytes(c):
        hd = 32 if c["head_dim"] <= 32 else 64 if c["head_dim"] <= 64 else 128
        shape = (c["layers"], c["n_sub"], 2, len(lens), c["kv_heads"], capacity_of(c), hd)
        dt = TORCH[c["compute"]]
        if c["call"] == "decode":
            x["cache"] = normal(shape, 1.0, dtype=dt)
            x["cache"][..., c["head_dim"]:] = 0       # a padded head's extra features
        else:
            x["cache"] = torch.zeros(shape, dtype=dt, device=DEVICE)
    return x


def prepare(c, seed):
    x = _inputs(c, seed)
    cfg = _config(c)
    model = kraken.Kraken(cfg)
    model.load_weights(kraken.pack_weights(x["layers"], x["w_concat"], cfg, device=DEVICE,
                                           embeddings=x["embeddings"]))
    s = {"call": c["call"], "model": model, "cfg": cfg, "lens": lens_of(c)}
    if c["call"] == "decode":
        s["hidden"] = x["hidden"]
    else:
        s["cu"] = kraken.cu_from_lens(lens_of(c))
        s["input"] = x["ids"] if c["call"] == "tokens" else x["hidden"]
    if "cache" in x:
        s["cache"] = kraken.KVCache(x["cache"].view(torch.uint8).reshape(-1), len(lens_of(c)),
                                    capacity_of(c))
    return s


def run(s):
    model = s["model"]
    if s["call"] == "prefill":
        return model.prefill(s["input"], s["cu"])[0]
    if s["call"] == "tokens":
        return model.forward_tokens(s["input"], s["cu"])[0]
    if s["call"] == "prefill_kv":
        out = model.prefill_kv(s["input"], s["cu"], s["cache"])[0]
    else:
        out = model.decode(s["hidden"], s["lens"], s["cache"])[0]
    return {"out": out, "cache": s["cache"].view(s["cfg"])}


# ------------------------------------------------------------------------------ correctness

# Bound of one layer's relative error by operand type: about four times what the listed and
# some drawn cases show against fp64 (fp32 up to 2.3e-6, fp16 4.4e-4, bf16 2.3e-3).
LAYER_REL = {"f32": 1e-5, "f16": 1.5e-3, "bf16": 1e-2}


def tolerance(c):
    rel = LAYER_REL[c["compute"]] * math.sqrt(c["layers"])
    return {"rel": rel, "max": 20 * rel}


def exact(c, seed):
    """The call in fp64: pre-LN layers, causal attention per sequence, exact GELU."""
    if c["layers"] * c["n_sub"] * c["heads"] * len(lens_of(c)) > 50000:
        return None                                   # too many single heads to go through
    x = _inputs(c, seed)
    d, H, Hkv, hd, N = c["d"], c["heads"], c["kv_heads"], c["head_dim"], c["n_sub"]
    dq, dkv = widths(c)
    lens, decode = lens_of(c), c["call"] == "decode"
    f64 = torch.float64
    cache = x["cache"].to(f64) if "cache" in x else None

    def norm(v, gain, bias):
        mean = v.mean(-1, keepdim=True)
        var = ((v - mean) ** 2).mean(-1, keepdim=True)
        return (v - mean) / torch.sqrt(var + 1e-5) * gain.to(f64) + bias.to(f64)

    def affine(v, weight, bias):
        return v @ weight.to(f64) + bias.to(f64)

    def attend(q, k, v, causal):                        # [rows, hd] of one head
        s = q @ k.T / math.sqrt(hd)
        if causal:
            s.masked_fill_(torch.ones(s.shape, dtype=torch.bool, device=DEVICE).triu_(1),
                           -math.inf)
        return torch.softmax(s, -1) @ v

    def attention(u, p, j, i):
        qkv = affine(u, p["Wqkv"], p["bqkv"])
        out = torch.empty((u.shape[0], dq), dtype=f64, device=DEVICE)
        row = 0
        for b, n in enumerate(lens):
            rows = 1 if decode else n
            for h in range(H):
                kh = h // (H // Hkv)
                part = qkv[row:row + rows]
                q = part[:, h * hd:(h + 1) * hd]
                k = part[:, dq + kh * hd:dq + (kh + 1) * hd]
                v = part[:, dq + dkv + kh * hd:dq + dkv + (kh + 1) * hd]
                if cache is not None:
                    at = n if decode else 0
                    cache[j, i, 0, b, kh, at:at + rows, :hd] = k
                    cache[j, i, 1, b, kh, at:at + rows, :hd] = v
                    if decode:
                        k = cache[j, i, 0, b, kh, :n + 1, :hd]
                        v = cache[j, i, 1, b, kh, :n + 1, :hd]
                out[row:row + rows, h * hd:(h + 1) * hd] = attend(q, k, v, not decode)
            row += rows
        return affine(out, p["Wo"], p["bo"])

    def ffn(u, p):
        return affine(torch.nn.functional.gelu(affine(u, p["W1"], p["b1"])), p["W2"], p["b2"])

    if c["call"] == "tokens":
        e = x["embeddings"]
        # token rows are held in the operand type
        tok = e["tok_emb"].to(TORCH[c["compute"]]).to(f64)
        pos = torch.cat([torch.arange(n, device=DEVICE) for n in lens])
        X = tok[torch.from_numpy(x["ids"]).to(DEVICE).long()] + e["pos_emb"].to(f64)[pos]
    else:
        X = x["hidden"].to(f64)
    subs = [X] * N
    for j, layer in enumerate(x["layers"]):
        y = X if j == 0 else sum(subs)
        new = []
        for i, p in enumerate(layer):
            u = norm(subs[i], p["ln1_g"], p["ln1_b"])
            h = subs[i] + attention(u, p, j, i)
            if c["arch"] == "kraken":
                u = norm(h + y, p["ln2_g"], p["ln2_b"])
            elif c["arch"] == "gpt":
                u = norm(h, p["ln2_g"], p["ln2_b"])
            new.append(h + ffn(u, p))
        subs = new
    out = subs[0]
    if c["arch"] == "kraken":
        out = torch.cat(subs, 1) @ x["w_concat"].to(f64)
    if c["call"] == "tokens":
        last = torch.tensor(lens, device=DEVICE).cumsum(0) - 1
        return norm(out[last], e["lnf_g"], e["lnf_b"]) @ tok.T
    return out if cache is None else {"out": out, "cache": cache}
