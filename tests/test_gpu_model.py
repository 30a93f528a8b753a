"""The whole model and the comparison architectures (through the C ABI) against the fp64
oracle.

* Widths and head sizes the kernels do not have natively (the paper's engine table uses
  d = 1248, 3120, 5472 and heads of 72, 96 and 104) run stored in padded widths; the
  results must be those of the logical model (``O.kraken_prefill`` on unpadded weights).
* The GPT-like and the parallel attention + FFN stacks the paper compares with (Section
  4.3) run from the same kernels: ``O.stack_forward``.
* ``kraken_forward_tokens``: embeddings, stack, W_concat, final LayerNorm and the tied
  unembedding, the logits of each sequence's last token against ``O.model_forward``,
  including the engine shapes of the 1.3B, 6.7B and 13B models at full depth.

Metric as in the prefill tests: max |gpu - oracle| / RMS(oracle), bound 2e-2 for 16-bit
storage and 1e-4 for fp32.
"""

import dataclasses
import sys

import numpy as np
import pytest
import torch

from oracle import kraken_oracle as O
from paper_2408_07802_amd import synth
from test_gemm_plans import F16, F32, RES, plan

pytestmark = pytest.mark.gpu

DEV = "cuda"
TOL = {"bf16": 2e-2, "f16": 2e-2, "f32": 1e-4}


def K():
    from paper_2408_07802_amd import kraken
    return kraken


def f64(t):
    return t.detach().double().cpu().numpy()


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def rel_err(got, ref):
    ref = np.asarray(ref)
    return float(np.max(np.abs(np.asarray(got) - ref)) / np.sqrt(np.mean(ref ** 2)))


def cfg_of(w, T):
    return K().Config(n_sub=w.n_sub, n_layers=w.n_layers, d_model=w.d_model, n_heads=w.n_heads,
                      d_ff=w.d_ff, max_tokens=T, dtype=w.dtype, compute=w.compute,
                      n_kv_heads=w.n_kv_heads, arch=w.arch, head_dim=w.head_size,
                      vocab=w.vocab, max_positions=w.max_positions)


def build_model(w, T, seed=0, affine="plain"):
    cfg = cfg_of(w, T)
    model = K().Kraken(cfg)
    layers = (synth.gen_layer(w, j, seed, DEV, affine) for j in range(w.n_layers))
    wc = synth.gen_w_concat(w, seed, DEV) if w.arch == "kraken" else None
    emb = synth.gen_embeddings(w, seed, DEV, affine) if w.vocab else None
    blob = K().pack_weights(layers, wc, cfg, device=DEV, embeddings=emb)
    model.load_weights(blob)
    torch.cuda.synchronize()
    del blob
    return model


def oracle_layers(w, seed=0, affine="plain", progress=False):
    for j in range(w.n_layers):
        if progress and j % 8 == 0:
            say(f"      oracle layer {j + 1}/{w.n_layers}")
        yield [{k: f64(v) for k, v in sub.items()}
               for sub in synth.gen_layer(w, j, seed, DEV, affine)]


def oracle_wc(w, seed=0):
    return f64(synth.gen_w_concat(w, seed, DEV)) if w.arch == "kraken" else None


def small(name, **kw):
    base = dict(name=name, n_sub=2, n_layers=2, d_model=128, n_heads=4, d_ff=512, dtype="bf16")
    base.update(kw)
    return synth.Workload(**base)


def prefill_vs_oracle(w, lens, affine="random", seed=0):
    cu = synth.cu_seqlens(lens)
    T = cu[-1]
    say(f"[model prefill] {w.name} arch={w.arch} d={w.d_model} H={w.n_heads} hd={w.head_dim} "
        f"F={w.d_ff} N={w.n_sub} {w.dtype}/{w.compute} lens={lens}")
    model = build_model(w, T, seed, affine)
    X = synth.gen_hidden(w, T, seed, DEV)
    model.poison_workspace()
    out, sub = model.prefill(X, cu, sub_out=True)
    model.sync()
    model.poison_workspace()
    plain, _ = model.prefill(X, cu)      # (another tail of the pass, the same sums)
    model.sync()
    model.close()
    assert torch.equal(plain, out), "out without sub_out != out with it"
    ref = O.stack_forward(f64(X), cu, w.arch, list(oracle_layers(w, seed, affine)), w.n_heads,
                          oracle_wc(w, seed), head_dim=w.head_size or None,
                          n_kv_heads=w.kv_heads)
    e = rel_err(f64(out), ref)
    say(f"    max|err|/rms out {e:.3e} (bound {TOL[w.dtype]})")
    assert e <= TOL[w.dtype], e
    if w.arch == "kraken":
        _, sub_o = O.kraken_prefill(f64(X), cu, list(oracle_layers(w, seed, affine)),
                                    oracle_wc(w, seed), w.n_heads, n_kv_heads=w.kv_heads,
                                    head_dim=w.head_size or None)
        es = rel_err(f64(sub), sub_o)
        say(f"    sub_out {es:.3e}")
        assert es <= TOL[w.dtype], es
    else:
        assert torch.equal(sub[0], out)      # one sub-layer: sub_out is the output


# ----------------------------------------------------------- padded widths and head sizes

PADDED = [  # d, heads, kv heads, dtype, compute: head sizes 104, 96, 72 and widths 1248-like
    (208, 2, 0, "f32", "storage"),       # hd 104 -> 128, d 208 -> 256
    (208, 2, 0, "bf16", "f16"),
    (192, 2, 0, "bf16", "storage"),      # hd 96 -> 128
    (144, 2, 0, "f32", "storage"),       # hd 72 -> 128, d 144 -> 192
    (416, 4, 2, "bf16", "f16"),          # grouped-query, hd 104
    (200, 5, 0, "bf16", "f16"),          # hd 40 -> 64, d 200 -> 256
]


@pytest.mark.parametrize("case", PADDED, ids=[f"d{c[0]}-h{c[1]}-kv{c[2]}-{c[3]}-{c[4]}" for c in PADDED])
def test_padded_widths_give_the_logical_model(case):
    d, H, Hkv, dtype, compute = case
    w = small(f"pad-d{d}-h{H}", d_model=d, n_heads=H, n_kv_heads=Hkv, d_ff=2 * d, dtype=dtype,
              compute=compute)
    prefill_vs_oracle(w, [130, 7, 300])


def test_padded_widths_decode_after_prefill_kv():
    # the KV cache of a padded model holds the stored head size; a decode step over it is
    # the last row of the extended prefill
    w = small("pad-decode", d_model=208, n_heads=2, d_ff=416, compute="f16")
    lens = [40, 9]
    cu = synth.cu_seqlens(lens)
    model = build_model(w, cu[-1], affine="random")
    cache = model.new_kv_cache(2, 64)
    X = synth.gen_hidden(w, cu[-1], 0, DEV)
    model.prefill_kv(X, cu, cache)
    Xn = synth.gen_hidden(w, 2, 1, DEV)
    model.poison_workspace()
    out, _ = model.decode(Xn, lens, cache)
    model.sync()
    model.close()
    layers = list(oracle_layers(w, 0, "random"))
    _, _, kv = O.kraken_prefill(f64(X), cu, layers, oracle_wc(w), w.n_heads, return_kv=True)
    out_o, _, _ = O.kraken_decode(f64(Xn), O.split_kv(kv, cu), layers, oracle_wc(w), w.n_heads)
    e = rel_err(f64(out), out_o)
    say(f"[padded decode] max|err|/rms {e:.3e}")
    assert e <= 2e-2


# ------------------------------------------------------------ the comparison architectures

@pytest.mark.parametrize("arch", ["gpt", "parallel"])
@pytest.mark.parametrize("dtype,compute", [("f32", "storage"), ("bf16", "f16")])
def test_comparison_architectures(arch, dtype, compute):
    w = small(f"{arch}-d256", n_sub=1, n_layers=3, d_model=256, n_heads=4, d_ff=1024,
              dtype=dtype, compute=compute, arch=arch)
    prefill_vs_oracle(w, [1, 200, 77])


@pytest.mark.parametrize("arch", ["gpt", "parallel", "kraken"])
def test_head_size_other_than_width_over_heads(arch):
    # the GPT-3 13B shape in small: d = 320 (stored 320), 2 heads of 128 (query width 256)
    w = small(f"{arch}-hd128-d320", n_sub=1 if arch != "kraken" else 2, n_layers=2, d_model=320,
              n_heads=2, d_ff=640, compute="f16", arch=arch, head_size=128)
    prefill_vs_oracle(w, [150, 33])


@pytest.mark.parametrize("arch", ["gpt", "parallel"])
@pytest.mark.parametrize("dtype,compute", [("f32", "storage"), ("bf16", "f16")])
def test_split_last_projection_of_the_comparison_architectures(arch, dtype, compute):
    """Few columns and a long reduction: the last FFN-down is split, and
    without sub_out the launch that sums its planes writes the caller's rows itself.  Prompts of
    20 and 130 rows, then a decode step, whose row equals that of the longer prompt."""
    w = small(f"{arch}-d256-f8192", n_sub=1, n_layers=2, d_model=256, n_heads=4, d_ff=8192,
              dtype=dtype, compute=compute, arch=arch)
    dt = F32 if dtype == "f32" else F16
    for T in (2, 20, 130):
        assert plan(dt, RES, T, 256, 8192, 1, 1, T * 256 * 4, own_sum=True).splits > 1, T
    prefill_vs_oracle(w, [20])
    prefill_vs_oracle(w, [100, 30])
    lens = [40, 9]
    cu = synth.cu_seqlens(lens)
    model = build_model(w, cu[-1], affine="random")
    cache = model.new_kv_cache(2, 64)
    X = synth.gen_hidden(w, cu[-1], 0, DEV)
    model.prefill_kv(X, cu, cache)
    Xn = synth.gen_hidden(w, 2, 1, DEV)
    model.poison_workspace()
    out, sub = model.decode(Xn, lens, cache, sub_out=True)
    model.poison_workspace()
    plain, _ = model.decode(Xn, lens, cache)
    model.sync()
    model.close()
    assert torch.equal(plain, out) and torch.equal(sub[0], out)
    longer = [v + 1 for v in lens]
    cu1 = synth.cu_seqlens(longer)
    X1 = torch.cat([t for b in range(2) for t in (X[cu[b]:cu[b + 1]], Xn[b:b + 1])])
    ref = O.stack_forward(f64(X1), cu1, arch, list(oracle_layers(w, 0, "random")), w.n_heads)
    e = rel_err(f64(plain), ref[[c - 1 for c in cu1[1:]]])
    say(f"[split decode] {arch} {dtype} max|err|/rms {e:.3e}")
    assert e <= TOL[dtype]


# --------------------------------------------------------------- token in, logits out

def logits_vs_oracle(w, lens, affine="random", seed=0, hidden=True):
    cu = synth.cu_seqlens(lens)
    T = cu[-1]
    say(f"[model tokens] {w.name} arch={w.arch} N={w.n_sub} L={w.n_layers} d={w.d_model} "
        f"H={w.n_heads} hd={w.head_dim} V={w.vocab} {w.dtype}/{w.compute} lens={lens}")
    model = build_model(w, T, seed, affine)
    ids = synth.gen_tokens(w, T, seed)
    model.poison_workspace()
    logits, hid = model.forward_tokens(ids, cu, hidden_out=hidden)
    model.sync()
    model.close()
    emb = {k: f64(v) for k, v in synth.gen_embeddings(w, seed, DEV, affine).items()}
    say("    oracle")
    lo, ho = O.model_forward(ids, cu, w.arch, oracle_layers(w, seed, affine, progress=True), emb,
                             w.n_heads, W_concat=oracle_wc(w, seed),
                             head_dim=w.head_size or None, n_kv_heads=w.kv_heads)
    e = rel_err(f64(logits), lo)
    msg = f"    logits max|err|/rms {e:.3e}"
    if hidden:
        eh = rel_err(f64(hid), ho)
        msg += f", hidden {eh:.3e}"
        assert eh <= TOL[w.dtype], eh
    say(msg + f" (bound {TOL[w.dtype]})")
    assert e <= TOL[w.dtype], e
    # the most likely next token agrees wherever the oracle's top two are apart
    top = np.argsort(lo, axis=1)[:, -2:]
    gap = lo[np.arange(len(lo)), top[:, 1]] - lo[np.arange(len(lo)), top[:, 0]]
    clear = gap > 4 * TOL[w.dtype] * np.sqrt(np.mean(lo ** 2))
    assert np.array_equal(np.argmax(f64(logits), axis=1)[clear], top[clear, 1])


@pytest.mark.parametrize("arch", ["kraken", "gpt", "parallel"])
@pytest.mark.parametrize("dtype,compute", [("f32", "storage"), ("bf16", "f16")])
def test_forward_tokens_small(arch, dtype, compute):
    w = small(f"tok-{arch}", n_sub=3 if arch == "kraken" else 1, d_model=208, n_heads=2,
              d_ff=416, dtype=dtype, compute=compute, arch=arch, vocab=777, max_positions=320)
    logits_vs_oracle(w, [300, 1, 64])


def test_forward_tokens_full_vocabulary():
    # the paper's 51,200-token vocabulary (Section 4.3), a ragged batch of 5 prompts
    w = small("tok-v51200", n_sub=4, d_model=256, n_heads=2, d_ff=512, compute="f16",
              vocab=51200, max_positions=2048)
    logits_vs_oracle(w, [128, 7, 300, 1, 64])


def test_forward_tokens_rejects_bad_ids_and_lengths():
    w = small("tok-err", n_sub=1, d_model=128, n_heads=2, d_ff=256, vocab=50, max_positions=8,
              arch="gpt")
    model = build_model(w, 16)
    kr = K()
    for ids, cu in [([0, 1, 50], [0, 3]), ([-1, 1, 2], [0, 3]), (list(range(9)), [0, 9])]:
        with pytest.raises(kr.KrakenError) as ei:
            model.forward_tokens(ids, cu)
        assert ei.value.status == kr.ERR_INVALID_ARG
    plain = build_model(small("no-emb", n_sub=1, arch="gpt"), 8)
    with pytest.raises(kr.KrakenError) as ei:
        plain.forward_tokens([0, 1], [0, 2])
    assert ei.value.status == kr.ERR_STATE
    model.close()
    plain.close()


# ----------------------------------------------------- buffers aligned to their elements alone

def offset_by_one(shape, dtype, fill):
    """A contiguous tensor one element past an aligned address, with the elements around it."""
    n = int(np.prod(shape))
    whole = torch.full((n + 2,), fill, dtype=dtype, device=DEV)
    return whole, whole[1:n + 1].view(shape)


@pytest.mark.parametrize("arch", ["kraken", "gpt", "parallel"])
@pytest.mark.parametrize("d,dtype", [(1024, "bf16"), (1000, "bf16"), (1024, "f32")])
def test_buffers_need_no_alignment_beyond_their_elements(arch, d, dtype):
    """Input and output one element past an aligned address, at row counts of each kind of
    kernel, where the last FFN-down or W_concat leaves planes that a launch of its own sums (into
    hidden_out, for the GPT-like and parallel stacks): the bits of the aligned call, and nothing
    written beside the rows.  (d = 1000 is stored 1024 wide; W_concat's plan for the stored rows
    may add in another order.)"""
    w = small(f"align-{arch}", n_sub=4 if arch == "kraken" else 1, n_layers=1, d_model=d, n_heads=8,
              head_size=128, d_ff=4096, dtype=dtype, compute="f16" if dtype == "bf16" else "storage",
              arch=arch)
    model = build_model(w, 300)
    for T in (3, 40, 130, 300):
        X = synth.gen_hidden(w, T, 1, DEV)
        ref, _ = model.prefill(X, [0, T])
        if dtype == "bf16":                # (an fp32 input is read where it is, in whole rows)
            _, Xu = offset_by_one(X.shape, X.dtype, 0)
            Xu.copy_(X)
        else:
            Xu = X
        whole, out = offset_by_one((T, d), torch.float32, 7.0)
        model.poison_workspace()
        model.prefill(Xu, [0, T], out=out)
        model.sync()
        say(f"[alignment] {arch} d={d} {dtype} T={T}")
        assert whole[0] == 7.0 and whole[-1] == 7.0
        if d % 64 == 0:
            assert torch.equal(out, ref)
        else:
            assert rel_err(f64(out), f64(ref)) <= 1e-5
    model.close()


def test_logits_need_no_alignment():
    # 40 and 100 sequences: the streaming kernel's rows, a vocabulary of whole groups of four
    w = small("align-tok", n_sub=1, n_layers=1, d_model=256, n_heads=2, d_ff=512, compute="f16",
              arch="gpt", vocab=6000, max_positions=8)
    model = build_model(w, 100)
    for B in (40, 100):
        ids, cu = synth.gen_tokens(w, B, 3), list(range(B + 1))
        ref, _ = model.forward_tokens(ids, cu)
        whole, logits = offset_by_one((B, w.vocab), torch.float32, 7.0)
        model.forward_tokens(ids, cu, logits=logits)
        model.sync()
        assert whole[0] == 7.0 and whole[-1] == 7.0 and torch.equal(logits, ref)
    model.close()


# ------------------------------------------ the paper's engine shapes (Section 4.3), full depth

ENGINE_CASES = [(m, a) for m in ("1.3b", "6.7b", "13b") for a in ("kraken4", "kraken8")] + \
               [("1.3b", "gpt"), ("1.3b", "parallel"), ("13b", "gpt")]


@pytest.mark.timeout(900)
@pytest.mark.parametrize("model,arch", ENGINE_CASES, ids=[f"{m}-{a}" for m, a in ENGINE_CASES])
def test_engine_shapes_128_token_prompt(model, arch):
    """Every layer of the engine (fp16, vocabulary 51,200) on one 128-token prompt; the
    last token's logits and every hidden row against the oracle."""
    w = synth.engine_workload(model, arch, 128)
    logits_vs_oracle(w, [128], affine="plain")


@pytest.mark.timeout(900)
@pytest.mark.parametrize("arch", ["gpt", "kraken8"])
def test_175b_engine_widths_two_layers(arch):
    """The 175B engines' widths at two layers: the GPT-like d = 12288 (LayerNorm rows of 12
    float4 per thread, FFN 49152 wide) and the 8-way Kraken d = 5472 (57 heads of 96,
    padded to 5504 and 128), fp16, one 64-token prompt."""
    w = synth.engine_workload("175b", arch, 64, layers=2)
    logits_vs_oracle(w, [64], affine="plain")
