"""Cases for measuring the library from the outside: whole translations and generations through `Engine`.

A case names a model of `lsq_synth`, a batch and its lengths, and the way the caller waits.  A pass is what one
request costs a user: source ids from host memory, encoder or prompt prefill, every decode step, results on the host.

Weights.  Matrices drawn from N(0, s^2) alone give an almost flat distribution over the vocabulary, which no trained
model has: there the last bits of a sum decide which of many equally good tokens is taken, and two correct programs
part after a few steps.  The models here are random too, but hold what a trained one is for: 256 tokens whose rows of
the embedding are orthogonal, and in the last feed-forward layer one hidden unit per such token, which sees the token
in the hidden row and adds its likely successors (one clear favourite, three alternatives 1 to 25 nats behind, at
distances that differ from token to token).  The last cross-attention copies: the token that makes up half of a
source sentence decides how its translation begins.  Every other matrix is random, and everything is computed at
full size; the rest of the network moves a hypothesis' score by a few per cent.
"""
from __future__ import annotations

import dataclasses
import functools
import math
import statistics

import numpy as np
import torch

import lsq_synth as S
import paper_2010_13887_amd as lsq

ACTIVE = 256        # tokens that have successors
FIRST = 4           # the first of them: ids 0..3 are special
GPT2S = dict(arch=1, n_enc=0, n_dec=12, d_model=768, n_heads=12, d_ffn=3072, vocab=50257, dtype=1, max_pos=256, act=1, norm=1)
SHAPES = {"tiny": dict(max_pos=64), "base": S.BASE, "big": S.BIG, "gpt2s": GPT2S}


def _case(name, model, batch, **kw):
    """Lengths between len_lo and len_hi (a prompt: len_hi), up to `new` tokens more in the output; groups > 1: diverse
    beam search; topk > 0: sampling; wait: decode steps between two waits for the count of unfinished sentences."""
    c = dict(name=name, model=model, dtype="f16", batch=batch, beam=4, len_law="uniform", len_lo=10, len_hi=60, new=50,
             topk=0, topp=1.0, groups=1, strength=0.0, wait=64)
    if model == "gpt2s":
        c.update(beam=1, len_law="fixed", topk=8)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest model and the shortest call: what the path costs when there is next to nothing to compute
        _case("tiny_f32", "tiny", 2, dtype="f32", len_lo=5, len_hi=8, new=0, wait=1),
        # one sentence, somebody waits for it: translate() as it comes, a wait after every step
        _case("base_1", "base", 1, len_lo=25, len_hi=25, wait=1),
        _case("big_1", "big", 1, len_lo=31, len_hi=31, wait=1),
        # a small batch on Transformer-base
        _case("base_8", "base", 8),
        # the same in float32
        _case("base_8_f32", "base", 8, dtype="f32"),
        # diverse beam search, an odd batch and three groups of two
        _case("base_5_diverse", "base", 5, beam=6, groups=3, strength=3.5, len_lo=7, len_hi=47),
        # text generation from an encoder-decoder model: top-k / top-p sampling
        _case("base_32_sampled", "base", 32, beam=1, topk=32, topp=0.75),
        # Transformer-big, a medium batch
        _case("big_32", "big", 32),
        # Transformer-big, a full batch of sentences of very different lengths: bulk translation
        _case("big_128", "big", 128, len_law="lognormal", len_lo=1, len_hi=128),
        # decoder-only model: one prompt, and a batch of them
        _case("gpt2s_1", "gpt2s", 1, len_hi=33, new=64, wait=1),
        _case("gpt2s_32", "gpt2s", 32, len_hi=64, new=128),
        # long prompts, short answers: mostly prefill
        _case("gpt2s_32_prefill", "gpt2s", 32, len_hi=240, new=16),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["base", "base", "base", "big", "big", "gpt2s", "gpt2s", "base_f32", "sampled", "diverse", "tiny"])
    wait = rng.choice([1, 16, 64])
    if kind == "gpt2s":
        prompt, new = rng.randint(2, 200), _log_int(rng, 4, 56)
        c = _case("", "gpt2s", _log_int(rng, 1, 64), len_hi=prompt, new=new, wait=wait, topk=rng.choice([1, 8, 32]), topp=rng.choice([0.75, 1.0]))
    elif kind == "tiny":
        c = _case("", "tiny", _log_int(rng, 1, 32), dtype=rng.choice(["f16", "f32"]), beam=rng.randint(1, 8), len_lo=1,
                  len_hi=rng.randint(2, 40), new=rng.randint(0, 20), wait=wait)
    else:
        lo = rng.randint(1, 40)
        c = _case("", "big" if kind == "big" else "base", _log_int(rng, 1, 32 if kind == "base_f32" else 100), beam=rng.randint(1, 5),
                  len_lo=lo, len_hi=rng.randint(lo, 60), new=rng.randint(5, 50), wait=wait)
        if kind == "base_f32":
            c.update(dtype="f32")
        elif kind == "sampled":
            c.update(beam=1, topk=rng.choice([4, 8, 32]), topp=rng.choice([0.75, 0.9, 1.0]))
        elif kind == "diverse":
            groups, of = rng.choice([(2, 2), (2, 3), (3, 1), (4, 2)])
            c.update(beam=groups * of, groups=groups, strength=3.5, batch=min(c["batch"], 48))
    del c["name"]
    return c


# ---- the model ---------------------------------------------------------------------------------
def _hparams(case):
    return S.HParams(**{**SHAPES[case["model"]], "dtype": int(case["dtype"] == "f16"), "cap_extra": case["new"],
                        "sample_topk": case["topk"], "sample_topp": case["topp"]})


@functools.lru_cache(maxsize=8)
def _tensors(hp):
    """The tensors that carry the successors (see the top of the file), by name."""
    d, F, n = hp.d_model, hp.d_ffn, min(ACTIVE, hp.d_model // 2)
    rng = np.random.Generator(np.random.PCG64(hp.seed + 1))
    gpt = hp.arch == 1
    std = 1.0 if gpt else 50.0 / d        # of the embedding: logits of a unit row reach 50 (decoder-only: through lnf_g)
    E = rng.standard_normal((hp.vocab, d), dtype=np.float32) * np.float32(std)
    q = np.linalg.qr(rng.standard_normal((d, n)))[0].T.astype(np.float32)     # unit rows
    E[FIRST:FIRST + n] = q * np.float32(std * math.sqrt(d))
    i = np.arange(n)
    u = np.modf(i * 0.6180339887)[0]
    behind = 1.2 + 7.0 * u                                                    # well apart along a chain of successors
    if hp.sample_topp < 1:
        behind = np.where(u < 0.1, 0.3 + 2.0 * u, 0.3 + behind)               # a nucleus needs open choices too
    weight = 1.0 - np.stack([0 * behind, behind, behind + 4, behind + 9]) / 25.0
    value = sum(weight[j][:, None] * q[(i + 1 + j * n // 4) % n] for j in range(4))
    value *= 25.0 / np.linalg.norm(value, axis=1, keepdims=True)
    last = f"dec{hp.n_dec - 1}."
    W1 = rng.standard_normal((d, F), dtype=np.float32) * np.float32(0.01)
    W2 = rng.standard_normal((F, d), dtype=np.float32) * np.float32(0.01)
    b1 = np.zeros(F, np.float32)
    W1[:, :n], b1[:n], W2[:n] = 4.0 * q.T, -0.4 * math.sqrt(d), value
    t = {"E": E, last + "W1": W1, last + "b1": b1, last + "W2": W2}
    if gpt:
        t["lnf_g"] = np.full(d, 50.0 / d, np.float32)
    else:
        eye = np.eye(d, dtype=np.float32)
        kv = rng.standard_normal((d, 2 * d), dtype=np.float32) * np.float32(0.01)
        kv[:, d:] = eye
        t.update({last + "Wkv_c": kv, last + "Wo_c": eye})
    return t


@functools.lru_cache(maxsize=8)
def _blob(hp):
    plain = dataclasses.replace(hp, cap_extra=0, sample_topk=0)   # what the tensors do not depend on
    return S.make_blob(hp, std=0.01, overrides=_tensors(plain))


# ---- the service: one model at a time, kept open over requests as a server keeps it -------------------
_open = {"key": None, "engine": None}


def _max_len(case):
    return case["len_hi"] + case["new"]


def _engine(case):
    hp = _hparams(case)
    key = (hp, case["batch"], case["beam"], _max_len(case), case["groups"], case["strength"])
    if _open["key"] != key:
        if _open["engine"] is not None:
            _open["engine"].close()
            _open.update(key=None, engine=None)
            torch.cuda.empty_cache()
        _open["engine"] = lsq.Engine(_blob(hp), case["batch"], case["beam"], _max_len(case))
        lsq.lsq_set_diversity(case["groups"], case["strength"])
        _open["key"] = key
    return _open["engine"]


def _lengths(case):
    """Source lengths: the quantiles of their distribution, so that every seed has the same work."""
    B, lo, hi = case["batch"], case["len_lo"], case["len_hi"]
    if case["len_law"] == "fixed":
        return [hi] * B
    u = [(i + 0.5) / B for i in range(B)]
    if case["len_law"] == "lognormal":       # mean 28 before the ends are cut off
        law = statistics.NormalDist(math.log(28.0) - 0.18, 0.6)
        a, b = law.cdf(math.log(lo)), law.cdf(math.log(hi))
        return [min(hi, max(lo, round(math.exp(law.inv_cdf(a + x * (b - a)))))) for x in u]
    return [min(hi, lo + int(x * (hi - lo + 1))) for x in u]


def prepare(case, seed):
    """The open service and one request: ids and lengths in host memory, where a tokenizer leaves them."""
    hp = _hparams(case)
    n = min(ACTIVE, hp.d_model // 2)
    rng = np.random.Generator(np.random.PCG64(seed))
    lens = rng.permutation(np.array(_lengths(case), np.int32))
    ids = np.full((case["batch"], int(lens.max())), hp.pad_id, np.int32)
    for b, size in enumerate(lens):
        ids[b, :size] = rng.integers(FIRST + n, hp.vocab, size)
        topic = FIRST + rng.integers(n)
        if hp.arch == 1:
            ids[b, size - 1] = topic
        else:
            ids[b, rng.permutation(size)[: (size + 1) // 2]] = topic
    _engine(case)
    return dict(case=case, src_ids=ids, src_lens=lens)


def run(state):
    case = state["case"]
    ids, lens, scores = _engine(case).translate(state["src_ids"], state["src_lens"], sync_every=case["wait"])
    return dict(ids=ids, lens=lens, scores=scores)


def work(case):
    """Products and attention of the encoder (or prompt) and of every step of every unfinished hypothesis; bytes: the
    encoder's weights once, the decoder's and the embedding once a step, every key and value once written and once read
    by each hypothesis that attends to it (those of the source once a sentence)."""
    hp = _hparams(case)
    d, F, V, L, k = hp.d_model, hp.d_ffn, hp.vocab, hp.n_dec, case["beam"]
    es = 2 if hp.dtype == 1 else 4
    lens = _lengths(case)
    block = 4 * d * d + 2 * d * F
    flops = bytes_ = 0.0
    if hp.arch == 1:
        P, B = lens[0], len(lens)
        flops += 2.0 * B * (P - 1) * L * block + 2.0 * B * L * d * P * (P - 1)
        bytes_ += es * (L * block * (P > 1) + B * (P - 1) * d * (1 + 2 * L))
        for t in range(case["new"]):
            flops += B * (2.0 * (L * block + V * d) + 4.0 * L * d * (P + t))
            bytes_ += es * (L * block + V * d + 2 * L * B * d * (P + t)) + 4 * B
        return dict(bytes=bytes_, flops=flops)
    caps = [min(n + hp.cap_extra, _max_len(case)) for n in lens]
    R = sum(lens)
    flops += 2.0 * R * (hp.n_enc * block + L * 2 * d * d) + sum(4.0 * hp.n_enc * d * n * n for n in lens)
    bytes_ += es * (hp.n_enc * block + L * 2 * d * d + R * d + 2 * L * R * d)
    for t in range(max(caps)):
        live = [n for n, c in zip(lens, caps) if c > t]
        M = len(live) * k
        flops += M * (2.0 * (L * (block + 2 * d * d) + V * d) + 4.0 * L * d * (t + 1)) + 4.0 * L * d * k * sum(live)
        bytes_ += es * (L * (block + 2 * d * d) + V * d + 2 * L * M * d * (t + 1) + 2 * L * d * sum(live)) + 8 * M
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    """Tokens and lengths: the same, but for a choice between two candidates closer than the rounding of their scores.
    Scores: sums of log-probabilities of some 1e-4 to 1e-2 each, differences of logits of which float16 keeps three digits."""
    return {"rel": 1e-2 if case["dtype"] == "f16" else 1e-4, "max": 5e-2 if case["dtype"] == "f16" else 1e-3, "differ": 0.01}
