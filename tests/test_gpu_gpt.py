"""Decoder-only model with top-k sampling: parity of the HIP library against the oracle (needs an MI355X)."""
import zlib

import numpy as np
import pytest

import lsq_synth as S
from oracle import lsq_oracle as O
from tests.parity import TOL_F16, TOL_F32, lockstep_gpt, logit_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2010_13887_amd as lib
    lib.load_library()
    yield lib
    lib.lsq_free()


def _small(dtype, seed):
    hp = S.HParams(arch=1, n_enc=0, n_dec=3, d_model=128, n_heads=2, d_ffn=264, vocab=1003, max_pos=64, act=1, norm=1,
                   dtype=dtype, sample_topk=5, cap_extra=9, seed=seed)
    return S.custom(hp, [6] * 5, beam=1, max_len=6 + 9, std=0.08, seed=seed)


@pytest.mark.parametrize("dtype", [0, 1])
def test_small_gpt_matches_oracle(lsq, dtype):
    w = _small(dtype, 11 + dtype)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, 6, 1, w.max_len) as eng:
        res = lockstep_gpt(lsq, eng, blob, w, verbose=True)
        assert res["strict"] >= (0.5 if dtype else 0.9) * res["steps"] * w.batch, res   # fp16: clear decisions only
        ids, lens, scores = eng.get_beams()
        st = res["state"]
        assert (lens[:, 0] == 9).all()
        assert np.array_equal(ids[:, 0, :9], st.tokens[:, 6:15])
        assert (ids[:, 0, 9:] == 0).all()
        np.testing.assert_allclose(scores[:, 0], st.logp, rtol=2e-5, atol=5e-2 if dtype else 1e-3)
        assert eng.decode_step() == 0                       # nothing left to generate


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("k,topp", [(32, 0.75), (16, 1.0), (32, 0.2), (3, 0.9)])
def test_topk_topp_sampling_matches_oracle(lsq, dtype, k, topp):
    """Wide candidate sets and a nucleus cut inside them (the paper's sampling runs use top-k 32, top-p 0.75)."""
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=128, n_heads=2, d_ffn=264, vocab=1003, max_pos=64, act=1, norm=1,
                   dtype=dtype, sample_topk=k, sample_topp=topp, cap_extra=8, seed=40 + k)
    w = S.custom(hp, [5] * 6, beam=1, max_len=5 + 8, std=0.3 if dtype == 0 else 0.08, seed=3)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, 6, 1, w.max_len) as eng:
        res = lockstep_gpt(lsq, eng, blob, w)
        # float16 with 32 candidates: the 32nd and 33rd logits are rarely further apart than the fp16 band, so most
        # draws are checked on the library's own logits (exactly) rather than against the oracle's
        assert res["strict"] >= (0.1 if dtype else 0.8) * res["steps"] * w.batch, res
        ids, lens, scores = eng.get_beams()
        st = res["state"]
        assert np.array_equal(ids[:, 0, :8], st.tokens[:, 5:13])
        np.testing.assert_allclose(scores[:, 0], st.logp, rtol=2e-5, atol=5e-2 if dtype else 1e-3)


@pytest.mark.parametrize("d,heads,batch,prompt,rows_per_workgroup", [
    (256, 4, 7, 5, 1),      # one row per workgroup
    (512, 8, 40, 3, 2),     # 40 * 8 workgroups would exceed the CUs: rows in pairs
    (512, 8, 33, 9, 1),     # ... an odd row count cannot pair
    (256, 4, 64, 4, 1),     # the most rows
])
def test_attention_blocks_match_oracle(lsq, d, heads, batch, prompt, rows_per_workgroup):
    """Float16 models with heads of 64 and at most 64 rows run each block's attention sublayer as one launch
    (LayerNorm, QKV, cache append, attention, per-head output projection) with the pre-LN arithmetic; lock-step
    with the oracle, then the same translation with the separate kernels: the logits behind every draw agree to
    float16 rounding, so the scores do wherever the same tokens were drawn."""
    hp = S.HParams(arch=1, n_enc=0, n_dec=3, d_model=d, n_heads=heads, d_ffn=2 * d + 8, vocab=1003, max_pos=64, act=1, norm=1,
                   dtype=1, sample_topk=4, cap_extra=10, seed=d + batch)
    w = S.custom(hp, [prompt] * batch, beam=1, max_len=prompt + 10, std=0.05, seed=batch)
    blob = w.blob(ln_jitter=0.1)
    del rows_per_workgroup   # what the library picks for this shape; documented here, not settable
    with lsq.Engine(blob, batch, 1, w.max_len) as eng:
        res = lockstep_gpt(lsq, eng, blob, w, verbose=True)
        assert res["steps"] == 10
        ids, lens, scores = eng.get_beams()
        st = res["state"]
        assert np.array_equal(ids[:, 0, :10], st.tokens[:, prompt:prompt + 10])
        np.testing.assert_allclose(scores[:, 0], st.logp, rtol=2e-5, atol=5e-2)
        try:
            lsq.lsq_set_attention_blocks(0)
            ids0, lens0, scores0 = eng.translate(w.src_ids, w.src_lens)
        finally:
            lsq.lsq_set_attention_blocks(64)
        same = (ids0[:, 0, :10] == ids[:, 0, :10]).all(axis=1)
        assert same.mean() >= 0.5, same
        np.testing.assert_allclose(scores0[same, 0], scores[same, 0], rtol=0, atol=3e-2)


def test_prompt_of_one_token_and_errors(lsq):
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=64, n_heads=4, d_ffn=128, vocab=300, max_pos=32, act=1, norm=1,
                   sample_topk=8, cap_extra=4, seed=5)
    w = S.custom(hp, [1, 1, 1], beam=1, max_len=8)
    blob = w.blob()
    with pytest.raises(lsq.LsqError):
        lsq.Engine(blob, 3, 2, 8)                            # sampling models run at beam 1
    with pytest.raises(lsq.LsqError):
        lsq.Engine(blob, 3, 1, 64)                           # more positions than the model has
    with lsq.Engine(blob, 3, 1, 8) as eng:
        res = lockstep_gpt(lsq, eng, blob, w)
        assert res["steps"] == 4
        with pytest.raises(lsq.LsqError):
            eng.encode(np.full((2, 3), 7, np.int32), [3, 2])   # prompts of different lengths
        with pytest.raises(lsq.LsqError):
            eng.encode(np.full((2, 6), 7, np.int32), [6, 6])   # 6 + 4 tokens do not fit 8 positions


@pytest.mark.parametrize("name", ["gpt2s", "gpt2s_k32p75"])
def test_gpt2_small_shape(lsq, name):
    """The GPT-2-small-shaped workload (batch 32, prompt 64, top-8 sampling; or top-32 with a 0.75 nucleus):
    40 steps in lock-step with the oracle, then the remaining steps without per-step waits; a second run is
    bit-identical."""
    w = S.workload(name)
    blob = w.blob()
    with lsq.Engine(blob, w.batch, 1, w.max_len) as eng:
        res = lockstep_gpt(lsq, eng, blob, w, n_steps=40, verbose=True)
        # random weights give nearly flat logits: most draws sit within the fp16 band of a rank swap or an
        # edge and are checked on the library's own logits instead (exactly, inside lockstep_gpt)
        if name == "gpt2s":      # with 32 candidates of a random model no draw is clear of the fp16 band: own-logit checks only
            assert res["strict"] >= 0.25 * 40 * w.batch, res
        while eng.decode_steps(32) > 0:
            pass
        assert lsq.lsq_step_index() == 128
        ids, lens, scores = eng.get_beams()
        assert (lens == 128).all() and ((ids[:, 0, :128] >= 0) & (ids[:, 0, :128] < w.hp.vocab)).all()
        assert np.isfinite(scores).all() and (scores < 0).all()
        ids2, lens2, scores2 = eng.translate(w.src_ids, w.src_lens, sync_every=9)
        assert np.array_equal(ids, ids2) and np.array_equal(scores, scores2)


@pytest.mark.parametrize("d,batch", [(256, 9), (512, 1), (512, 17), (512, 129), (768, 40), (768, 63), (1024, 6), (1024, 128)])
def test_decoder_stack_matches_oracle(lsq, d, batch):
    """All blocks of a step as one launch (float16, heads of 64, d_ffn = 4 d), at the edges of its row counts: the
    first steps in lock-step with the oracle; a second generation gives the same bits."""
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=203, max_pos=32, act=1, norm=1, dtype=1,
                   sample_topk=4, cap_extra=8, seed=d + batch)
    w = S.custom(hp, [3] * batch, beam=1, max_len=11, std=0.03, seed=batch)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, 1, w.max_len) as eng:
        lockstep_gpt(lsq, eng, blob, w, n_steps=3)
        one, two = (eng.translate(w.src_ids, w.src_lens, sync_every=n) for n in (1, 4))
        assert all(np.array_equal(a, b) for a, b in zip(one, two))
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("d,batch,fusion", [(256, 2, True), (512, 12, True), (128, 3, True), (128, 3, False)])
def test_row_without_candidates_reads_a_row_of_the_embedding(lsq, d, batch, fusion):
    """Logits that are all NaN leave a sampled row without candidates: it appends -1, and its next decoder input comes from
    embedding row 0, not from the memory before the table (the stack kernels, embedding with and without LayerNorm).
    The workspace starts inside a larger allocation, so that what lies before the table is known."""
    import torch
    P = 5
    hp = S.HParams(arch=1, n_enc=0, n_dec=1, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=301, max_pos=16, act=1, norm=1,
                   dtype=1, sample_topk=4, cap_extra=4)
    w = S.custom(hp, [P] * batch, beam=1, max_len=P + 4, std=0.05)
    rng = np.random.default_rng(d)
    t = {n: rng.standard_normal(s).astype(np.float16) * np.float16(0.25) for n, s in S.tensor_list(hp)
         if n in ("E", "P", "dec0.Wqkv", "dec0.bqkv", "dec0.ln1_g", "dec0.ln1_b")}
    blob = S.make_blob(hp, std=0.05, overrides={**t, "lnf_g": np.full(d, np.nan)})
    n = lsq.lsq_workspace_bytes(blob, batch, 1, w.max_len)
    before = 4096
    memory = torch.full((before // 2 + (n + 1) // 2,), 3.0, dtype=torch.float16, device="cuda:0")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    lsq.lsq_set_workspace(memory.data_ptr() + before, n, stream.cuda_stream)
    try:
        lsq.lsq_init(blob, batch, 1, w.max_len)
        lsq.lsq_set_layernorm_fusion(fusion)
        lsq.lsq_encode(w.src_ids, w.src_lens)
        assert lsq.lsq_decode_steps(2) == batch
        tokens = lsq.lsq_debug_read(lsq.DBG.TOKENS, (batch, w.max_len + 1), np.int32)
        assert (tokens[:, P:P + 2] == -1).all()
        K = lsq.lsq_debug_read(lsq.DBG.CACHE_K, (batch, w.max_len, d))[:, P]
    finally:
        lsq.lsq_free()
        lsq.lsq_set_layernorm_fusion(True)
    f = {k: v.astype(np.float64) for k, v in t.items()}
    x = f["E"][0] + f["P"][P]
    y = (x - x.mean()) / np.sqrt(x.var() + 1e-5) * f["dec0.ln1_g"] + f["dec0.ln1_b"]
    want = (y @ f["dec0.Wqkv"] + f["dec0.bqkv"])[d:2 * d]
    # float16 input rows and results: 3 roundings of 2^-11 in the row, averaged over d products, one in the result
    np.testing.assert_allclose(K, np.broadcast_to(want, K.shape), rtol=0, atol=2e-3 * np.abs(want).max())


@pytest.mark.parametrize("d,batch,prompt,kernel", [
    (768, 2, 270, "groups_of_8"),           # 256 keys a trip
    (768, 2, 61, "groups_of_8"),            # ... of which 64 take one key of each lane group, 128 two
    (768, 12, 125, "groups_of_8"),
    (768, 32, 132, "groups_of_8"),          # four groups of rows: 128 keys a trip
    (512, 12, 236, "die"),                  # groups of 8 rows on dies: 64 keys a trip
    (768, 41, 72, "groups_of_16_or_32"),    # of 16: 64 keys a trip
    (768, 90, 40, "groups_of_16_or_32"),    # of 32: 32 keys a trip
])
def test_decoder_stack_past_its_first_trip_for_keys(lsq, d, batch, prompt, kernel):
    """All blocks of a step in one launch, behind prompts so long that the history takes several trips."""
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=203, max_pos=300, act=1, norm=1,
                   dtype=1, sample_topk=4, cap_extra=8)
    w = S.custom(hp, [prompt] * batch, beam=1, max_len=prompt + 8, std=0.04)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, 1, w.max_len) as eng:
        lsq.lsq_profile_enable(True)
        res = lockstep_gpt(lsq, eng, blob, w)
        launches = lsq.lsq_profile_read()["decoder_stack"][1]
        lsq.lsq_profile_enable(False)
        assert res["steps"] == 8 and launches == 8 and lsq.lsq_debug_stack_launches()[kernel] == 8


@pytest.mark.parametrize("batch,kernel,text", [(12, "groups_of_8", 0x410470bb), (32, "groups_of_8", 0x8971686e),
                                               (60, "groups_of_16_or_32", 0x861d19c9), (90, "groups_of_16_or_32", 0x59e73968)])
def test_draws_do_not_turn(lsq, batch, kernel, text):
    """Text of a model whose distributions are flat: with some thousand draws a few lie so near a boundary of the cumulative weights that the
    order of the float sums of an attention decides them, and the rest of that row.  `text`: a checksum of the tokens, recorded with the
    order that Attention (stack_attend.h) states; sums of the same precision in another one gave another text for each of these batches."""
    hp = S.HParams(arch=1, n_enc=0, n_dec=4, d_model=768, n_heads=12, d_ffn=3072, vocab=1003, max_pos=200, act=1, norm=1, dtype=1,
                   sample_topk=8, cap_extra=120)
    w = S.custom(hp, [40] * batch, beam=1, max_len=160, std=0.02)
    with lsq.Engine(w.blob(ln_jitter=0.1), batch, 1, w.max_len) as eng:
        prompts = np.random.default_rng(0).integers(4, hp.vocab, (batch, 40)).astype(np.int32)
        ids, _, _ = eng.translate(prompts, w.src_lens, sync_every=32)
        assert lsq.lsq_debug_stack_launches()[kernel] == 120
    assert zlib.crc32(ids.tobytes()) == text


@pytest.mark.parametrize("heads,dh,P", [(4, 64, 2), (4, 64, 34), (2, 128, 131), (8, 32, 66), (8, 16, 40)])
@pytest.mark.parametrize("dtype", [1, 0])
def test_prefill_leaves_keys_and_values_in_the_cache(lsq, heads, dh, P, dtype):
    """Every position of every prompt but its last, of both layers; blocks of 32 rows that lie across prompts, and the launches that
    copy the rows where the attention kernel does not (float32, heads of 16)."""
    d, B = heads * dh, 5
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=d, n_heads=heads, d_ffn=2 * d, vocab=101, dtype=dtype, max_pos=160, act=1, norm=1,
                   cap_extra=3, sample_topk=2)
    w = S.custom(hp, [P] * B, beam=1, max_len=P + 4, std=0.1)
    blob = w.blob(ln_jitter=0.1)
    model = O.Model(blob, ctype=np.float64, storage="wide")
    st = O.GptState(model, w.src_ids[:, :P], P + 4)
    O.gpt_prefill(model, st)
    with lsq.Engine(blob, B + 1, 1, P + 4) as eng:
        eng.encode(w.src_ids, w.src_lens)
        for l in range(2):
            for kind, want in ((lsq.DBG.CACHE_K, st.Kc[l]), (lsq.DBG.CACHE_V, st.Vc[l])):
                got = eng.debug(kind + l, (B, P + 4, d))[:, :P - 1]
                assert logit_error(got.reshape(-1, d), want[:, :P - 1].reshape(-1, d)) <= (TOL_F16 if dtype else TOL_F32)
