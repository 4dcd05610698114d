"""End-to-end parity of the HIP library against the CPU oracle (needs an MI355X)."""
import numpy as np
import pytest

import lsq_synth as S
from oracle import lsq_oracle as O
from tests.parity import lockstep, lockstep_gpt, lockstep_sample

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2010_13887_amd as lib
    lib.load_library()
    yield lib
    lib.lsq_free()


def _final_check(lsq, eng, blob, w, res):
    ids, lens, scores = eng.get_beams()
    (o_ids, o_lens, o_scores) = O.finalize(res["judge"], res["state"])
    # the oracle followed the library through every near-tie, so the final beams must agree except
    # for the order of beams whose normalised scores are closer than the deviations measured along
    # their histories (res["bound"], per hypothesis, raw scores; dividing by len^alpha >= 1 only shrinks it)
    k = w.beam
    for b in range(w.batch):
        tol = float(res["bound"][b * k:(b + 1) * k].max()) + 1e-5
        fin = np.isfinite(o_scores[b])
        assert np.array_equal(np.isfinite(scores[b]), fin)
        np.testing.assert_allclose(scores[b][fin], o_scores[b][fin], rtol=2e-5, atol=tol)
        if (np.abs(np.diff(o_scores[b][fin])) > 2 * tol + 1e-4).all():
            assert np.array_equal(lens[b], o_lens[b])
            assert np.array_equal(ids[b], o_ids[b])


def test_tiny_fp32_matches_oracle(lsq):
    w = S.workload("tiny")
    blob = w.blob()
    with lsq.Engine(blob, w.batch, w.beam, w.max_len) as eng:
        res = lockstep(lsq, eng, blob, w, verbose=True)
        # near-flat distributions: a sentence stops being compared once a margin drops below 1e-3
        assert res["strict"] >= 4
        assert res["steps"] == 8
        _final_check(lsq, eng, blob, w, res)


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_small_vocab_eos_and_caps_fp32(lsq, seed):
    # vocabulary 12: EOS is drawn often, hypotheses finish at different steps, some hit their cap
    hp = S.HParams(n_enc=1, n_dec=2, d_model=32, n_heads=2, d_ffn=64, vocab=12, max_pos=32, cap_extra=3,
                   seed=100 + seed)
    w = S.custom(hp, [1, 4, 7, 2, 9], beam=3, max_len=11, std=0.6, seed=seed)
    blob = w.blob(ln_jitter=0.2)
    with lsq.Engine(blob, 6, w.beam, w.max_len) as eng:     # max_batch above the batch in use
        res = lockstep(lsq, eng, blob, w)
        assert res["strict"] > 0
        _final_check(lsq, eng, blob, w, res)


def test_small_fp16_ragged(lsq):
    hp = S.HParams(n_enc=2, n_dec=2, d_model=128, n_heads=2, d_ffn=264, vocab=1003, max_pos=64, dtype=1,
                   cap_extra=4)
    w = S.custom(hp, [3, 17, 9, 1, 12, 6, 11], beam=4, max_len=20, std=0.05)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, 7, w.beam, w.max_len) as eng:
        res = lockstep(lsq, eng, blob, w, verbose=True)
        assert res["strict"] >= 20, res
        _final_check(lsq, eng, blob, w, res)


@pytest.mark.parametrize("alpha,dtype", [(0.6, 0), (1.7, 1), (0.0, 0)])
def test_length_penalty_other_than_one(lsq, alpha, dtype):
    """score / len^alpha with alpha != 1 (the power branch of the final ranking): lock-step to the end, then
    the returned order, lengths and normalised scores against the oracle's, which a hand-worked case pins."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=64, n_heads=4, d_ffn=96, vocab=24, max_pos=32, dtype=dtype, cap_extra=5,
                   length_penalty=alpha, seed=77)
    w = S.custom(hp, [2, 7, 4, 1, 9, 3], beam=4, max_len=14, std=0.5 if not dtype else 0.15)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, w.batch, w.beam, w.max_len) as eng:
        res = lockstep(lsq, eng, blob, w)
        assert res["judge"].alpha == np.float32(alpha)
        _final_check(lsq, eng, blob, w, res)
        ids, lens, scores = eng.get_beams()
        st = res["state"]
        assert len(set(st.len.tolist())) > 1                  # hypotheses of different lengths: alpha matters
        # the normalisation really is the power: raw scores read back, divided here
        raw = eng.debug(lsq.DBG.SCORE, (w.batch * w.beam,)).reshape(w.batch, w.beam).astype(np.float64)
        ln = eng.debug(lsq.DBG.LEN, (w.batch * w.beam,), np.int32).reshape(w.batch, w.beam)
        want = np.sort(raw / np.maximum(ln, 1).astype(np.float64) ** float(np.float32(alpha)), axis=1)[:, ::-1]
        np.testing.assert_allclose(scores, want, rtol=3e-6, atol=1e-6)


def test_reencode_reuses_everything(lsq):
    w = S.workload("tiny")
    blob = w.blob()
    with lsq.Engine(blob, 4, w.beam, w.max_len) as eng:
        a = eng.translate(w.src_ids, w.src_lens)
        w2 = S.workload("tiny", batch=4, seed=77)
        eng.translate(w2.src_ids, w2.src_lens, sync_every=3)
        c = eng.translate(w.src_ids, w.src_lens, sync_every=100)
        for x, y in zip(a, c):
            assert np.array_equal(x, y)          # run-to-run bit identical, whatever ran in between


def test_errors_leave_no_device_work(lsq):
    w = S.workload("tiny")
    blob = w.blob()
    with pytest.raises(lsq.LsqError):
        lsq.lsq_decode_step()
    with lsq.Engine(blob, 2, w.beam, w.max_len) as eng:
        with pytest.raises(lsq.LsqError):
            lsq.lsq_decode_step()                      # before encode
        bad = w.src_ids.copy(); bad[0, 0] = 5000
        with pytest.raises(lsq.LsqError):
            eng.encode(bad, w.src_lens)
        with pytest.raises(lsq.LsqError):
            eng.encode(w.src_ids, [0, 8])
        with pytest.raises(lsq.LsqError):
            eng.encode(np.zeros((3, 8), np.int32) + 5, [1, 1, 1])   # batch above max_batch
        eng.translate(w.src_ids, w.src_lens)


def test_graph_replay_matches_eager_launches(lsq):
    """Decode steps replayed from captured hipGraphs (several replays per graph, with eager work and
    synchronisations in between) give bit-identical beams to the same kernels launched one by one."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=128, n_heads=2, d_ffn=256, vocab=504, max_pos=64, dtype=1, cap_extra=6)
    w = S.custom(hp, [3, 17, 9, 1, 12, 6, 11, 2], beam=4, max_len=24, std=0.05)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, 8, w.beam, w.max_len) as eng:
        lsq.lsq_set_graphs(False)
        eager = eng.translate(w.src_ids, w.src_lens)
        lsq.lsq_set_graphs(True)
        eng.encode(w.src_ids, w.src_lens)
        steps = 0
        while eng.decode_step() > 0:                      # one replay per call, a read-back between replays
            eng.debug(lsq.DBG.SCORE, (w.batch * w.beam,))
            steps += 1
        graphed = eng.get_beams()
        again = eng.translate(w.src_ids, w.src_lens, sync_every=5)   # graphs already captured: pure replays
        assert steps >= 10
        for a, b, c in zip(eager, graphed, again):
            assert np.array_equal(a, b) and np.array_equal(a, c)


def test_cache_refresh_modes_agree_and_cache_matches_oracle(lsq):
    """Moving cache rows by parent and reading through the slab table are the same computation:
    bit-identical beams, and after some steps the cache handed back (row r = history of hypothesis r)
    holds the oracle's keys and values in both modes."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=128, n_heads=2, d_ffn=256, vocab=504, max_pos=64, dtype=0, cap_extra=8)
    w = S.custom(hp, [3, 17, 9, 1, 12, 6], beam=4, max_len=26, std=0.3)
    blob = w.blob(ln_jitter=0.1)
    m = O.Model(blob)
    B, k, T, d = w.batch, w.beam, w.max_len, hp.d_model
    results = []
    try:
        for mode in (lsq.REFRESH_MOVE, lsq.REFRESH_TABLE):
            lsq.lsq_set_cache_refresh(mode)
            with lsq.Engine(blob, B, k, T) as eng:
                res = lockstep(lsq, eng, blob, w, max_steps=7)
                st = res["state"]                            # oracle state after 7 steps, resynced to the library
                moved = (eng.debug(lsq.DBG.PARENT, (B * k,), np.int32).reshape(B, k) != np.arange(k)).any()
                for l in range(hp.n_dec):
                    for item, ref in ((lsq.DBG.CACHE_K, st.Kc[l]), (lsq.DBG.CACHE_V, st.Vc[l])):
                        got = eng.debug(item + l, (B * k, T, d))
                        alive = np.repeat(st.cap > 7, k) & ~st.finished.reshape(-1)   # rows both sides still extend
                        np.testing.assert_allclose(got[alive, :7], np.asarray(ref)[alive, :7], rtol=1e-4, atol=1e-4)
                results.append(eng.translate(w.src_ids, w.src_lens, sync_every=3) + (moved,))
    finally:
        lsq.lsq_set_cache_refresh(lsq.REFRESH_TABLE)
    assert results[0][3] or results[1][3]                    # beams really changed parents
    for a, b in zip(results[0][:3], results[1][:3]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n_dec", [1, 2])
def test_layernorm_fusion_agrees_with_standalone_kernel(lsq, n_dec):
    """LayerNorm inside the consuming kernel (default) against the stand-alone LayerNorm kernel: the same
    tokens, scores equal to the last bits (the row arithmetic is the same; the cross-attention kernel that
    normalises its own rows sums over fewer split-K slabs and shares the keys among four wavefronts).
    Lock-step with the oracle runs on the fused path."""
    hp = S.HParams(n_enc=1, n_dec=n_dec, d_model=128, n_heads=2, d_ffn=256, vocab=504, max_pos=64, dtype=1, cap_extra=9)
    w = S.custom(hp, [3, 17], beam=4, max_len=29, std=0.05)           # 8 rows from the first step on
    w3 = S.custom(hp, [3, 17, 1, 9, 20], beam=4, max_len=29, std=0.05)  # 20 rows, then 8 and 4 near the end
    blob = w.blob(ln_jitter=0.1)
    out, many = {}, {}
    try:
        for on in (False, True):
            lsq.lsq_set_layernorm_fusion(on)
            with lsq.Engine(blob, 5, 4, 29) as eng:
                out[on] = eng.translate(w.src_ids, w.src_lens, sync_every=2)
                many[on] = eng.translate(w3.src_ids, w3.src_lens, sync_every=3)
                if on:
                    res = lockstep(lsq, eng, blob, w)
                    assert res["steps"] >= 10
                    _final_check(lsq, eng, blob, w, res)
                    hidden = eng.debug(lsq.DBG.HIDDEN, (w.batch * w.beam, hp.d_model))
                    assert np.isfinite(hidden).all() and np.abs(hidden).max() > 0.1
    finally:
        lsq.lsq_set_layernorm_fusion(True)
    # the products that normalise their own input give the bits of the stand-alone LayerNorm kernel; the
    # cross-attention kernel that makes its own queries shares a sentence's keys among four wavefronts where
    # the stand-alone one may use a single wavefront, so its softmax sums are taken in another order: the same
    # tokens, scores equal to float16 rounding
    for (ids0, lens0, sc0), (ids1, lens1, sc1) in ((out[False], out[True]), (many[False], many[True])):
        assert np.array_equal(ids0, ids1) and np.array_equal(lens0, lens1)
        # (a query that differs in its last float32 bit can round to the neighbouring float16 value, which the
        # following layers carry along: differences of a few 1e-5 in a score of about 2)
        np.testing.assert_allclose(sc0, sc1, rtol=0, atol=2e-4)


@pytest.mark.parametrize("vocab,beam", [(504, 4), (8200, 3), (37, 8)])
def test_retrieve_from_group_statistics_agrees_with_full_rows(lsq, vocab, beam):
    """Retrieve stage from the logit product's group statistics (default) against the kernel that reads every
    row: the same tokens and lengths, scores equal to the rounding of the normaliser; a batch that shrinks from
    more than 64 rows (large-tile product) to a few (skinny product) on its way; retrieve and re-rank as one launch
    (default) and as two."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=128, n_heads=2, d_ffn=256, vocab=vocab, max_pos=64, dtype=1, cap_extra=9)
    lens = [2 + (7 * i) % 19 for i in range(23)]
    w = S.custom(hp, lens, beam=beam, max_len=29, std=0.05)
    blob = w.blob(ln_jitter=0.1)
    out = {}
    try:
        for mode in (0, 2, 1):
            lsq.lsq_set_topk_statistics(mode)
            with lsq.Engine(blob, 23, beam, 29) as eng:
                out[mode] = eng.translate(w.src_ids, w.src_lens, sync_every=3)
                if mode:
                    res = lockstep(lsq, eng, blob, w)
                    _final_check(lsq, eng, blob, w, res)
    finally:
        lsq.lsq_set_topk_statistics(1)
    for a, b in zip(out[1], out[2]):
        assert np.array_equal(a, b)                      # one launch or two: the same bits
    (ids0, lens0, sc0), (ids1, lens1, sc1) = out[0], out[1]
    same = (ids0 == ids1).all(axis=-1)
    assert same.mean() >= 0.95 and np.array_equal(lens0[same], lens1[same])   # a near-tie may flip on the last bit
    np.testing.assert_allclose(sc0[same], sc1[same], rtol=0, atol=2e-5)


@pytest.mark.parametrize("beam,period", [(4, 410), (2, 410), (4, 82), (8, 82)])
def test_retrieve_in_one_launch_agrees_with_two_on_tied_logits(lsq, beam, period):
    """Embedding rows that repeat: 20 or 100 tokens of equal logits, each in a group of its own, so that more groups reach the
    threshold than one pass of the merged kernel takes, with up to and more than 64 candidates: the bits of the two launches,
    and of ties the lowest tokens."""
    V, d = 8200, 128
    hp = S.HParams(n_enc=1, n_dec=1, d_model=d, n_heads=2, d_ffn=256, vocab=V, max_pos=64, dtype=1, cap_extra=6)
    w = S.custom(hp, [3, 9, 5], beam=beam, max_len=20, std=0.05)
    blob = bytearray(w.blob(ln_jitter=0.1))
    E = np.frombuffer(blob, np.float16, V * d, offset=256).reshape(V, d)
    E[:] = E[np.arange(V) % period].copy()
    out = {}
    try:
        for mode in (2, 1):
            lsq.lsq_set_topk_statistics(mode)
            with lsq.Engine(bytes(blob), 3, beam, 20) as eng:
                out[mode] = eng.translate(w.src_ids, w.src_lens, sync_every=2)
    finally:
        lsq.lsq_set_topk_statistics(1)
    for a, b in zip(out[1], out[2]):
        assert np.array_equal(a, b)
    ids, lens, _ = out[1]
    first = np.asarray(ids)[..., 1] if np.asarray(ids).ndim == 3 else np.asarray(ids)[:, 1]
    assert (np.asarray(lens) >= 1).all() and (first < period * beam).all()   # ties at one step: the first `beam` of them


@pytest.mark.parametrize("beam,heads,refresh", [(4, 4, "table"), (3, 8, "move"), (1, 4, "table"), (2, 8, "table")])
def test_attention_blocks_agree_with_separate_kernels(lsq, beam, heads, refresh):
    """Attention sublayers as one launch each (default, at most 64 rows alive) against the separate kernels: the
    same tokens, scores equal to float16 rounding (the output projection is summed head by head, the new
    position's key and value join the softmax last).  Lock-step with the oracle runs on the block path,
    eager and through graph replays; a batch that starts above 64 rows switches to the blocks on its way."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=64 * heads, n_heads=heads, d_ffn=320, vocab=504, max_pos=64, dtype=1,
                   cap_extra=9)
    w = S.custom(hp, [3, 17, 1, 9, 20], beam=beam, max_len=29, std=0.05)
    lens_many = [2 + (7 * i) % 19 for i in range(23)]                  # 92 rows at beam 4, 23 at beam 1
    wm = S.custom(hp, lens_many, beam=beam, max_len=29, std=0.05)
    blob = w.blob(ln_jitter=0.1)
    out, many = {}, {}
    lsq.lsq_set_cache_refresh(lsq.REFRESH_TABLE if refresh == "table" else lsq.REFRESH_MOVE)
    try:
        for rows in (0, 64):
            lsq.lsq_set_attention_blocks(rows)
            with lsq.Engine(blob, 23, beam, 29) as eng:
                out[rows] = eng.translate(w.src_ids, w.src_lens, sync_every=2)
                many[rows] = eng.translate(wm.src_ids, wm.src_lens, sync_every=3)
                if rows:
                    res = lockstep(lsq, eng, blob, w)
                    assert res["steps"] >= 10
                    _final_check(lsq, eng, blob, w, res)
                    res = lockstep(lsq, eng, blob, wm)
                    _final_check(lsq, eng, blob, wm, res)
                    lsq.lsq_set_graphs(False)
                    eager = eng.translate(wm.src_ids, wm.src_lens, sync_every=1)
                    lsq.lsq_set_graphs(True)
                    for a, b in zip(eager, many[rows]):
                        assert np.array_equal(a, b)                  # replays against eager launches: bit for bit
    finally:
        lsq.lsq_set_attention_blocks(64)
        lsq.lsq_set_graphs(True)
        lsq.lsq_set_cache_refresh(lsq.REFRESH_TABLE)
    for (ids0, lens0, sc0), (ids1, lens1, sc1) in ((out[0], out[64]), (many[0], many[64])):
        same = (ids0 == ids1).all(axis=-1)
        # a hypothesis whose margin over the next candidate is below float16 rounding may differ; nearly all agree
        assert same.mean() >= 0.9 and np.array_equal(lens0[same], lens1[same])
        # (both paths round to float16 at the same storage points, from sums taken in different orders)
        np.testing.assert_allclose(sc0[same], sc1[same], rtol=0, atol=2e-3)


@pytest.mark.parametrize("beam,lens,vocab,cap_extra,max_len,dtype", [
    (1, [1], 37, 3, 6, 0),            # one sentence of one token, greedy
    (8, [4, 2, 7], 64, 2, 9, 0),      # the widest beam
    (4, [5, 3], 5, 0, 5, 0),          # vocabulary barely above the beam; cap = source length, = max_len for one
    (3, [2, 6, 6, 1], 301, 4, 7, 1),  # caps cut off by max_len, float16, beam that does not divide 64
    (2, [9], 1000, 1, 12, 1),         # single sentence, float16: the few-row kernels from the first step on
])
def test_edge_shapes_match_oracle(lsq, beam, lens, vocab, cap_extra, max_len, dtype):
    hp = S.HParams(n_enc=1, n_dec=2, d_model=64, n_heads=4, d_ffn=96, vocab=vocab, max_pos=16, dtype=dtype,
                   cap_extra=cap_extra)
    w = S.custom(hp, lens, beam=beam, max_len=max_len, std=0.08 if dtype else 0.3)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, len(lens), beam, max_len) as eng:
        res = lockstep(lsq, eng, blob, w)
        assert res["steps"] == min(max(lens) + cap_extra, max_len)
        _final_check(lsq, eng, blob, w, res)
        ids, out_lens, scores = eng.get_beams()
        assert ((out_lens >= 0) & (out_lens <= max_len)).all()
        assert ((ids >= 0) & (ids < vocab)).all()


def test_no_kernel_writes_outside_its_region(lsq):
    """Red zones behind every region of the workspace (weights, caches, beam state, each decoder intermediate, the
    end) stay untouched through whole translations -- float32 and float16 models, both cache-refresh modes, a
    decoder-only model, ragged sizes, a batch smaller than the maximum -- and a byte written into one is seen."""
    cases = []
    w = S.workload("tiny")
    cases.append((w, w.blob(), {}))
    hp = S.HParams(n_enc=2, n_dec=2, d_model=128, n_heads=2, d_ffn=264, vocab=1003, max_pos=64, dtype=1, cap_extra=4)
    w = S.custom(hp, [3, 17, 9, 1, 12, 6, 11], beam=4, max_len=20, std=0.05)
    cases.append((w, w.blob(ln_jitter=0.1), {}))
    cases.append((w, w.blob(ln_jitter=0.1), dict(refresh=lsq.REFRESH_MOVE)))
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=96, n_heads=3, d_ffn=136, vocab=301, max_pos=64, act=1, norm=1,
                   dtype=1, sample_topk=5, cap_extra=7)
    w = S.custom(hp, [6] * 5, beam=1, max_len=14, std=0.08)
    cases.append((w, w.blob(ln_jitter=0.1), {}))
    try:
        lsq.lsq_set_canaries(True)
        for w, blob, opt in cases:
            lsq.lsq_set_cache_refresh(opt.get("refresh", lsq.REFRESH_TABLE))
            with lsq.Engine(blob, w.batch + 2, w.beam, w.max_len) as eng:
                assert lsq.lsq_debug_check_canaries() == 0
                for _ in range(2):
                    eng.translate(w.src_ids, w.src_lens, sync_every=3)
                    assert lsq.lsq_debug_check_canaries() == 0
                eng.encode(w.src_ids[:1], w.src_lens[:1])
                eng.decode_steps(2)
                assert lsq.lsq_debug_check_canaries() == 0
                eng.workspace[-1] = 0                        # the last byte of the workspace lies in the last red zone
                assert lsq.lsq_debug_check_canaries() == 1
        with pytest.raises(lsq.LsqError):
            with lsq.Engine(cases[0][1], 2, 4, 8):
                lsq.lsq_set_canaries(False)                  # the plan of a loaded model is fixed
    finally:
        lsq.lsq_free()
        lsq.lsq_set_canaries(False)
        lsq.lsq_set_cache_refresh(lsq.REFRESH_TABLE)


@pytest.mark.parametrize("d,batch,beam,dtype", [
    (256, 1, 1, 1), (256, 16, 4, 1),                               # groups of 8 rows only: the smallest and the largest
    (512, 2, 4, 1), (512, 3, 3, 1), (512, 32, 8, 1), (512, 33, 8, 1),    # 8 rows, 9 (ragged groups), 256 rows, one sentence more
    (768, 5, 8, 1), (768, 41, 1, 1), (768, 40, 4, 1),                 # 40 rows, 41 (one row a group is left over), 160
    (1024, 1, 7, 1), (1024, 13, 5, 1), (1024, 32, 4, 1),              # 7 rows, 65 (past the attention blocks), 128
    (256, 1, 1, 0), (256, 64, 4, 0), (256, 65, 4, 0),         # float32: one row, 256 rows, too many for one launch
    (512, 2, 8, 0), (512, 11, 3, 0), (512, 33, 4, 0), (512, 32, 8, 0),   # 16 rows, 33 (5 a group), 132 (17), 256
])
def test_decoder_stack_matches_oracle(lsq, d, batch, beam, dtype):
    """All decoder layers as one launch (heads of 64, d_ffn = 4 d), at the edges of its row counts: the
    first steps in lock-step with the oracle; a second translation gives the same bits."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=203, max_pos=32, dtype=dtype, cap_extra=3)
    w = S.custom(hp, [1 + (5 * i) % 7 for i in range(batch)], beam=beam, max_len=12, std=0.03 if dtype else 0.1)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, beam, 12) as eng:
        lockstep(lsq, eng, blob, w, max_steps=3)
        one, two = (eng.translate(w.src_ids, w.src_lens, sync_every=n) for n in (1, 4))
        assert all(np.array_equal(a, b) for a, b in zip(one, two))
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("d,heads,ffn,vocab,beam,dtype", [
    (64, 4, 64, 31, 1, 0), (64, 2, 448, 1000, 8, 0), (128, 8, 512, 1001, 5, 0), (128, 4, 192, 97, 3, 0),
    (64, 4, 512, 33, 8, 1), (128, 8, 64, 1024, 1, 1), (128, 4, 512, 65, 4, 1),
])
def test_small_model_step_matches_oracle(lsq, d, heads, ffn, vocab, beam, dtype):
    """A whole step of a small model as one launch, at the edges of its shapes (row widths, head sizes, vocabularies that
    end inside a group of 32 or a block of 64 columns, sources and histories of more than 64 positions)."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=d, n_heads=heads, d_ffn=ffn, vocab=vocab, max_pos=96, dtype=dtype, cap_extra=6)
    w = S.custom(hp, [5, 1, 70, 64], beam=beam, max_len=75, std=0.3 if dtype == 0 else 0.08)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, 5, beam, 75) as eng:
        lockstep(lsq, eng, blob, w, max_steps=4)
        one, two = (eng.translate(w.src_ids, w.src_lens, sync_every=n) for n in (1, 5))
        assert all(np.array_equal(a, b) for a, b in zip(one, two))
        lsq.lsq_set_attention_blocks(0)
        ids, lens, scores = eng.translate(w.src_ids, w.src_lens)
        lsq.lsq_set_attention_blocks(64)
        same = (ids == one[0]).all(axis=-1)
        assert same.mean() >= (0.3 if dtype else 0.9)
        np.testing.assert_allclose(scores[same], one[2][same], rtol=0, atol=5e-2 if dtype else 1e-3)
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("d,batch,beam,dtype,kind,kernel", [
    (512, 2, 4, 1, "", "die"), (512, 12, 4, 1, "", "die"), (512, 5, 1, 1, "sampling", "die"),
    (256, 2, 4, 1, "", "groups_of_8"), (1024, 3, 4, 1, "", "groups_of_16_or_32"), (512, 3, 4, 0, "", "float32"),
    (256, 4, 1, 1, "decoder-only", "groups_of_8")])
def test_translation_survives_a_wait_that_ran_out(lsq, d, batch, beam, dtype, kind, kernel):
    """Where a wait inside a stack kernel has run out, the steps that are already queued behind it do not wait as well (64 of
    them would take half a second each), and the translation is decoded again with the kernels that need less company (on dies: those
    that are spread over the chip; otherwise the separate ones), which the model then keeps: the same tokens as before up to rounding,
    and from then on the same bits."""
    import time
    gpt = kind == "decoder-only"
    hp = S.HParams(n_enc=0 if gpt else 1, n_dec=2, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=203, max_pos=96, dtype=dtype,
                   cap_extra=64, sample_topk=3 if kind else 0, **(dict(arch=1, act=1, norm=1) if gpt else {}))
    w = S.custom(hp, [8] * batch, beam=beam, max_len=80, std=0.03 if dtype else 0.1)
    blob = w.blob(ln_jitter=0.1)
    lock = (lockstep_gpt if gpt else lockstep_sample) if kind else lockstep
    with lsq.Engine(blob, batch, beam, 80) as eng:
        want = eng.translate(w.src_ids, w.src_lens, sync_every=64)
        assert {k for k, n in lsq.lsq_debug_stack_launches().items() if n} == {kernel}
        eng.encode(w.src_ids, w.src_lens)
        assert eng.decode_steps(7) > 0
        lsq.lsq_debug_end_stack_waits()
        t0 = time.perf_counter()
        while eng.decode_steps(64) > 0:
            pass
        assert time.perf_counter() - t0 < 2.0
        got = eng.get_beams()
        before = lsq.lsq_debug_stack_launches()
        again = eng.translate(w.src_ids, w.src_lens)
        after = lsq.lsq_debug_stack_launches()
        assert (after != before) == (kernel == "die") and after[kernel] == before[kernel]
        assert all(np.array_equal(a, b) for a, b in zip(got, again))
        same = (got[0] == want[0]).all(axis=-1)
        assert same.mean() >= (0.3 if dtype else 0.9)        # 64 steps of a nearly flat distribution in float16
        np.testing.assert_allclose(got[2][same], want[2][same], rtol=0, atol=5e-2 if dtype else 1e-3)
        lock(lsq, eng, blob, w, **{"n_steps" if gpt else "max_steps": 4})
    for stop in ("at once", "in the last step"):             # every call that waits for the device notices
        with lsq.Engine(blob, batch, beam, 80) as eng:
            eng.encode(w.src_ids, w.src_lens)
            if stop == "at once":
                lsq.lsq_debug_end_stack_waits()
                lsq.lsq_decode_all(1)
            else:
                n = int(got[1].max())
                eng.decode_steps(n - 1)
                lsq.lsq_debug_end_stack_waits()
                eng.decode_steps(1)
                assert np.isfinite(eng.debug(lsq.DBG.HIDDEN, (batch * beam, d))).all()
                while eng.decode_steps(64) > 0:
                    pass
            assert all(np.array_equal(a, b) for a, b in zip(eng.get_beams(), got))


def test_masked_queues_run_the_separate_kernels(lsq, monkeypatch):
    """The stack kernels need the whole chip: where the environment masks the process's queues the separate kernels run
    (the variable is only read here, the runtime looked at it when it started)."""
    import torch
    hp = S.HParams(n_enc=1, n_dec=2, d_model=512, n_heads=8, d_ffn=2048, vocab=203, max_pos=32, dtype=1, cap_extra=6)
    w = S.custom(hp, [5, 3, 7], beam=4, max_len=14, std=0.05)
    blob = w.blob(ln_jitter=0.1)

    def translate(stream):
        n = lsq.lsq_workspace_bytes(blob, w.batch, w.beam, w.max_len)
        memory = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        torch.cuda.synchronize()
        lsq.lsq_set_workspace(memory.data_ptr(), n, stream)
        try:
            lsq.lsq_init(blob, w.batch, w.beam, w.max_len)
            lsq.lsq_profile_enable(True)
            lsq.lsq_encode(w.src_ids, w.src_lens)
            lsq.lsq_decode_all(4)
            out = lsq.lsq_get_beams(w.batch, w.beam, w.max_len)
            launches = lsq.lsq_profile_read()["decoder_stack"][1]
            lsq.lsq_profile_enable(False)
        finally:
            lsq.lsq_free()
        return out, launches

    whole = torch.cuda.Stream()
    want, launches = translate(whole.cuda_stream)
    assert launches > 0
    monkeypatch.setenv("HSA_CU_MASK", "0:0-127")
    got, launches = translate(whole.cuda_stream)
    assert launches == 0
    same = (got[0] == want[0]).all(axis=-1)
    assert same.mean() >= 0.9                          # a near-tie may flip: sums in another order, float16
    np.testing.assert_allclose(got[2][same], want[2][same], rtol=0, atol=2e-3)


def _long_workload(d, heads, lens, beam, steps, dtype, n_dec=2, ffn=None, vocab=203, std=None):
    """A model that does not end its sentences: EOS lies far behind along the shift of the last LayerNorm."""
    hp = S.HParams(n_enc=1, n_dec=n_dec, d_model=d, n_heads=heads, d_ffn=ffn or 4 * d, vocab=vocab, max_pos=512, dtype=dtype,
                   cap_extra=steps)
    w = S.custom(hp, lens, beam=beam, max_len=max(lens) + steps, std=std or (0.03 if dtype else 0.1))
    E = np.random.default_rng(d).standard_normal((vocab, d)) * w.std
    E[hp.eos_id] = -16.0 / d
    return w, w.blob(ln_jitter=0.1, overrides={"E": E, f"dec{n_dec - 1}.ln3_b": np.ones(d)})


@pytest.mark.parametrize("d,batch,beam,dtype,steps,kernel", [
    (256, 1, 2, 1, 270, "groups_of_8"),           # 256 keys a trip
    (512, 10, 4, 1, 140, "die"),                  # groups of 8 rows on dies; the other kernels at these sizes: tests/test_gpu_die.py
    (768, 12, 4, 1, 72, "groups_of_16_or_32"),    # of 16: 64 keys a trip
    (512, 40, 4, 1, 72, "groups_of_16_or_32"),    # of 32: 32 keys a trip
    (512, 2, 1, 0, 72, "float32"), (512, 16, 4, 0, 72, "float32"), (256, 33, 4, 0, 72, "float32"), (512, 40, 4, 0, 72, "float32"),   # 64, 32, 16 and 8 keys a trip
])
def test_decoder_stack_past_its_first_trip_for_keys(lsq, d, batch, beam, dtype, steps, kernel):
    """One sentence of the batch in lock-step with the oracle until the histories (and the slab table) have been read in
    several trips, beside a source of 70 tokens."""
    w, blob = _long_workload(d, d // 64, [3 + (5 * i) % 7 for i in range(batch - 1)] + [70], beam, steps, dtype)
    with lsq.Engine(blob, batch, beam, w.max_len) as eng:
        assert lockstep(lsq, eng, blob, w, max_steps=steps, sentences=[batch - 1])["steps"] == steps
        assert lsq.lsq_debug_stack_launches()[kernel] == steps


@pytest.mark.parametrize("d,batch,beam", [
    (768, 1, 1), (768, 4, 4), (768, 2, 3),      # three k-steps a wavefront, eight columns a workgroup: the last pair is half empty
    (768, 3, 7), (1024, 1, 8), (256, 2, 8),     # sixteen columns; four k-steps; one
])
def test_pairs_of_k_steps_match_oracle(lsq, d, batch, beam):
    """Groups of 8 rows: two k-steps share a 16 x 16 product."""
    w, blob = _long_workload(d, d // 64, [2 + (5 * i) % 7 for i in range(batch)], beam, 4, 1)
    with lsq.Engine(blob, batch, beam, w.max_len) as eng:
        assert lockstep(lsq, eng, blob, w, max_steps=4)["steps"] == 4
        assert lsq.lsq_debug_stack_launches()["groups_of_8"] == 4


@pytest.mark.parametrize("lens", [(64, 65), (128, 129), (7, 257)])
def test_sources_around_the_forms_of_a_trip_match_oracle(lsq, lens):
    """Eight wavefronts share a source's keys: one per lane group up to 64, two up to 128, then four, and a second trip."""
    w, blob = _long_workload(1024, 16, list(lens), 4, 3, 1)
    with lsq.Engine(blob, 2, 4, w.max_len) as eng:
        assert lockstep(lsq, eng, blob, w, max_steps=3)["steps"] == 3
        assert lsq.lsq_debug_stack_launches()["groups_of_8"] == 3


@pytest.mark.parametrize("d,batch,beam,steps", [
    (1024, 5, 4, 132),   # groups of 16 rows, two wavefronts a head: through LDS from 65 keys on and again from 129 on
    (1024, 17, 4, 68),   # groups of 32 rows, one wavefront: 32 keys a trip
    (768, 21, 5, 100),   # a fourth trip, whose places in the cache are looked up two trips ahead
])
def test_trips_of_keys_through_lds_match_oracle(lsq, d, batch, beam, steps):
    """Groups of 16 and 32 rows at every length around the ends of their trips, sources of 1, 33 and 65 tokens among them."""
    w, blob = _long_workload(d, d // 64, [1, 33] + [3 + (5 * i) % 7 for i in range(batch - 3)] + [65], beam, steps, 1)
    with lsq.Engine(blob, batch, beam, w.max_len) as eng:
        assert lockstep(lsq, eng, blob, w, max_steps=steps, sentences=[0, 1, batch - 1])["steps"] == steps
        assert lsq.lsq_debug_stack_launches()["groups_of_16_or_32"] == steps
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("d,batch,beam,steps", [(1024, 17, 4, 100), (1024, 5, 4, 132), (768, 21, 5, 132)])
def test_trips_of_keys_through_lds_without_a_slab_table(lsq, d, batch, beam, steps):
    """The third trip and those behind it in groups of 32 and 16 rows when cache rows move with the beams: every row reads its own
    history.  In lock-step with the oracle, and the same bits as with the table."""
    w, blob = _long_workload(d, d // 64, [5, 9] + [3 + (5 * i) % 7 for i in range(batch - 3)] + [65], beam, steps, 1)
    out = {}
    try:
        for mode in (lsq.REFRESH_TABLE, lsq.REFRESH_MOVE):
            lsq.lsq_set_cache_refresh(mode)
            with lsq.Engine(blob, batch, beam, w.max_len) as eng:
                out[mode] = eng.translate(w.src_ids, w.src_lens, sync_every=64)
                assert lsq.lsq_debug_stack_launches()["groups_of_16_or_32"] > steps // 2
                if mode == lsq.REFRESH_MOVE:
                    assert lockstep(lsq, eng, blob, w, max_steps=steps, sentences=[0, batch - 1])["steps"] == steps
                    assert lsq.lsq_debug_check_canaries() == 0
    finally:
        lsq.lsq_set_cache_refresh(lsq.REFRESH_TABLE)
    assert all(np.array_equal(a, b) for a, b in zip(out[lsq.REFRESH_TABLE], out[lsq.REFRESH_MOVE]))


def test_long_histories_leave_the_stack_kernel(lsq):
    """256 rows, d = 256, float32: from a history of 850 on (less half of the source) the separate launches are ahead and take
    over in the middle of a translation.  The same tokens as with the separate launches alone."""
    w, blob = _long_workload(256, 4, [8] * 64, 4, 860, 0, n_dec=1)
    out = {}
    try:
        for rows in (0, 64):
            lsq.lsq_set_attention_blocks(rows)
            with lsq.Engine(blob, 64, 4, w.max_len) as eng:
                lsq.lsq_profile_enable(True)
                out[rows] = eng.translate(w.src_ids, w.src_lens, sync_every=64)
                stack = lsq.lsq_profile_read()["decoder_stack"][1]
                lsq.lsq_profile_enable(False)
                assert stack == (850 - 4 + 1 if rows else 0)
    finally:
        lsq.lsq_set_attention_blocks(64)
    same = (out[0][0] == out[64][0]).all(axis=-1)
    assert same.mean() >= 0.9                              # float32 sums in another order: a near-tie may flip
    np.testing.assert_allclose(out[0][2][same], out[64][2][same], rtol=0, atol=1e-3)


@pytest.mark.parametrize("d,heads,beam,dtype,src", [(64, 4, 2, 1, 70), (128, 4, 1, 1, 9), (64, 2, 4, 0, 70), (128, 8, 2, 0, 130)])
def test_small_model_step_past_its_first_trip_for_keys(lsq, d, heads, beam, dtype, src):
    """The one-launch step of a small model in lock-step with the oracle until histories and slab table have been read in
    several trips of 64, with sources of one trip, two and three."""
    w, blob = _long_workload(d, heads, [2, src], beam, 80, dtype, n_dec=1, vocab=97, std=0.08 if dtype else 0.3)
    with lsq.Engine(blob, 2, beam, w.max_len) as eng:
        lsq.lsq_profile_enable(True)
        res = lockstep(lsq, eng, blob, w, max_steps=80, sentences=[1])
        launches = lsq.lsq_profile_read()
        lsq.lsq_profile_enable(False)
        assert res["steps"] == 80 and launches["decoder_stack"][1] == 80 and launches["gemm_vocab"][1] == 0


def test_long_histories_leave_the_small_model_kernel(lsq):
    """8 heads and 2 layers, 8 rows: past a history of 128 positions the separate launches take over in
    the middle of a translation; the same tokens as with the separate launches alone."""
    w, blob = _long_workload(128, 8, [9, 4], 4, 170, 0, vocab=97, std=0.3)
    out = {}
    try:
        for rows in (0, 64):
            lsq.lsq_set_attention_blocks(rows)
            with lsq.Engine(blob, 2, 4, w.max_len) as eng:
                lsq.lsq_profile_enable(True)
                out[rows] = eng.translate(w.src_ids, w.src_lens, sync_every=64)
                launches = lsq.lsq_profile_read()
                lsq.lsq_profile_enable(False)
                # 4 passes of 8 pairs, a trip of the history counts 2: 4 (2 * 2 + 1) = 20 trips are within the bound, 4 (2 * 3 + 1) are not
                assert launches["decoder_stack"][1] == (128 if rows else 0)
    finally:
        lsq.lsq_set_attention_blocks(64)
    same = (out[0][0] == out[64][0]).all(axis=-1)
    assert same.mean() >= 0.9                              # float32 sums in another order: a near-tie may flip
    np.testing.assert_allclose(out[0][2][same], out[64][2][same], rtol=0, atol=1e-3)
