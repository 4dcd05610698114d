"""Decoder layers with each group of rows on a die of its own (float16, d = 512): edges of the group sizes, of the wavefronts that
share a pair's keys, and of the lengths at which rows are dealt out differently."""
import numpy as np
import pytest
import torch

import lsq_synth as S
from tests.parity import lockstep, lockstep_gpt
from tests.test_gpu_e2e import _long_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsq():
    import paper_2010_13887_amd as m
    return m


def _ran(lsq):
    return {k: n for k, n in lsq.lsq_debug_stack_launches().items() if n}


@pytest.mark.parametrize("d,batch,beam", [
    (512, 1, 1), (512, 13, 1), (512, 5, 5), (512, 33, 1), (512, 13, 5), (512, 16, 8),   # groups of 4, 8, 4, 8, 16 and 16 rows, ragged but the last
])
def test_groups_of_rows_match_oracle(lsq, d, batch, beam):
    hp = S.HParams(n_enc=1, n_dec=2, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=203, max_pos=32, dtype=1, cap_extra=3)
    w = S.custom(hp, [1 + (5 * i) % 7 for i in range(batch)], beam=beam, max_len=12, std=0.03, seed=batch)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, beam, 12) as eng:
        lsq.lsq_profile_enable(True)
        lockstep(lsq, eng, blob, w, max_steps=3)
        assert lsq.lsq_profile_read()["decoder_stack"][1] == 3
        lsq.lsq_profile_enable(False)
        assert _ran(lsq) == {"die": 3}
        one, two = (eng.translate(w.src_ids, w.src_lens, sync_every=n) for n in (1, 4))
        assert all(np.array_equal(a, b) for a, b in zip(one, two))
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("d,batch,beam,steps,expected", [
    (512, 2, 2, 140, {"die": 140}),     # one group of 4 rows: 32, 64, 128 and 256 keys a trip; from position 129 on a group per sentence
    (512, 30, 4, 72, {"die": 72}),      # groups of 16 rows: 64 keys a trip
    (512, 17, 4, 375, {"die": 366, "groups_of_16_or_32": 9}),   # beams of more than 64 rows up to position 400, less half of the source
])
def test_long_histories_match_oracle(lsq, d, batch, beam, steps, expected):
    w, blob = _long_workload(d, d // 64, [3 + (5 * i) % 7 for i in range(batch - 1)] + [70], beam, steps, 1)
    with lsq.Engine(blob, batch, beam, w.max_len) as eng:
        assert lockstep(lsq, eng, blob, w, max_steps=steps, sentences=[batch - 1])["steps"] == steps
        assert _ran(lsq) == expected


@pytest.mark.parametrize("batch,prompt,expected", [
    (12, 296, {"die": 6, "groups_of_8": 2}),            # up to 32 rows: up to position 300, then 128 workgroups a group
    (40, 156, {"die": 6, "groups_of_16_or_32": 2}),     # up to 64 rows: 160
    (40, 236, {"groups_of_16_or_32": 5, "groups_of_8": 3}),   # ... and from 240 on groups of 8 rows, of 64 workgroups
    (100, 52, {"die": 6, "groups_of_16_or_32": 2}),     # more: 56
])
def test_prompts_across_the_change_of_kernel_match_oracle(lsq, batch, prompt, expected):
    """Decoder-only model: past some position the groups all over the chip take over."""
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=512, n_heads=8, d_ffn=2048, vocab=203, max_pos=320, act=1, norm=1, dtype=1,
                   sample_topk=4, cap_extra=8)
    w = S.custom(hp, [prompt] * batch, beam=1, max_len=prompt + 8, std=0.04)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, 1, w.max_len) as eng:
        lsq.lsq_profile_enable(True)
        res = lockstep_gpt(lsq, eng, blob, w)
        launches = lsq.lsq_profile_read()["decoder_stack"][1]
        lsq.lsq_profile_enable(False)
        assert res["steps"] == 8 and launches == 8 and _ran(lsq) == expected


@pytest.mark.parametrize("batch,beam,steps,expected", [
    (1, 1, 12, {"groups_of_8": 12}), (2, 4, 12, {"groups_of_8": 12}), (16, 1, 12, {"groups_of_16_or_32": 12}),
    (10, 4, 140, {"groups_of_16_or_32": 95, "groups_of_8": 45}),   # groups of 8 rows from position 112 on, of which a source of 70 tokens counts as 17
])
def test_models_without_dies_match_oracle(lsq, batch, beam, steps, expected):
    """Where the workgroups are not found on the dies where the die kernel wants them, d = 512 runs the kernels that are spread over
    the chip: few rows and long histories in groups of 8 rows, as other widths do."""
    w, blob = _long_workload(512, 8, [3 + (5 * i) % 7 for i in range(batch - 1)] + [70], beam, steps, 1)
    with lsq.Engine(blob, batch, beam, w.max_len) as eng:
        lsq.lsq_debug_forget_dies()
        assert lockstep(lsq, eng, blob, w, max_steps=steps, sentences=[batch - 1])["steps"] == steps
        assert _ran(lsq) == expected


def test_other_streams_do_not_move_a_model_off_its_dies(lsq):
    """Which die the first workgroup of a launch is on changes for a stream when the process opens others: the groups go by the die they
    find themselves on, whatever the model's workgroups were on when it was loaded."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=512, n_heads=8, d_ffn=2048, vocab=203, max_pos=32, dtype=1, cap_extra=6)
    w = S.custom(hp, [5, 7, 3, 6, 4], beam=4, max_len=14, std=0.03)
    with lsq.Engine(w.blob(ln_jitter=0.1), 5, 4, 14) as eng:
        want = eng.translate(w.src_ids, w.src_lens)
        torch.zeros(1 << 16, device="cuda").sum().item()
        streams = []
        for _ in range(4):
            streams.append(torch.cuda.Stream())
            with torch.cuda.stream(streams[-1]):
                torch.ones(1000, device="cuda").mul_(2)
            streams[-1].synchronize()
            assert all(np.array_equal(a, b) for a, b in zip(eng.translate(w.src_ids, w.src_lens), want))
        assert set(_ran(lsq)) == {"die"}


@pytest.mark.parametrize("stop", ["at once", "under way", "in the last step"])
def test_a_wait_that_ran_out_on_a_die_takes_the_dies_only(lsq, stop):
    """The first wait that runs out in a model of d = 512 leaves it the kernels that are spread over the chip, the second one the separate
    kernels; each time the translation comes out as those kernels make it, whichever call notices."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=512, n_heads=8, d_ffn=2048, vocab=203, max_pos=96, dtype=1, cap_extra=12)
    w = S.custom(hp, [8, 8, 8], beam=4, max_len=20, std=0.03)
    blob = w.blob(ln_jitter=0.1)
    want = {}
    for kernels in ("dies", "chip", "separate"):
        with lsq.Engine(blob, 3, 4, 20) as eng:
            if kernels == "chip":
                lsq.lsq_debug_forget_dies()
            elif kernels == "separate":
                lsq.lsq_set_attention_blocks(0)
            want[kernels] = eng.translate(w.src_ids, w.src_lens, sync_every=64)
            assert set(_ran(lsq)) == {"dies": {"die"}, "chip": {"groups_of_16_or_32"}, "separate": set()}[kernels]
            lsq.lsq_set_attention_blocks(64)

    def stopped(eng):
        eng.encode(w.src_ids, w.src_lens)
        if stop != "at once":
            eng.decode_steps(2 if stop == "under way" else int(want["dies"][1].max()) - 1)
        lsq.lsq_debug_end_stack_waits()
        if stop == "in the last step":
            assert eng.decode_steps(1) >= 0
            assert np.isfinite(eng.debug(lsq.DBG.HIDDEN, (12, 512))).all()
        lsq.lsq_decode_all(1)   # a step is queued before the count of the one before is known
        return eng.get_beams()

    with lsq.Engine(blob, 3, 4, 20) as eng:
        assert all(np.array_equal(a, b) for a, b in zip(eng.translate(w.src_ids, w.src_lens), want["dies"]))
        for kernels, kind in (("chip", "groups_of_16_or_32"), ("separate", None)):
            got = stopped(eng)
            before = lsq.lsq_debug_stack_launches()
            again = eng.translate(w.src_ids, w.src_lens, sync_every=64)
            after = lsq.lsq_debug_stack_launches()
            assert {k for k in after if after[k] > before[k]} == ({kind} if kind else set())
            assert all(np.array_equal(a, b) for a, b in zip(again, got))
            if kernels == "chip":
                assert all(np.array_equal(a, b) for a, b in zip(got, want["chip"]))
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("batch,beam,vocab,taken", [
    (1, 1, 1003, True),       # a block that ends inside its 32 columns and outside a group of 4
    (1, 4, 7200, True),       # 225 blocks for 224 workgroups: the first one has two
    (2, 4, 49149, True),      # two groups leave 192 workgroups of eight blocks, 49152 columns
    (2, 4, 49153, False),
    (24, 1, 40960, True),     # most rows at this history; three groups: 40960 columns
    (25, 1, 1003, False),     # seven groups: one die to spare, which would be behind
])
def test_dies_to_spare_take_the_vocabulary_product(lsq, batch, beam, vocab, taken):
    """Its logits against the oracle's, and the same bits as the separate product: row by row the same translation."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=512, n_heads=8, d_ffn=2048, vocab=vocab, max_pos=32, dtype=1, cap_extra=3)
    w = S.custom(hp, [1 + (5 * i) % 7 for i in range(batch)], beam=beam, max_len=12, std=0.03, seed=batch)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, beam, 12) as eng:
        lsq.lsq_profile_enable(True)
        lockstep(lsq, eng, blob, w, max_steps=3, sentences=[batch - 1])
        launches = lsq.lsq_profile_read()
        lsq.lsq_profile_enable(False)
        assert launches["decoder_stack"][1] == 3 and launches["gemm_vocab"][1] == (0 if taken else 3)
        logits = eng.debug(lsq.DBG.LOGITS, (batch * beam, vocab))
        hidden = torch.from_numpy(eng.debug(lsq.DBG.HIDDEN, (batch * beam, 512))).half().cuda()
        E = torch.from_numpy(np.frombuffer(blob, np.float16, vocab * 512, 256).reshape(vocab, 512).copy()).cuda()
        separate = torch.empty(batch * beam, vocab, dtype=torch.float32, device="cuda")
        packed = lsq.k_pack_weights(E)
        lsq.k_gemm(hidden, packed, None, separate, packed=True)
        torch.cuda.synchronize()
        assert np.array_equal(separate.cpu().numpy(), logits)
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("batch,beam", [(4, 8), (4, 7)])
def test_dies_to_spare_take_the_vocabulary_product_of_32_rows(lsq, batch, beam):
    """Past position 128 a sentence of 7 or 8 hypotheses is a group: four groups, and as many rows as the dies to spare have room for."""
    hp = S.HParams(n_enc=1, n_dec=3, d_model=512, n_heads=8, d_ffn=2048, vocab=1003, max_pos=160, dtype=1, cap_extra=140)
    w = S.custom(hp, [3] * batch, beam=beam, max_len=143, std=0.03)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, beam, 143) as eng:
        eng.encode(w.src_ids, w.src_lens)
        E = torch.from_numpy(np.frombuffer(blob, np.float16, 1003 * 512, 256).reshape(1003, 512).copy()).cuda()
        packed = lsq.k_pack_weights(E)
        for first, n, taken in ((0, 129, False), (129, 2, True), (131, 1, True)):
            lsq.lsq_profile_enable(True)
            assert eng.decode_steps(n) == batch
            launches = lsq.lsq_profile_read()
            lsq.lsq_profile_enable(False)
            assert launches["decoder_stack"][1] == n and launches["gemm_vocab"][1] == (0 if taken else n)
            logits = eng.debug(lsq.DBG.LOGITS, (batch * beam, 1003))
            hidden = torch.from_numpy(eng.debug(lsq.DBG.HIDDEN, (batch * beam, 512))).half().cuda()
            separate = torch.empty(batch * beam, 1003, dtype=torch.float32, device="cuda")
            lsq.k_gemm(hidden, packed, None, separate, packed=True)
            torch.cuda.synchronize()
            assert np.isfinite(logits).all() and np.array_equal(separate.cpu().numpy(), logits)
        assert lsq.lsq_debug_stack_launches()["die"] == 132
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("vocab,batch,beam", [(37, 10, 1), (203, 1, 4), (224, 1, 4), (1000, 2, 4), (7200, 5, 3)])
def test_dies_to_spare_leave_the_statistics_of_the_separate_product(lsq, vocab, batch, beam):
    """Candidates' scores bit for bit those that the retrieve kernel makes of the separate product's logits and group statistics: few groups, where a
    last bit of one sum of exponentials is not lost among the others."""
    hp = S.HParams(n_enc=1, n_dec=3, d_model=512, n_heads=8, d_ffn=2048, vocab=vocab, max_pos=32, dtype=1, cap_extra=25, seed=34)
    w = S.custom(hp, [10] * batch, beam=beam, max_len=32, std=0.05)
    blob = w.blob(ln_jitter=0.1)
    M = batch * beam
    E = torch.from_numpy(np.frombuffer(blob, np.float16, vocab * 512, 256).reshape(vocab, 512).copy()).cuda()
    with lsq.Engine(blob, batch, beam, 32) as eng:
        eng.encode(w.src_ids, w.src_lens)
        for step in range(8):
            score = torch.from_numpy(eng.debug(lsq.DBG.SCORE, (M,))).cuda()
            finished = torch.from_numpy(eng.debug(lsq.DBG.FINISHED, (M,), np.int32)).cuda()
            assert eng.decode_step() > 0
            hidden = torch.from_numpy(eng.debug(lsq.DBG.HIDDEN, (M, 512))).half().cuda()
            logits = torch.empty(M, vocab, dtype=torch.float32, device="cuda")
            stats = torch.empty(M, (vocab + 31) // 32, 2, dtype=torch.float32, device="cuda")
            lsq.k_gemm_logits(hidden, E, logits, stats)
            want, idx = torch.empty(M, beam, device="cuda"), torch.empty(M, beam, dtype=torch.int32, device="cuda")
            lsq.k_row_topk_groups(logits, stats, score, finished, beam, hp.eos_id, want, idx)
            torch.cuda.synchronize()
            assert np.array_equal(eng.debug(lsq.DBG.LOGITS, (M, vocab)), logits.cpu().numpy()), step
            assert np.array_equal(eng.debug(lsq.DBG.CAND_IDX, (M, beam), np.int32), idx.cpu().numpy()), step
            assert np.array_equal(eng.debug(lsq.DBG.CAND_SCORE, (M, beam)), want.cpu().numpy()), step
        assert lsq.lsq_debug_stack_launches()["die"] == 8
