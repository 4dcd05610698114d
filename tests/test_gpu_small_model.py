"""Small models: the encoder as one launch, and several steps of a translation as one launch (needs an MI355X)."""
import numpy as np
import pytest

import lsq_synth as S
from oracle import lsq_oracle as O
from tests.parity import TOL_F16, TOL_F32, logit_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2010_13887_amd as lib
    lib.load_library()
    yield lib
    lib.lsq_free()


@pytest.mark.parametrize("d,heads,ffn,dtype,lens,one", [
    (64, 4, 64, 0, [1], True), (64, 2, 448, 0, [16, 3, 17], True), (128, 8, 512, 0, [1] * 66 + [32, 33], True), (128, 4, 192, 0, [5] * 94 + [48, 47], True),
    (64, 4, 512, 1, [48, 2], True), (64, 2, 64, 1, [15, 16], True), (128, 8, 512, 1, [17] * 60 + [31, 9], True), (64, 4, 128, 1, [48, 49], False),
    (128, 4, 128, 1, [2, 1, 1], False), (128, 4, 192, 0, [5] * 93 + [48, 47], False),
])
def test_encoder_of_a_small_model(lsq, d, heads, ffn, dtype, lens, one):
    """Encoder output and cross-attention keys and values at the edges of the blocks of 16 rows, with one token, and either side of
    the lines to the separate launches (49 tokens; d = 128: fewer than twice as many sentences as tokens), against the oracle in 64 bits."""
    hp = S.HParams(n_enc=2, n_dec=3, d_model=d, n_heads=heads, d_ffn=ffn, vocab=97, max_pos=64, dtype=dtype, cap_extra=2)
    w = S.custom(hp, lens, beam=2, max_len=52, std=0.1 if dtype else 0.3)
    blob = w.blob(ln_jitter=0.1)
    R = sum(lens)

    def oracle(ctype):
        memory, cross = O.encode(O.Model(blob, ctype=ctype, storage="wide"), w.src_ids, w.src_lens)
        return [np.concatenate(memory)] + [np.concatenate([np.concatenate(c[l], axis=-1) for c in cross]) for l in range(hp.n_dec)]

    def read(eng):
        return [eng.debug(lsq.DBG.MEMORY, (R, d))] + [eng.debug(lsq.DBG.CROSS_KV + l, (R, 2 * d)) for l in range(hp.n_dec)]

    want = oracle(np.float64)
    # float32: as everywhere here, 1e-4 or four times what plain numpy float32 loses on this model, whichever is larger
    tol = [TOL_F16 if dtype else max(TOL_F32, 4 * logit_error(a, b)) for a, b in zip(oracle(np.float32), want)]
    with lsq.Engine(blob, len(lens), 2, 52) as eng:
        eng.encode(w.src_ids, w.src_lens)
        error = [logit_error(a, b) for a, b in zip(read(eng), want)]
        assert lsq.lsq_debug_small_launches()["encoders"] == one
        lsq.lsq_set_attention_blocks(0)
        try:
            eng.encode(w.src_ids, w.src_lens)
            separate = [logit_error(a, b) for a, b in zip(read(eng), want)]
            assert lsq.lsq_debug_small_launches()["encoders"] == one   # no other
        finally:
            lsq.lsq_set_attention_blocks(64)
    print("one launch", error, "separate launches", separate, "bounds", tol)
    assert all(e <= t for e, t in zip(error + separate, tol + tol))


# alive: unfinished sentences after 40 steps; 5: nothing but the caps ends one
@pytest.mark.parametrize("d,heads,vocab,beam,dtype,n_dec,std,seed,alive", [
    (64, 4, 12, 3, 0, 1, 0.5, 3, 5), (64, 2, 11, 8, 0, 3, 0.5, 3, 5), (128, 8, 12, 4, 1, 2, 0.15, 3, 5), (128, 4, 31, 1, 0, 1, 0.5, 3, 5),
    (64, 4, 31, 3, 0, 1, 0.3, 7, 1), (64, 2, 11, 8, 0, 3, 0.15, 0, 3), (128, 8, 13, 4, 1, 2, 0.3, 3, 4), (128, 4, 31, 1, 0, 1, 0.3, 4, 2),
])
def test_steps_of_a_small_model_in_one_launch(lsq, d, heads, vocab, beam, dtype, n_dec, std, seed, alive):
    """A translation whose steps share launches, against the same one step at a time: sentences that finish early (a small
    vocabulary draws EOS often), caps that differ, histories past 64 positions, chunks that end in the middle."""
    hp = S.HParams(n_enc=1, n_dec=n_dec, d_model=d, n_heads=heads, d_ffn=128, vocab=vocab, max_pos=96, dtype=dtype, cap_extra=70, seed=seed)
    w = S.custom(hp, [1, 4, 9, 2, 20], beam=beam, max_len=80, std=std)
    blob = w.blob(ln_jitter=0.2)
    with lsq.Engine(blob, 6, beam, 80) as eng:
        eng.encode(w.src_ids, w.src_lens)
        counts = []
        while not counts or counts[-1] > 0:
            counts.append(lsq.lsq_decode_step())
        want = eng.get_beams()
        before = lsq.lsq_debug_small_launches()
        assert before["launches"] == before["steps"] == len(counts) > 64 and counts[39] == alive
        got = eng.translate(w.src_ids, w.src_lens, sync_every=1)
        assert all(np.array_equal(a, b) for a, b in zip(got, want))
        after = lsq.lsq_debug_small_launches()
        assert after["launches"] == before["launches"] + 1 and after["steps"] == before["steps"] + 80   # all of them in one
        for n in (1, 7, 64, 1000):
            got = eng.translate(w.src_ids, w.src_lens, sync_every=n)
            assert all(np.array_equal(a, b) for a, b in zip(got, want))
            eng.encode(w.src_ids, w.src_lens)
            for at in range(n, len(counts), n):
                assert lsq.lsq_decode_steps(n) == counts[at - 1] and lsq.lsq_step_index() == at
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.fixture
def foul_workspace(lsq):
    """load(blob, max_batch, beam, max_len, byte): a model in a workspace that held nothing but this byte."""
    import torch

    def load(blob, max_batch, beam, max_len, byte):
        lsq.lsq_free()
        nbytes = lsq.lsq_workspace_bytes(blob, max_batch, beam, max_len)
        held.append((torch.full((nbytes,), byte, dtype=torch.uint8, device="cuda"), torch.cuda.Stream()))
        torch.cuda.synchronize()
        lsq.lsq_set_workspace(held[-1][0].data_ptr(), nbytes, held[-1][1].cuda_stream)
        lsq.lsq_init(blob, max_batch, beam, max_len)

    held = []
    yield load
    lsq.lsq_free()


@pytest.mark.parametrize("d,heads,beam,n_dec,dtype,lens,extra,seed,at", [(64, 4, 8, 4, 0, [1, 4, 9, 2, 6], 140, 1, 128), (128, 8, 8, 1, 1, [1, 4, 9], 80, 0, 64)])
def test_separate_launches_take_over_behind_a_shared_one(lsq, foul_workspace, d, heads, beam, n_dec, dtype, lens, extra, seed, at):
    """A shared launch that ends where the separate ones are ahead, with sentences that it has finished (whose keys, values and table entries were
    never written from there on: here they are NaN) beside others that go on: as one step at a time."""
    hp = S.HParams(n_enc=1, n_dec=n_dec, d_model=d, n_heads=heads, d_ffn=128, vocab=13, max_pos=200, dtype=dtype, cap_extra=extra, seed=seed)
    T = max(lens) + extra + 5
    w = S.custom(hp, lens, beam=beam, max_len=T, std=0.3)
    blob = w.blob(ln_jitter=0.2)
    out = []
    for shared in (True, False):
        foul_workspace(blob, len(lens), beam, T, 0xFF)
        lsq.lsq_encode(w.src_ids, w.src_lens)
        if shared:
            assert lsq.lsq_decode_all(1000) == 0
        else:
            active = []
            while not active or active[-1] > 0:
                active.append(lsq.lsq_decode_step())
            assert 0 < active[at - 1] < len(lens) and len(active) > at + 10
        n = lsq.lsq_debug_small_launches()
        assert n["steps"] == at and n["launches"] == (1 if shared else at)
        out.append(lsq.lsq_get_beams(len(lens), beam, T))
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    assert np.isfinite(out[0][2]).all()


@pytest.mark.parametrize("beam,cap", [(3, 70), (1, 70), (3, 2)])
def test_steps_counted_where_they_shared_a_launch(lsq, beam, cap):
    """decode_all(n) counts its steps as a wait after every n of them would, wherever the sentences finished in a shared launch."""
    hp = S.HParams(n_enc=1, n_dec=1, d_model=64, n_heads=4, d_ffn=128, vocab=11, max_pos=96, dtype=0, cap_extra=cap, seed=1)
    w = S.custom(hp, [1, 4, 9, 2], beam=beam, max_len=80, std=0.3)
    with lsq.Engine(w.blob(ln_jitter=0.2), 4, beam, 80) as eng:
        eng.encode(w.src_ids, w.src_lens)
        finished = 1
        while lsq.lsq_decode_step() > 0:
            finished += 1
        want, last = eng.get_beams(), int((w.src_lens + cap).max())
        assert finished == {(3, 70): 13, (1, 70): 23, (3, 2): 6}[beam, cap] < last   # EOS, or the cap of a shorter sentence, ends them
        for n in (1, 2, 5, 64):
            for before in (0, 1):   # steps taken one by one before
                eng.encode(w.src_ids, w.src_lens)
                for _ in range(before):
                    lsq.lsq_decode_step()
                lsq.lsq_decode_all(n)
                steps = finished - before
                assert lsq.lsq_step_index() == min(last, before + (steps + 1 if n == 1 else -(-steps // n) * n))
                assert lsq.lsq_decode_step() == 0
                assert all(np.array_equal(a, b) for a, b in zip(eng.get_beams(), want))


def test_steps_counted_past_the_end_of_a_shared_launch(lsq):
    """A launch ends behind step 64, where the separate ones are ahead; the sentence is finished inside it.  Waits after every n would have come
    upon that behind a round whose last steps lie beyond the launch."""
    hp = S.HParams(n_enc=1, n_dec=1, d_model=128, n_heads=8, d_ffn=128, vocab=11, max_pos=200, dtype=0, cap_extra=90, seed=30)
    w = S.custom(hp, [4], beam=8, max_len=99, std=0.12)
    with lsq.Engine(w.blob(ln_jitter=0.2), 1, 8, 99) as eng:
        eng.encode(w.src_ids, w.src_lens)
        finished = 1
        while lsq.lsq_decode_step() > 0:
            finished += 1
        want = eng.get_beams()
        assert finished == 42
        for n, index in ((1, 43), (20, 60), (33, 66), (41, 82), (42, 42), (64, 64)):
            eng.encode(w.src_ids, w.src_lens)
            before = lsq.lsq_debug_small_launches()
            lsq.lsq_decode_all(n)
            after = lsq.lsq_debug_small_launches()
            assert after["launches"] == before["launches"] + 1 and after["steps"] == before["steps"] + 64
            assert lsq.lsq_step_index() == index
            assert lsq.lsq_decode_step() == 0
            assert all(np.array_equal(a, b) for a, b in zip(eng.get_beams(), want))


def test_cache_of_sentences_that_ended_inside_a_launch(lsq, foul_workspace):
    """Keys and values as the debug reader hands them back, in a workspace whose every byte was something else: those of the steps that a
    sentence took, whether its launch went on without it or not."""
    hp = S.HParams(n_enc=1, n_dec=1, d_model=64, n_heads=4, d_ffn=128, vocab=11, max_pos=96, dtype=0, cap_extra=70, seed=1)
    w = S.custom(hp, [1, 4, 9, 2], beam=3, max_len=80, std=0.3)
    foul_workspace(w.blob(ln_jitter=0.2), 4, 3, 80, 0x7F)

    def caches():
        return [lsq.lsq_debug_read(kind, (4, 3, 80, 64)) for kind in (lsq.DBG.CACHE_K, lsq.DBG.CACHE_V)]

    lsq.lsq_encode(w.src_ids, w.src_lens)
    lsq.lsq_decode_all(64)
    got = caches()
    lsq.lsq_encode(w.src_ids, w.src_lens)
    steps = np.zeros(4, int)
    for t in range(1, 14):
        lsq.lsq_decode_step()
        fin = lsq.lsq_debug_read(lsq.DBG.FINISHED, (4, 3), np.int32)
        steps[(steps == 0) & fin.all(axis=1)] = t
    want = caches()
    assert steps.max() == 13 and steps.min() < 13 and (steps > 0).all()
    for b in range(4):
        for a, e in zip(got, want):
            assert np.isfinite(a[b, :, :steps[b]]).all() and np.array_equal(a[b, :, :steps[b]], e[b, :, :steps[b]])
