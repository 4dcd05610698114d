"""Encoder and prefill of a few hundred rows: what a sentence's rows become does not depend on what is encoded beside it (needs an MI355X)."""
import numpy as np
import pytest

import lsq_synth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2010_13887_amd as lib
    lib.load_library()
    yield lib
    lib.lsq_free()


# within each list the products run on the same tiles, so a row's sums have one order: the same bits
@pytest.mark.parametrize("d,heads,batches", [(512, 8, (1, 2, 5, 6, 10)), (1024, 16, (1, 2, 3, 4))])
def test_a_sentence_is_encoded_the_same_alone_and_beside_others(lsq, d, heads, batches):
    hp = S.HParams(n_enc=2, n_dec=2, d_model=d, n_heads=heads, d_ffn=4 * d, vocab=97, max_pos=64, dtype=1, cap_extra=2)
    w = S.custom(hp, [50] * max(batches), beam=1, max_len=52, std=0.03)
    with lsq.Engine(w.blob(ln_jitter=0.1), max(batches), 1, 52) as eng:
        got = []
        for B in batches:
            eng.encode(w.src_ids[:B], w.src_lens[:B])
            got.append([eng.debug(lsq.DBG.MEMORY, (50 * B, d))[:50], eng.debug(lsq.DBG.CROSS_KV + 1, (50 * B, 2 * d))[:50]])
    for other in got[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got[0], other))


@pytest.mark.parametrize("batches", [(1, 2, 3, 5)])
def test_a_prompt_is_prefilled_the_same_alone_and_beside_others(lsq, batches):
    hp = S.HParams(arch=1, n_enc=0, n_dec=2, d_model=768, n_heads=12, d_ffn=3072, vocab=97, dtype=1, max_pos=64, act=1, norm=1, cap_extra=2,
                   sample_topk=4)
    w = S.custom(hp, [51] * max(batches), beam=1, max_len=53, std=0.03)
    with lsq.Engine(w.blob(ln_jitter=0.1), max(batches), 1, 53) as eng:
        got = []
        for B in batches:
            eng.encode(w.src_ids[:B], w.src_lens[:B])
            got.append([eng.debug(kind + 1, (B, 53, 768))[0, :50] for kind in (lsq.DBG.CACHE_K, lsq.DBG.CACHE_V)])
    for other in got[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got[0], other))
