"""More rows than a decoder stack kernel takes, as two launches of it (needs an MI355X)."""
import numpy as np
import pytest

import lsq_synth as S
from tests.parity import lockstep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2010_13887_amd as lib
    lib.load_library()
    yield lib
    lib.lsq_free()


# the fewest rows and the most, halves of one size and of two, beams of 2 and 5; the first number of rows past the line
@pytest.mark.parametrize("batch,beam,twice", [(33, 4, True), (52, 4, True), (26, 5, True), (81, 2, True), (53, 4, False)])
def test_rows_dealt_out_to_two_launches(lsq, batch, beam, twice):
    hp = S.HParams(n_enc=1, n_dec=2, d_model=1024, n_heads=16, d_ffn=4096, vocab=203, max_pos=32, dtype=1, cap_extra=3)
    w = S.custom(hp, [1 + (5 * i) % 7 for i in range(batch)], beam=beam, max_len=12, std=0.03)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, beam, 12) as eng:
        lockstep(lsq, eng, blob, w, max_steps=3, sentences=[0, batch // 2 - 1, batch // 2, batch // 2 + 1, batch - 1])
        assert lsq.lsq_debug_stack_launches()["groups_of_16_or_32"] == (6 if twice else 0)
        one, two = (eng.translate(w.src_ids, w.src_lens, sync_every=n) for n in (1, 4))
        assert all(np.array_equal(a, b) for a, b in zip(one, two))
        assert lsq.lsq_debug_check_canaries() == 0


@pytest.mark.parametrize("batch", [5, 40])
def test_a_limit_on_the_rows_is_not_met_by_halves(lsq, batch):
    """20 rows where 16 are allowed: neither one launch nor two; 160 rows, of which two launches would have 80 each, likewise."""
    hp = S.HParams(n_enc=1, n_dec=2, d_model=1024, n_heads=16, d_ffn=4096, vocab=203, max_pos=32, dtype=1, cap_extra=3)
    w = S.custom(hp, [1 + (5 * i) % 7 for i in range(batch)], beam=4, max_len=12, std=0.03)
    blob = w.blob(ln_jitter=0.1)
    with lsq.Engine(blob, batch, 4, 12) as eng:
        lsq.lsq_set_attention_blocks(16 if batch == 5 else 63)
        try:
            eng.encode(w.src_ids, w.src_lens)
            assert eng.decode_steps(2) > 0
            assert not any(lsq.lsq_debug_stack_launches().values())
        finally:
            lsq.lsq_set_attention_blocks(64)
        assert eng.decode_steps(1) > 0
        assert lsq.lsq_debug_stack_launches()["groups_of_16_or_32"] == (1 if batch == 5 else 2)
        assert lsq.lsq_debug_check_canaries() == 0
