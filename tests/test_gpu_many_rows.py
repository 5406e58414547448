"""Batched verification (the many-row GEMM): launches whose weight row groups are split along K inside the kernel, at row
counts around its tile blocks, head dimensions of 64 and 128, against the oracle at the bf16 bar."""
import numpy as np
import pytest

from gpu_harness import Case, compare_logits_and_greedy, rel_err_rows

pytestmark = pytest.mark.gpu


# rows: 65 (five tiles, one row in the last), 120, 128, 195, 243 (sixteen tiles: two blocks of eight)
@pytest.mark.parametrize("batch,widths,head_dim", [(5, [1, 4, 8], 128), (2, [1, 4, 8, 12, 12, 12, 11], 128), (4, [1, 4, 8, 12, 7], 64),
                                                   (5, [1, 4, 8, 12, 14], 128), (9, [1, 4, 8, 14], 64)])
def test_split_groups_match_oracle(batch, widths, head_dim):
    c = Case("cfg5_small", n_layers=1, batch=batch, ctx=(30, 90), capacity=192, hidden=1536, n_heads=1536 // head_dim,
             head_dim=head_dim, ffn=2560, vocab=1000, tree=dict(topk=[4, 2, 2, 2, 1, 1][:len(widths) - 1], widths=widths))
    c.fill_kv_normal()
    c.upload_kv()
    tt = c.random_tree_tokens()
    feat, lg, greedy = c.gpu_verify(tt)
    rfeat, rlg, rgreedy = c.oracle_verify(tt)
    compare_logits_and_greedy(c, lg, greedy, rlg, rgreedy)
    assert rel_err_rows(feat, rfeat).max() < c.tol
    # the same launches again give the same bits: the order of the additions does not depend on who arrives last
    for _ in range(3):
        feat2, lg2, _ = c.gpu_verify(tt)
        assert np.array_equal(lg, lg2) and np.array_equal(feat, feat2)


# vocabularies that leave a row group, a workgroup's groups or four columns of a lane partly empty; 65 and 240 rows
@pytest.mark.parametrize("vocab", [5, 63, 257, 1001, 4099, 12345, 20481])
@pytest.mark.parametrize("batch,widths", [(5, [1, 4, 8]), (4, [1, 4, 8, 16, 16, 15])])
def test_output_head_of_many_rows(vocab, batch, widths):
    """Logits finished in the GEMM: as the oracle's, and the greedy token is the first largest of the logits returned, also
    where no logits are returned."""
    c = Case("cfg5_small", n_layers=1, batch=batch, ctx=(20, 40), capacity=128, hidden=256, n_heads=2, head_dim=128, ffn=256,
             vocab=vocab, tree=dict(topk=[4, 2, 2, 1, 1][:len(widths) - 1], widths=widths))
    c.fill_kv_normal()
    c.upload_kv()
    tt = c.random_tree_tokens()
    feat, lg, greedy = c.gpu_verify(tt)
    rfeat, rlg, rgreedy = c.oracle_verify(tt)
    compare_logits_and_greedy(c, lg, greedy, rlg, rgreedy)
    assert rel_err_rows(feat, rfeat).max() < c.tol
    assert np.array_equal(greedy, lg.argmax(-1))
    assert np.array_equal(greedy, c.gpu_verify(tt, want_logits=False)[2])
