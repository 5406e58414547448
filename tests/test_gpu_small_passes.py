"""Calls of few rows: the fp32 kernels, the row-group GEMM and the accept walk at the sizes where their tiles, splits and
rules change, against the oracle at the library's bars (1e-4 of the row maximum in fp32, 2e-2 in bf16)."""
import numpy as np
import pytest

import oracle

from gpu_harness import Case, compare_draft_tokens, compare_logits_and_greedy, rel_err_rows

pytestmark = pytest.mark.gpu

T17 = dict(topk=[4, 2, 1], widths=[1, 4, 6, 6])
T64 = dict(topk=[4, 2, 2, 2, 1, 1], widths=[1, 4, 8, 12, 13, 13, 13])


# one row with fewer k than a workgroup's waves take in one step; 51 rows of three sequences, a vocabulary beyond the register
# form of the top-k and an ffn that fills no column group; 64 rows with contexts cut into many key ranges; 16 catch-up rows
@pytest.mark.parametrize("tree,batch,ctx,cap,heads,head_dim,ffn,vocab,m", [
    (dict(topk=[], widths=[1]), 1, [1], 8, 1, 64, 36, 21, 1),
    (T17, 3, [5, 64, 200], 256, 3, 128, 100, 4099, 1),
    (T64, 1, [1900], 2048, 5, 64, 452, 1000, 1),
    (dict(topk=[4, 2], widths=[1, 4, 8]), 2, [33, 700], 1024, 1, 128, 688, 4096, 16)])
def test_fp32_calls_match_oracle(tree, batch, ctx, cap, heads, head_dim, ffn, vocab, m):
    c = Case("cfg1", n_layers=2, K=1, batch=batch, ctx=ctx, capacity=cap, hidden=heads * head_dim, n_heads=heads,
             head_dim=head_dim, ffn=ffn, vocab=vocab, tree=tree, max_m=m)
    c.fill_kv_normal(m)
    c.upload_kv()
    feat_in, tok_in = c.normal_draft_inputs(m)
    tokens, scores = c.gpu_draft(feat_in, tok_in)
    _, skipped = compare_draft_tokens(c, tokens, scores, c.oracle_draft(feat_in.astype(np.float64), tok_in))
    assert skipped <= 1
    tt = c.random_tree_tokens()
    feat, lg, greedy = c.gpu_verify(tt)
    rfeat, rlg, rgreedy = c.oracle_verify(tt)
    compare_logits_and_greedy(c, lg, greedy, rlg, rgreedy)
    assert rel_err_rows(feat, rfeat).max() < c.tol
    # and the accepted rows move to the context's end
    k0, _ = c.download_kv()
    a, path, nxt = c.gpu_accept(tt, greedy, commit=True)
    k1, _ = c.download_kv()
    for b in range(batch):
        ra, rpath, rnxt = oracle.accept_greedy(tt[b], greedy[b], c.tree.parent)
        assert (a[b], nxt[b]) == (ra, rnxt) and list(path[b][:ra + 1]) == rpath
        for j, node in enumerate(rpath):
            assert np.array_equal(k1[:, b, :, ctx[b] + j], k0[:, b, :, ctx[b] + node])
        assert int(c.kv["ctx_len"][b].item()) == ctx[b] + ra + 1


# contractions of two 64-k tiles (fewer than a workgroup's waves) and of a count that leaves some waves one tile more, at one,
# two and four activation tiles, each part-filled and full
@pytest.mark.parametrize("hidden,ffn", [(128, 384), (1280, 1408)])
@pytest.mark.parametrize("tree", [dict(topk=[], widths=[1]), T17, dict(topk=[4, 2, 2, 1], widths=[1, 4, 8, 10, 10]), T64])
def test_row_groups_match_oracle(hidden, ffn, tree):
    c = Case("cfg2_small", n_layers=1, K=1, ctx=40, capacity=128, hidden=hidden, n_heads=hidden // 128, head_dim=128, ffn=ffn,
             vocab=600, tree=tree)
    c.fill_kv_normal()
    c.upload_kv()
    tt = c.random_tree_tokens()
    feat, lg, greedy = c.gpu_verify(tt)
    rfeat, rlg, rgreedy = c.oracle_verify(tt)
    compare_logits_and_greedy(c, lg, greedy, rlg, rgreedy)
    assert rel_err_rows(feat, rfeat).max() < c.tol


# the output head of up to 64 rows: one workgroup per eight row groups where that is one round of the chip, at both ends of
# the rule (20480 rows are the last before it, 32768 the last within it) and with a part-filled last group
@pytest.mark.parametrize("vocab", [20480, 20490, 24010, 28672, 28680, 32000, 32768, 32770])
@pytest.mark.parametrize("tree", [dict(topk=[], widths=[1]), dict(topk=[3, 2, 1], widths=[1, 3, 6, 6]), T17, T64])
def test_wide_output_head_matches_oracle(vocab, tree):
    c = Case("cfg2_small", n_layers=1, K=1, ctx=20, capacity=96, hidden=256, n_heads=2, head_dim=128, ffn=256, vocab=vocab, tree=tree)
    c.fill_kv_normal()
    c.upload_kv()
    tt = c.random_tree_tokens()
    feat, lg, greedy = c.gpu_verify(tt)
    rfeat, rlg, rgreedy = c.oracle_verify(tt)
    compare_logits_and_greedy(c, lg, greedy, rlg, rgreedy)


# smaller vocabularies: four, six or eight row groups a workgroup, all of them part-filled somewhere; logits' rows not 16-byte aligned
@pytest.mark.parametrize("vocab", [5, 64, 1001, 4001, 16384, 16390, 19999])
@pytest.mark.parametrize("tree", [dict(topk=[], widths=[1]), T17, T64])
def test_output_head_of_small_vocabularies(vocab, tree):
    c = Case("cfg2_small", n_layers=1, K=1, ctx=20, capacity=96, hidden=256, n_heads=2, head_dim=128, ffn=256, vocab=vocab, tree=tree)
    c.fill_kv_normal()
    c.upload_kv()
    tt = c.random_tree_tokens()
    feat, lg, greedy = c.gpu_verify(tt)
    rfeat, rlg, rgreedy = c.oracle_verify(tt)
    compare_logits_and_greedy(c, lg, greedy, rlg, rgreedy)
    assert rel_err_rows(feat, rfeat).max() < c.tol
    assert np.array_equal(greedy, lg.argmax(-1))


@pytest.mark.parametrize("V", [700, 5000])
def test_fp32_top_k_never_repeats_a_token(V):
    """A not-a-number among the logits compares false with everything, so what a lane of the workgroup has seen of the others
    goes by the order it met them in; the tokens handed out must be different ones all the same."""
    import torch
    from koala_synth import make_tree
    from test_gpu_sampling_rows import _context
    tree = make_tree([6], [1, 6])
    c, g, lm, blocks = _context(V, tree, 1)
    for block in blocks:
        block.zero_()                                     # a head's output is its input
    feat = torch.zeros(1, 1, 128, device="cuda")
    feat[0, 0, 0] = 1.0                                   # and the logits are the first column of the output head
    for nan, largest, second in ((5, 37, 36), (5, 69, 64), (3, 133, 130), (0, 1, 2), (255, 511, 254)):
        lm.zero_()
        lm[:, 0] = torch.randn(V, generator=g, device="cuda")
        lm[largest, 0], lm[second, 0] = 50.0, 40.0
        for row in (False, True):
            if row:
                lm[nan, 0] = float("nan")
            tok, scores = torch.zeros(1, 7, dtype=torch.int32, device="cuda"), torch.zeros(1, 7, device="cuda")
            c.draft_expand(1, feat, torch.ones(1, 1, dtype=torch.int32, device="cuda"), 1, tok, scores)
            kids = [int(tok[0, i]) for i in sorted(range(1, 7), key=lambda i: tree.rank[i])]
            assert len(set(kids)) == 6 and 0 <= min(kids) and max(kids) < V, (nan, largest, second, kids)
            if not row:
                assert kids == torch.topk(lm[:, 0], 6).indices.tolist()


def test_fp32_batches_beyond_16383_sequences():
    """Four groups of sixteen tree rows for each of 16400 sequences: more attention workgroups than the third dimension of a
    launch holds.  Equal sequences give equal bits, those of a call of one sequence."""
    import torch
    import paper_2408_08146_amd as K
    from koala_synth import make_tree
    H, V, F, batch, cap = 64, 12, 8, 16400, 64
    tree = make_tree([8, 6], [1, 8, 40])
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda") * 0.1
    one = torch.ones(H, device="cuda")
    w = dict(embed=rnd(V, H), lm_head=rnd(V, H), final_norm=one, fc=None, draft=[rnd(H, H)] * 2,
             layers=[(one, rnd(3 * H, H), rnd(H, H), one, rnd(2 * F, H), rnd(H, F))])
    shape = dict(hidden=H, n_heads=1, head_dim=64, ffn=F, vocab=V, n_layers=1, rms_eps=1e-6, rope_base=1e4, dtype=K.KOALA_FP32)
    rows, tokens, results = rnd(2, 8, 64), torch.randint(0, V, (1, tree.n_nodes), generator=g, device="cuda").int(), []
    for n in (1, batch):
        c = K.KoalaContext(shape, dict(kind=K.KOALA_DRAFT_MEDUSA, K=1, medusa_heads=2, max_m=1), tree, n)
        kv = K.alloc_kv(dict(n_layers=1, n_heads=1, head_dim=64, dtype="fp32"), n, cap, "cuda")
        kv["target_k"][..., :8, :], kv["target_v"][..., :8, :] = rows[0], rows[1]
        kv["ctx_len"].fill_(8)
        c.bind(w, kv, torch.empty(c.workspace_bytes(), dtype=torch.uint8, device="cuda"))
        feat, greedy = torch.zeros(n, tree.n_nodes, H, device="cuda"), torch.zeros(n, tree.n_nodes, dtype=torch.int32, device="cuda")
        c.tree_verify(n, tokens.expand(n, -1).contiguous(), feat, None, greedy)
        results.append((feat, greedy))
    assert results[0][0].abs().max() > 0.1
    for a, b in zip(*results):
        assert (a == b).all()


def test_accept_takes_the_first_of_equal_children():
    """Siblings with the same token: the walk goes to the lowest-numbered one, in every sequence."""
    c = Case("cfg5_small", n_layers=1, K=1)
    c.fill_kv_normal()
    c.upload_kv()
    rng = np.random.default_rng(3)
    for _ in range(20):
        tt = rng.integers(0, 2, (c.B, c.T)).astype(np.int32)
        g = rng.integers(0, 2, (c.B, c.T)).astype(np.int32)
        a, path, nxt = c.gpu_accept(tt, g, commit=False)
        for b in range(c.B):
            ra, rpath, rnxt = oracle.accept_greedy(tt[b], g[b], c.tree.parent)
            assert (a[b], nxt[b]) == (ra, rnxt) and list(path[b][:ra + 1]) == rpath and all(path[b][ra + 1:] == -1)
