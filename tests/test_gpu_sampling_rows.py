"""Sampled drafting and stochastic acceptance at vocabularies around the sizes where the kernels change form (rows in
registers up to 4096, 16384 and 32768 tokens, in memory beyond), with masked (-inf) logits, and the heads of a Medusa-style
draft in groups of one launch (more heads than a launch takes, more rows than the grouped form takes).

A decision is compared where the oracle's own does not change when the uniforms move by 2e-6, ten times the relative error
of the device's fp32 exponentials; the fraction compared is asserted."""
import numpy as np
import pytest

import oracle
from koala_synth import chain_tree, make_tree

pytestmark = pytest.mark.gpu
DELTA = 2e-6


def _context(V, tree, batch, dtype="fp32", hidden=128, heads=None):
    import torch
    import paper_2408_08146_amd as K
    g = torch.Generator(device="cuda").manual_seed(V + tree.n_nodes)
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    rnd = lambda *s: (torch.randn(*s, generator=g, device="cuda") * 0.05).to(dt)
    mat = K.device_matrix if dtype == "bf16" else (lambda a: a)
    H, F = hidden, 256
    lm, blocks = rnd(V, H) * 4, [rnd(H, H) for _ in range(max(1, tree.depth))]
    layer = (torch.ones(H, device="cuda", dtype=dt), mat(rnd(3 * H, H)), mat(rnd(H, H)), torch.ones(H, device="cuda", dtype=dt),
             mat(rnd(2 * F, H)), mat(rnd(H, F)))
    w = dict(embed=rnd(V, H), lm_head=mat(lm), final_norm=torch.ones(H, device="cuda", dtype=dt), layers=[layer], fc=None,
             draft=[mat(b) for b in blocks])
    cfg = dict(n_layers=1, n_heads=H // 64, head_dim=64, dtype=dtype)
    kv = K.alloc_kv(cfg, batch, 128, "cuda")
    kv["ctx_len"].fill_(8)
    shape = dict(hidden=H, n_heads=H // 64, head_dim=64, ffn=F, vocab=V, n_layers=1, rms_eps=1e-6, rope_base=1e4,
                 dtype=K.KOALA_FP32 if dtype == "fp32" else K.KOALA_BF16)
    c = K.KoalaContext(shape, dict(kind=K.KOALA_DRAFT_MEDUSA, K=1, medusa_heads=max(1, tree.depth), max_m=2), tree, batch)
    ws = torch.full((c.workspace_bytes(),), 0x7f, dtype=torch.uint8, device="cuda")
    c.bind(w, kv, ws)
    return c, g, lm, blocks


def _sample(c, g, tree, V, batch, hidden, temperature=0.8):
    import torch
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")
    feat = torch.randn(batch, 2, hidden, generator=g, device="cuda")
    u = torch.rand(batch, tree.n_nodes, generator=g, device="cuda")
    tok, logits = i32(batch, tree.n_nodes), torch.zeros(batch, tree.n_nodes, V, device="cuda")
    c.draft_expand_sample(batch, feat, i32(batch, 2) + 1, 2, u, temperature, tok, logits)
    torch.cuda.synchronize()
    return feat, u, tok, logits


@pytest.mark.parametrize("V", [100, 4096, 4099, 16384, 16385, 32000, 32768, 32771])
def test_draws_and_acceptance_at_every_row_form(V):
    import torch
    tree, batch, temperature = make_tree([5, 3, 2], [1, 5, 9, 7]), 2, 0.8
    c, g, _, _ = _context(V, tree, batch)
    _, u, tok, logits = _sample(c, g, tree, V, batch, 128, temperature)
    ch = [sorted(k, key=lambda x: tree.rank[x]) for k in oracle.children_lists(tree.parent)]
    u_np, tok_np, lg = u.double().cpu().numpy(), tok.cpu().numpy(), logits.double().cpu().numpy()
    seen = total = 0
    for b in range(batch):
        for n in range(tree.n_nodes):
            if not ch[n]:
                continue
            p, us = oracle.softmax_t(lg[b, n], temperature), u_np[b, ch[n]]
            want = [oracle.draw_without_replacement(p, np.clip(us + s, 0, 1 - 1e-12)) for s in (0.0, -DELTA, DELTA)]
            total += len(us)
            for j, x in enumerate(ch[n]):
                if not want[0][:j + 1] == want[1][:j + 1] == want[2][:j + 1]:
                    break
                assert tok_np[b, x] == want[0][j], (V, b, n, j)
                seen += 1
    assert seen >= 0.7 * total, (seen, total)
    # acceptance: target logits near the draft's, some of both masked out
    seen = 0
    for trial in range(6):
        q = logits + 0.5 * torch.randn(logits.shape, generator=g, device="cuda") * (trial % 3)
        d = logits.clone()
        if trial >= 3:
            q[:, :, V // 2:V // 2 + 7] = float("-inf")
            d[:, :, V // 3:V // 3 + 5] = float("-inf")
        ua, ur = (torch.rand(batch, tree.n_nodes, generator=g, device="cuda") for _ in range(2))
        acc, path, nxt = (torch.zeros(s, dtype=torch.int32, device="cuda") for s in ((batch,), (batch, tree.depth + 1), (batch,)))
        c.accept_sample(batch, tok, q, d, ua, ur, temperature, acc, path, nxt, False)
        torch.cuda.synchronize()
        qn, dn = q.double().cpu().numpy(), d.double().cpu().numpy()
        for b in range(batch):
            walk = lambda s: oracle.accept_sample(tok_np[b], tree.parent, tree.rank,
                                                  [oracle.softmax_t(r, temperature) for r in qn[b]],
                                                  [oracle.softmax_t(r, temperature) for r in dn[b]],
                                                  np.clip(ua[b].double().cpu().numpy() + s, 0, 1),
                                                  np.clip(ur[b].double().cpu().numpy() + s, 0, 1 - 1e-12))
            want = [walk(s) for s in (0.0, -DELTA, DELTA)]
            if want[0] == want[1] == want[2]:
                a, p, n = want[0]
                assert (int(acc[b]), path[b, :a + 1].tolist(), int(nxt[b])) == (a, list(p), n), (V, trial, b)
                assert (path[b, a + 1:] == -1).all()
                seen += 1
    assert seen >= 8, seen


@pytest.mark.parametrize("V", [100, 4099, 16385, 32000, 32768, 32771])
def test_infinite_temperature_is_uniform(V):
    """1/temperature is zero: every token weighs the same, and columns past the vocabulary weigh nothing.  Sums of ones and
    the product of an fp32 u with a count are exact in fp64, so each draw is known: id number floor(u * left) among those not
    drawn yet.  Equal distributions accept every first child."""
    import torch
    tree, batch, inf = make_tree([5, 3, 2], [1, 5, 9, 7]), 2, float("inf")
    c, g, _, _ = _context(V, tree, batch)
    _, u, tok, logits = _sample(c, g, tree, V, batch, 128, inf)
    ch = [sorted(k, key=lambda x: tree.rank[x]) for k in oracle.children_lists(tree.parent)]
    u_np, tok_np = u.double().cpu().numpy(), tok.cpu().numpy()
    for b in range(batch):
        for n in range(tree.n_nodes):
            left = list(range(V))
            for x in ch[n]:
                assert tok_np[b, x] == left.pop(int(u_np[b, x] * len(left))), (V, b, n, x)
    ua, ur = torch.full((batch, tree.n_nodes), 0.5, device="cuda"), torch.full((batch, tree.n_nodes), 0.25, device="cuda")
    acc, path, nxt = (torch.zeros(s, dtype=torch.int32, device="cuda") for s in ((batch,), (batch, tree.depth + 1), (batch,)))
    c.accept_sample(batch, tok, logits, logits, ua, ur, inf, acc, path, nxt, False)
    for b in range(batch):
        want, cur = [0], 0
        while ch[cur]:
            cur = ch[cur][0]
            want.append(cur)
        assert path[b, :len(want)].tolist() == want and int(acc[b]) == len(want) - 1
        # V equal probabilities of one rounding each: the id is within one of a quarter of the vocabulary
        assert abs(int(nxt[b]) - V // 4) <= 1


@pytest.mark.parametrize("depth,batch", [(1, 1), (4, 8), (9, 3), (8, 8), (9, 8), (3, 40)])
def test_grouped_heads(depth, batch):
    """Logits of every head against float64: bf16-valued weights, inputs rounded to fp16 twice on the way (2^-11 of a value
    each), so 2e-3 of a row's norm."""
    import torch
    V, H, tree = 1000, 512, chain_tree(depth)
    c, g, lm, blocks = _context(V, tree, batch, "bf16", H)
    feat, _, _, logits = _sample(c, g, tree, V, batch, H)
    x0 = feat[:, -1].double()
    for j in range(depth):
        y = x0 @ blocks[j].double().T
        want = (x0 + y * torch.sigmoid(y)) @ lm.double().T
        err = (logits[:, j].double() - want).norm(dim=1) / want.norm(dim=1)
        assert err.max().item() < 2e-3, (j, err)


@pytest.mark.parametrize("V, batch", [(100, 1), (100, 11), (300, 12), (4099, 40), (300, 93), (300, 94), (300, 186), (300, 187), (16385, 14)])
@pytest.mark.parametrize("near", [True, False])
def test_acceptance_of_a_batch_equals_that_of_its_sequences(V, batch, near):
    """22 nodes a sequence, all at once in up to 2048 workgroups (93 sequences), the first 256 of which (11 sequences) start
    without a look at what other nodes have told, and in turn beyond.  near: target distributions near their draft's, whose
    paths go down the tree; else unrelated ones, where nodes are told that their branch was turned down while they are under
    way.  Whichever way, the outcome of a sequence is its own, bit for bit, and a call leaves nothing behind for the next."""
    import torch
    tree, temperature = make_tree([5, 3, 2], [1, 5, 9, 7]), 0.8
    c, g, _, _ = _context(V, tree, batch)
    T, D = tree.n_nodes, tree.depth
    d = 3.0 * torch.randn(batch, T, V, generator=g, device="cuda")
    q = (d if near else 0.0) + 1.5 * torch.randn(batch, T, V, generator=g, device="cuda")
    tok = torch.zeros(batch, T, dtype=torch.int32, device="cuda")
    top = torch.topk(d, 5, dim=2).indices.to(torch.int32)
    for i in range(1, T):
        tok[:, i] = top[:, int(tree.parent[i]), int(tree.rank[i])]
    ua, ur = (torch.rand(batch, 24, generator=g, device="cuda")[:, :T].contiguous() for _ in range(2))

    def accept(q, d, tok, ua, ur):
        n = tok.shape[0]
        acc, path, nxt = (torch.full(s, -7, dtype=torch.int32, device="cuda") for s in ((n,), (n, D + 1), (n,)))
        c.accept_sample(n, tok, q, d, ua, ur, temperature, acc, path, nxt, False)
        return acc, path, nxt

    whole = [accept(q, d, tok, ua, ur) for _ in range(3)]
    for again in whole[1:]:
        for x, y in zip(again, whole[0]):
            assert torch.equal(x, y)
    for b in range(min(batch, 40)):   # copies: rows of a batch of 22 nodes need not be 16-byte aligned
        one = accept(*(x[b:b + 1].clone() for x in (q, d, tok, ua, ur)))
        for x, y in zip(one, whole[0]):
            assert torch.equal(x[0], y[b]), b
    acc = whole[0][0]
    if batch > 8:
        assert int(acc.min()) == 0 and (int(acc.max()) >= 2 if near else float(acc.float().mean()) < 0.5)   # rejections at once, and paths


def test_acceptance_along_a_chain_of_64_nodes():
    """The deepest tree: equal logits accept every node (ratio 1 is above any uniform), a first uniform of 1 - 2^-24 beside a
    draft that has its token too often rejects the first."""
    import torch
    V, tree = 300, chain_tree(63)
    c, g, _, _ = _context(V, tree, 2)
    T = tree.n_nodes
    d = torch.randn(2, T, V, generator=g, device="cuda")
    q = d.clone()
    tok = torch.zeros(2, T, dtype=torch.int32, device="cuda")
    tok[:, 1:] = d.argmax(2).to(torch.int32)[:, :-1]
    q[1, 0, int(tok[1, 1])] -= 2.0
    ua, ur = torch.full((2, T), 1 - 2.0 ** -24, device="cuda"), torch.full((2, T), 0.5, device="cuda")
    ua[0] = 0.5
    acc, path, nxt = (torch.zeros(s, dtype=torch.int32, device="cuda") for s in ((2,), (2, T), (2,)))
    c.accept_sample(2, tok, q, d, ua, ur, 1.0, acc, path, nxt, False)
    assert acc.tolist() == [63, 0]
    assert path[0].tolist() == list(range(64)) and path[1].tolist() == [0] + [-1] * 63
