"""The dense products of the training step at the edges of their tiles (rows 32 / 64 / 128 and one more, columns not
a multiple of 64, contraction lengths around a chunk of 32, split and unsplit sums) against float64.

Bound: a product may be off by 2^-24 (the products of low pieces that are left out) and each sum is rounded at most once per
term, 2.53e-8 of it each, so over K terms the relative error of a sum of random terms is about 2.53e-8 sqrt((K + 1) / 2); five
times that, at K = 1030, is 2.9e-6 in the 2-norm (the fp32 additions of the splits and of the residual block are fewer).  The
sums by themselves are held to that bound itself further down."""
import numpy as np
import pytest

from test_train_forms import form

pytestmark = pytest.mark.gpu

TOL = 3.3e-6


def _rel(got, ref):
    got = got.double().cpu().numpy()
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def _head(n, H, V, K, seed):
    import torch
    rng = np.random.default_rng(seed)
    f32 = lambda a: a.astype(np.float32)
    blocks = [f32(rng.normal(size=(H, H)) * 0.05) for _ in range(K)]
    w_lm, h, g = f32(rng.normal(size=(V, H)) * 0.1), f32(rng.normal(size=(n, H))), f32(rng.normal(size=(n, V)) * 0.1)
    dev = lambda a: torch.from_numpy(a.copy()).cuda()
    return blocks, w_lm, h, g, dev


def _head_ref(blocks, w_lm, h, g, lr):
    from oracle import train as T
    b64 = [b.astype(np.float64) for b in blocks]
    logits, _ = T.medusa_head_forward(b64, w_lm.astype(np.float64), h.astype(np.float64))
    new, grads = T.medusa_head_step(b64, w_lm.astype(np.float64), h.astype(np.float64), g.astype(np.float64), lr)
    return logits, grads


@pytest.mark.parametrize("n,H,V,K", [(1, 64, 100, 1), (16, 63, 129, 2), (32, 64, 512, 1), (33, 97, 1030, 2), (64, 128, 300, 1),
                                     (65, 260, 1000, 2), (128, 96, 700, 1), (129, 130, 1030, 2), (300, 65, 260, 1)])
def test_head_products(n, H, V, K):
    import torch
    import paper_2408_08146_amd as KO
    blocks, w_lm, h, g, dev = _head(n, H, V, K, n + H)
    lr = 0.5
    logits, grads = _head_ref(blocks, w_lm, h, g, lr)
    db = [dev(b) for b in blocks]
    head = KO.MedusaHeadTrainer(db, dev(w_lm))
    d = torch.zeros(n, V, device="cuda")
    head.forward(dev(h), d)
    assert _rel(d, logits) < TOL
    head.step(dev(h), dev(g), lr)
    for k in range(K):
        # the update is seen through the rounding of the weights themselves: 2^-24 of a weight each
        upd = db[k].double().cpu().numpy() - blocks[k]
        floor = 2.0 ** -24 * np.linalg.norm(blocks[k])
        assert np.linalg.norm(upd + lr * grads[k]) < TOL * 4 * np.linalg.norm(lr * grads[k]) + floor


@pytest.mark.parametrize("terms", [1, 2, 3, 4, 8, 16, 32, 33, 64, 65, 130, 1030])
@pytest.mark.parametrize("form", ["forward", "input_gradient", "update"])
@pytest.mark.parametrize("scale", [0, -118])
def test_sums_are_as_exact_as_fp32_chains(form, terms, scale):
    """Every form of product against float64, at the error of a chain of fp32 multiply-adds: each addition is rounded once, a
    rounding is 2^-24 / sqrt(3) * sqrt((1 - 1/4) / (2 ln 2)) = 2.53e-8 of a value (2-norm, mantissas as in random data), and the
    partial sums of K random terms are sqrt(1 .. K) of a term, so sqrt((K + 1) / 2) of that for the whole; 15 % on top for the
    finite sample and because the products and additions of pieces may round a little more than once at a single term.
    The head is set up so that nothing else rounds: zero blocks pass h on as it is, and powers of two or identities stand
    in for the other factors.  scale: one operand in units of 2^-118, where low bits are below the smallest normal bfloat16,
    the other in units of 2^60."""
    import torch
    import paper_2408_08146_amd as KO
    rng = np.random.default_rng(terms)
    small, large = np.float32(2.0 ** scale), np.float32(2.0 ** (60 if scale else 0))
    f32 = lambda *s: rng.normal(size=s).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    exact = lambda a, b: a.astype(np.float64) @ b.astype(np.float64)
    if form == "forward":            # d = h w_lm^T
        h, w_lm = f32(40, terms) * small, f32(1000, terms) * large
        got, want = torch.zeros(40, 1000, device="cuda"), exact(h, w_lm.T)
        KO.MedusaHeadTrainer([dev(np.zeros((terms, terms)))], dev(w_lm)).forward(dev(h), got)
    elif form == "input_gradient":   # W = -(g w_lm)^T / 2 * 2 with an identity for h
        g, w_lm, w = f32(128, terms) * small, f32(terms, 128) * large, dev(np.zeros((128, 128)))
        KO.MedusaHeadTrainer([w], dev(w_lm)).step(dev(np.eye(128)), dev(g), 2.0)
        got, want = -w.T, exact(g, w_lm)
    else:                            # W = -g^T h, with w_lm twice an identity
        g, h, w = f32(terms, 200) * small, f32(terms, 200) * large, dev(np.zeros((200, 200)))
        KO.MedusaHeadTrainer([w], dev(2 * np.eye(200))).step(dev(h), dev(g), 1.0)
        got, want = -w, exact(g.T, h)
    assert _rel(got, want) < 1.15 * 2.53e-8 * np.sqrt((terms + 1) / 2)


def _room(n, H):   # floats that a head's workspace has for partial sums: eight slots of n x H in whole 256 bytes
    return 8 * ((n * H * 4 + 255) // 256 * 64)


def _both_products(n, V, H):
    """d = h w_lm^T and g w_lm, set up and bounded as above, where V and H are both the length of the sums and the number of
    columns"""
    import torch
    import paper_2408_08146_amd as KO
    rng = np.random.default_rng(n + V + H)
    f32 = lambda *s: rng.normal(size=s).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    h, g, w_lm = f32(n, H), f32(n, V), f32(V, H)
    bound = lambda terms: 1.15 * 2.53e-8 * np.sqrt((terms + 1) / 2)
    got, w = torch.zeros(n, V, device="cuda"), dev(np.zeros((H, H)))
    KO.MedusaHeadTrainer([w], dev(w_lm)).forward(dev(h), got)
    assert _rel(got, h.astype(np.float64) @ w_lm.T.astype(np.float64)) < bound(H)
    m = min(n, H)
    KO.MedusaHeadTrainer([w], dev(w_lm)).step(dev(np.eye(n, H)), dev(g), 2.0)   # W = -(g w_lm)^T / 2 * 2 [identity]
    assert _rel(-w.T[:m], g[:m].astype(np.float64) @ w_lm.astype(np.float64)) < bound(V)


@pytest.mark.parametrize("n,V,H", [(1, 32, 64), (32, 31, 64), (33, 33, 63), (48, 127, 65), (49, 128, 127), (64, 129, 128), (65, 160, 192),
                                   (96, 161, 193), (97, 64, 320), (128, 65, 1000), (129, 1000, 96), (200, 515, 449), (20, 4099, 640)])
def test_products_of_few_columns_or_terms(n, V, H):
    """Matrices around 32 columns and 64 terms, one row tile up to several blocks of them"""
    _both_products(n, V, H)


@pytest.mark.parametrize("n,tiles", [(1, 2), (20, 2), (33, 3), (60, 4), (90, 6), (128, 8), (129, 6), (200, 8), (300, 8)])
@pytest.mark.parametrize("V,H", [(4099, 1001), (5056, 1024)])
def test_products_at_the_edges_of_a_streamed_tile(n, tiles, V, H):
    """Both forms streamed, with each count of row tiles and several blocks of them; 4099 x 1001: the last columns' and the last
    stage's loads are moved back into what the one before has taken, as columns and as terms; 5056 x 1024: whole stages."""
    assert form(n, V, H, False, _room(n, H))[0] == tiles and form(n, H, V, True, _room(n, H))[0] == tiles
    _both_products(n, V, H)


def _forward_and_update(h, w_lm, g, lr=1.0):
    """d = h w_lm^T, and W = -(g w_lm / 2)^T h from a zero W"""
    import torch
    import paper_2408_08146_amd as KO
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    n, (V, H) = len(h), w_lm.shape
    d, w = torch.zeros(n, V, device="cuda"), torch.zeros(H, H, device="cuda")
    KO.MedusaHeadTrainer([w], dev(w_lm)).forward(dev(h), d)
    w.zero_()
    KO.MedusaHeadTrainer([w], dev(w_lm)).step(dev(h), dev(g), lr)
    return d.double().cpu().numpy(), w.double().cpu().numpy()


@pytest.mark.parametrize("n", [20, 33, 60, 90, 128, 200])
def test_infinities_in_a_streamed_product(n):
    """One infinite weight among the columns and the terms that the last loads take a second time, in both forms: its column of
    the result is infinite, the rest, the other tiles' and its own, what it would be without (bound as for sums, over what the
    update behind the input gradient adds)."""
    V, H, v0, j0 = 4099, 1001, 4080, 948   # terms 937 .. 959 of 1001 and 4035 .. 4095 of 4099 are in two stages
    assert form(n, V, H, False, _room(n, H))[0] and form(n, H, V, True, _room(n, H))[0]
    rng = np.random.default_rng(n)
    h, g = (np.abs(rng.normal(size=s)).astype(np.float32) for s in ((n, H), (n, V)))
    w_lm = rng.normal(size=(V, H)).astype(np.float32)
    d_ref = h.astype(np.float64) @ w_lm.T
    w_ref = -(g.astype(np.float64) @ w_lm / 2).T @ h
    w_lm[v0, j0] = np.inf
    d, w = _forward_and_update(h, w_lm, g)
    assert (d[:, v0] == np.inf).all() and (w[j0] == -np.inf).all()
    for got, ref, at in ((d, d_ref, (slice(None), v0)), (w, w_ref, (j0, slice(None)))):
        got[at] = ref[at] = 0.0
        assert np.isfinite(got).all()
        assert np.linalg.norm(got - ref) < 5e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [20, 60, 128, 200])
@pytest.mark.parametrize("weights", [True, False])
def test_small_operands_of_a_streamed_product(n, weights):
    """One operand in units of 2^-118, where low bits are below the smallest normal bfloat16, the other in units of 2^60: the
    weights or the activations, in both forms.  An identity for h makes the update a copy of the input gradient."""
    import torch
    import paper_2408_08146_amd as KO
    V, H = 4099, 1001
    assert form(n, V, H, False, _room(n, H))[0] and form(n, H, V, True, _room(n, H))[0]
    rng = np.random.default_rng(n)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    scale = (60, -118) if weights else (-118, 60)
    f32 = lambda e, *s: rng.normal(size=s).astype(np.float32) * np.float32(2.0 ** e)
    h, g, w_lm = f32(scale[0], n, H), f32(scale[0], n, V), f32(scale[1], V, H)
    bound = lambda terms: 1.15 * 2.53e-8 * np.sqrt((terms + 1) / 2)
    d, w = torch.zeros(n, V, device="cuda"), dev(np.zeros((H, H)))
    KO.MedusaHeadTrainer([w], dev(w_lm)).forward(dev(h), d)
    assert _rel(d, h.astype(np.float64) @ w_lm.T.astype(np.float64)) < bound(H)
    KO.MedusaHeadTrainer([w], dev(w_lm)).step(dev(np.eye(n, H)), dev(g), 2.0)
    assert _rel(-w.T[:n], g.astype(np.float64) @ w_lm.astype(np.float64)) < bound(V)


@pytest.mark.parametrize("n,V,H,streams", [(20, 4099, 1001, True), (40, 4099, 1001, True), (48, 5056, 1024, True), (20, 300, 64, False),
                                          (40, 300, 130, False)])
@pytest.mark.parametrize("small", [-110, -125, -140])
def test_input_gradients_of_values_of_any_size(n, V, H, streams, small):
    """Gradients of which every second row is in units of 2^small, beside rows around 2^20 in the same tile: each row as exact as
    by itself.  Bound as for sums, and for results below the smallest normal float, whole multiples of 2^-149, half of one for
    each split of a sum and one for the product with SiLU'(0) = 1/2, which the learning rate doubles.  An identity for h makes the
    update, by up to 48 rows, a copy of the input gradient."""
    import torch
    import paper_2408_08146_amd as KO
    tiles, splits = form(n, H, V, True, _room(n, H))
    assert bool(tiles) == streams
    rng = np.random.default_rng(n)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    g = (rng.normal(size=(n, V)) * np.where(np.arange(n) % 2, 2.0 ** 20, 2.0 ** small)[:, None]).astype(np.float32)
    w_lm = rng.normal(size=(V, H)).astype(np.float32)
    m, w = min(n, H), dev(np.zeros((H, H)))
    KO.MedusaHeadTrainer([w], dev(w_lm)).step(dev(np.eye(n, H)), dev(g), 2.0)
    got, want = -w.T[:m].double().cpu().numpy(), (g.astype(np.float64) @ w_lm.astype(np.float64))[:m]
    bound = 1.15 * 2.53e-8 * np.sqrt((V + 1) / 2)
    off = np.linalg.norm(got - want, axis=1)
    assert (off <= bound * np.linalg.norm(want, axis=1) + np.sqrt(H) * (splits / 2 + 1) * 2.0 ** -149).all()


@pytest.mark.parametrize("n,V,H,streams", [(20, 4099, 1001, True), (200, 5056, 1024, True), (20, 300, 64, False), (100, 300, 130, False)])
@pytest.mark.parametrize("gv,wv", [(1.998, 0.9999 * 2.0 ** 127), (1.3 * 2.0 ** 60, 1.7 * 2.0 ** 50), (1.3 * 2.0 ** 110, 1.7 * 2.0 ** -60)])
def test_input_gradients_near_overflow(n, V, H, streams, gv, wv):
    """A product of 0.998 of the largest float, whose first pieces alone, rounded up, are past it, and products and factors that
    would be past it times 2^24"""
    import torch
    import paper_2408_08146_amd as KO
    assert bool(form(n, H, V, True, _room(n, H))[0]) == streams
    g, w_lm = torch.zeros(n, V, device="cuda"), torch.zeros(V, H, device="cuda")
    g[:, V - 2], w_lm[V - 2] = gv, wv
    w = torch.zeros(H, H, device="cuda")
    KO.MedusaHeadTrainer([w], w_lm).step(torch.eye(n, H, device="cuda"), g, 1.0)
    want = g[0, V - 2].double() * w_lm[V - 2, 0].double() / 2   # SiLU'(0)
    m = min(n, H)
    assert ((w.double().T[:m] / -want - 1).abs() <= 2.0 ** -23).all()


@pytest.mark.parametrize("rows,H", [(1, 1), (33, 1), (32, 2), (31, 63), (32, 65), (33, 64), (64, 127), (97, 128), (127, 129), (128, 193), (129, 130),
                                    (160, 191), (256, 66), (257, 515), (20, 1030)])
@pytest.mark.parametrize("scale", [0, -118])
def test_updates_at_the_edges_of_a_tile(rows, H, scale):
    """W = -g^T h, set up and bounded as above: a matrix that a tile of 64 x 128, a wave's 32 columns or a pair of columns does
    not fill, chunks of 32 rows and blocks of 128 that the rows do not fill; scale: where the pieces do not hold.  That bound is
    one for a sample of many sums; each by itself is within (rows + 2) roundings of 2^-24 of its terms' magnitudes."""
    import torch
    import paper_2408_08146_amd as KO
    rng = np.random.default_rng(rows + H)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    g, h = (rng.normal(size=(rows, H)).astype(np.float32) * np.float32(2.0 ** e) for e in (scale, -scale // 2))
    w = dev(np.zeros((H, H)))
    KO.MedusaHeadTrainer([w], dev(2 * np.eye(H))).step(dev(h), dev(g), 1.0)
    g, h = g.astype(np.float64), h.astype(np.float64)
    off = np.abs(-w.double().cpu().numpy() - g.T @ h)
    assert (off <= (rows + 2) * 2.0 ** -24 * (np.abs(g).T @ np.abs(h))).all()
    if H >= 31:
        assert _rel(-w, g.T @ h) < 1.15 * 2.53e-8 * np.sqrt((rows + 1) / 2)


def test_head_with_the_smallest_workspace():
    """A workspace without room for split sums is accepted (one byte less is not) and gives the same results to rounding."""
    import torch
    import paper_2408_08146_amd as KO
    n, H, V, K = 20, 256, 600, 2
    blocks, w_lm, h, g, dev = _head(n, H, V, K, 5)
    slot = (n * H * 4 + 255) // 256 * 256
    need = slot * (2 * K + 4)
    head = KO.MedusaHeadTrainer([dev(b) for b in blocks], dev(w_lm))
    full = torch.zeros(n, V, device="cuda")
    head.forward(dev(h), full)
    head._workspace = lambda rows: small
    small = torch.empty(need, dtype=torch.uint8, device="cuda")
    d = torch.zeros(n, V, device="cuda")
    head.forward(dev(h), d)
    head.step(dev(h), dev(g), 0.1)
    logits, grads = _head_ref(blocks, w_lm, h, g, 0.1)
    assert _rel(d, logits) < TOL and _rel(full, logits) < TOL
    for k in range(K):
        upd = head.blocks[k].double().cpu().numpy() - blocks[k]
        assert np.linalg.norm(upd + 0.1 * grads[k]) < 1e-3 * np.linalg.norm(0.1 * grads[k])
    small = torch.empty(need - 1, dtype=torch.uint8, device="cuda")
    with pytest.raises(KO.KoalaError):
        head.forward(dev(h), d)


def test_head_results_do_not_depend_on_earlier_calls():
    """The binding keeps its largest workspace: the same rows give the same bits before and after a call of many rows."""
    import torch
    import paper_2408_08146_amd as KO
    n, H, V = 20, 512, 4096
    blocks, w_lm, h, g, dev = _head(n, H, V, 1, 11)
    block = dev(blocks[0])
    head = KO.MedusaHeadTrainer([block], dev(w_lm))
    results = []
    for many in (False, True):
        if many:
            head.forward(torch.zeros(300, H, device="cuda"), torch.zeros(300, V, device="cuda"))
        block.copy_(dev(blocks[0]))
        d = torch.zeros(n, V, device="cuda")
        head.forward(dev(h), d)
        head.step(dev(h), dev(g), 0.5)
        results.append((d, block.clone()))
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])


@pytest.mark.parametrize("n,H,V,DH,n_fc", [(1, 64, 100, 0, 1), (16, 33, 1030, 40, 2), (17, 256, 2000, 64, 3), (65, 300, 700, 129, 3)])
def test_discriminator_products(n, H, V, DH, n_fc):
    _discriminator_products(n, H, V, DH, n_fc)


@pytest.mark.parametrize("n,H,V,DH,n_fc", [(20, 300, 16387, 40, 2), (64, 300, 16387, 0, 1), (40, 300, 16387, 33, 3)])
def test_logits_joined_to_a_streamed_product(n, H, V, DH, n_fc):
    """The mapped hidden state streamed in one split, so that the product itself adds both sets of logits, in rows whose length is
    no multiple of four"""
    assert form(n, V, H, False, 2 * n * V) == (max(2, -(-n // 16)), 1)
    _discriminator_products(n, H, V, DH, n_fc)


def _discriminator_products(n, H, V, DH, n_fc):
    import torch
    import paper_2408_08146_amd as KO
    from oracle import train as T
    rng = np.random.default_rng(n)
    theta = T.disc_params(rng, H, V, max(DH, 1), n_fc, std=0.05)
    r32 = lambda a: a.astype(np.float32).astype(np.float64)
    theta = dict(w_lin=r32(theta["w_lin"]), w_fc=[r32(w) for w in theta["w_fc"]], b_fc=[r32(b) for b in theta["b_fc"]])
    h, q = r32(rng.normal(size=(n, H))), r32(rng.normal(size=(n, V)))
    d = r32(q + rng.normal(size=(n, V)))
    loss_ref, _, grads = T.disc_step(theta, h, q, d, 0.3)
    dev = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    w_lin, w_fc, b_fc = dev(theta["w_lin"]), [dev(w) for w in theta["w_fc"]], [dev(b) for b in theta["b_fc"]]
    D = KO.Discriminator(w_lin, w_fc, b_fc, fc_hidden=DH)
    loss = torch.zeros(1, device="cuda")
    D.step(dev(h), dev(q), dev(d), 0.3, loss)
    assert abs(loss.item() - loss_ref) < 1e-5 * abs(loss_ref)
    for got, old, g in [(w_lin, theta["w_lin"], grads["w_lin"])] + list(zip(w_fc, theta["w_fc"], grads["w_fc"])):
        upd = got.double().cpu().numpy() - old
        floor = 2.0 ** -24 * np.linalg.norm(old)
        # the gradient passes through up to four products and a sigmoid of a sum over V terms
        assert np.linalg.norm(upd + 0.3 * g) < 3e-5 * np.linalg.norm(0.3 * g) + floor


def test_infinite_operand_stays_infinite():
    """One logit of minus infinity times a negative weight switches the only unit to +inf, whose negative score weight makes
    the draft row's score -inf and its loss zero; a not-a-number on the way would give the loss of a silent unit."""
    import torch
    import paper_2408_08146_amd as KO
    n, H, V = 4, 32, 96
    z = lambda *s: torch.zeros(*s, device="cuda")
    w_fc = [z(1, V), torch.full((1, 1), -1.0, device="cuda")]
    w_fc[0][0, 5] = -2.0
    w_fc[0][0, :5] = 0.25
    d = z(n, V)
    d[:, 5] = float("-inf")
    D = KO.Discriminator(z(V, H), w_fc, [z(1), z(1)], fc_hidden=1)
    loss = z(1)
    # the zero weights beside column 5 meet finite logits only; target rows: score 0, loss log 2
    D.step(z(n, H), z(n, V), d, 0.0, loss)
    assert abs(loss.item() - np.log(2.0)) < 1e-6


@pytest.mark.parametrize("H,rows", [(1, 3), (63, 8), (65, 9), (127, 16), (127, 17), (128, 24), (129, 31), (257, 32), (257, 33), (515, 48),
                                    (1030, 128), (1030, 129)])
def test_update_by_few_rows(H, rows):
    """-g^T h on both sides of the 32 rows up to which an update takes its operands in one piece and of the 128 that others take at
    a time, at widths around its tiles of 64 and 128 and with columns of a wave left over, at the error of an fp32 chain: on
    average as above, and every element within rows * 2^-24 of the sum of its terms' magnitudes (a single element has no
    average)."""
    import torch
    import paper_2408_08146_amd as KO
    gen = torch.Generator(device="cuda").manual_seed(H + rows)
    h, g = (torch.randn(rows, H, generator=gen, device="cuda") for _ in range(2))
    w = torch.zeros(H, H, device="cuda")
    KO.MedusaHeadTrainer([w], 2 * torch.eye(H, device="cuda")).step(h, g, 1.0)
    want = g.double().T @ h.double()
    assert ((w.double() + want).abs() <= rows * 2.0 ** -24 * (g.double().abs().T @ h.double().abs())).all()
    assert H == 1 or ((w.double() + want).norm() / want.norm()).item() < 1.2 * 2.53e-8 * np.sqrt((rows + 1) / 2)


@pytest.mark.parametrize("n", [1, 37, 70, 200])
@pytest.mark.parametrize("form", ["forward", "input_gradient", "update"])
def test_infinities_in_every_form(form, n):
    """One infinite element where the other operand is positive: its row or column of the result is infinite and the rest, the
    tile beside it too, is what it would be without (TOL: those sums are fp32 chains of up to 200 terms, 2.5e-7)."""
    import torch
    import paper_2408_08146_amd as KO
    rng = np.random.default_rng(n)
    V, H, v0, j0 = 70, 130, 41, 67
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    h, w_lm, g = (np.abs(rng.normal(size=s)).astype(np.float32) for s in ((n, H), (V, H), (n, V)))
    w_lm *= np.where(rng.random(w_lm.shape) < 0.5, -1, 1)
    w = dev(np.zeros((H, H)))
    if form == "forward":            # d[:, v0] = +inf
        want = h.astype(np.float64) @ w_lm.T
        w_lm[v0, j0] = np.inf
        got, where = torch.zeros(n, V, device="cuda"), (slice(None), v0)
        KO.MedusaHeadTrainer([w], dev(w_lm)).forward(dev(h), got)
    else:                            # the gradient at unit j0 is +inf, so its row of the update -inf
        if form == "update":         # through an input gradient of one infinite and one zero-free factor
            w_lm, g = np.abs(w_lm[:1]), g[:, :1]
            w_lm[0, j0] = np.inf
            gx = g.astype(np.float64) * np.where(np.isinf(w_lm), 0, w_lm)
        else:
            gx = g.astype(np.float64) @ w_lm
            w_lm[v0, j0] = np.inf
        want, where = -(gx / 2).T @ h.astype(np.float64), (j0, slice(None))
        KO.MedusaHeadTrainer([w], dev(w_lm)).step(dev(h), dev(g), 1.0)
        got = w
    got = got.double().cpu().numpy()
    assert np.isinf(got[where]).all() and (np.sign(got[where]) == (1 if form == "forward" else -1)).all()
    got[where] = want[where] = 0.0
    assert np.linalg.norm(got - want) < TOL * np.linalg.norm(want)


def _one_layer(n, H, V, w, bias, h, q, d, w_lin, lr):
    """One discriminator step with a single layer: the new w_lin, and float64's change of it per lr"""
    import torch
    import paper_2408_08146_amd as KO
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    out, loss = dev(w_lin), torch.zeros(1, device="cuda")
    KO.Discriminator(out, [dev(w[None])], [dev(np.array([bias]))]).step(dev(h), dev(q), dev(d), lr, loss)
    h, q, d, w, w_lin = (a.astype(np.float64) for a in (h, q, d, w, w_lin))
    with np.errstate(all="ignore"):
        z = h @ w_lin.T
        sd, sq = (z + d) @ w + bias, (z + q) @ w + bias
        ds = (1 / (1 + np.exp(-sd)) - 1 / (1 + np.exp(sq))) / n
    return out.double().cpu().numpy(), ds, w, h


@pytest.mark.parametrize("rows,H", [(1, 1), (1, 255), (7, 256), (8, 257), (8, 2896), (8, 2897), (9, 130), (15, 1030), (16, 1619), (16, 1620),
                                    (17, 1000), (24, 515)])
def test_update_of_a_small_or_large_matrix(rows, H):
    """-g^T h on both sides of the sizes up to which an update by 8 and 16 rows is plain multiply-adds, with columns of a wave of
    256 and rows of a panel left over: every element within rows roundings of 2^-24 of its terms' magnitudes."""
    import torch
    import paper_2408_08146_amd as KO
    gen = torch.Generator(device="cuda").manual_seed(H + rows)
    h, g = (torch.randn(rows, H, generator=gen, device="cuda") for _ in range(2))
    old = torch.randn(H, H, generator=gen, device="cuda").round()
    w = old.clone()
    KO.MedusaHeadTrainer([w], 2 * torch.eye(H, device="cuda")).step(h * 0, g, 1.0)   # zero terms leave what was there
    assert torch.equal(w, old)
    w.zero_()
    KO.MedusaHeadTrainer([w], 2 * torch.eye(H, device="cuda")).step(h, g, 1.0)
    want = g.double().T @ h.double()
    assert ((w.double() + want).abs() <= (1 + 2.0 ** -6) * rows * 2.0 ** -24 * (g.double().abs().T @ h.double().abs())).all()


@pytest.mark.parametrize("n,H,V,DH,n_fc", [(1, 5, 3, 2, 3), (3, 70, 130, 1, 2), (4, 130, 1030, 130, 3), (8, 33, 513, 17, 3), (12, 33, 513, 16, 2),
                                           (13, 33, 513, 0, 1), (25, 33, 513, 0, 1)])
def test_discriminator_updates_of_small_matrices(n, H, V, DH, n_fc):
    """Weights, biases and the mapping's two gradients in multiply-adds: matrices of one row and of few, up to 8, 16 and 24 rows
    and, with both halves of the logits, twice the positions"""
    _discriminator_products(n, H, V, DH, n_fc)


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
@pytest.mark.parametrize("H", [4100])
def test_update_by_few_rows_to_the_last_bit(H, rows):
    """A chain of fp32 multiply-adds rounds each term and each sum of several once: every element within rows roundings of 2^-24
    of its terms' magnitudes (the matrix pipe, which cuts off what its sums do not hold, would need three at two rows).  2^-6 of
    that on top: products of pieces are added among themselves first, at 2^-8 of the whole.  In the 2-norm a chain's rounding of
    a single term, 2.53e-8, and that times the root of 1.5 at two rows, which are such a chain; less than a chain's beyond."""
    import torch
    import paper_2408_08146_amd as KO
    gen = torch.Generator(device="cuda").manual_seed(H + rows)
    h, g = (torch.randn(rows, H, generator=gen, device="cuda") for _ in range(2))
    w = torch.zeros(H, H, device="cuda")
    KO.MedusaHeadTrainer([w], 2 * torch.eye(H, device="cuda")).step(h, g, 1.0)
    want = g.double().T @ h.double()
    off = (w.double() + want).abs()
    assert (off <= (1 + 2.0 ** -6) * rows * 2.0 ** -24 * (g.double().abs().T @ h.double().abs())).all()
    assert (off.norm() / want.norm()).item() < 2.56e-8 * (1.0, 1.5 ** 0.5, 1.05, 1.07)[rows - 1]


@pytest.mark.parametrize("n", [1, 4, 20, 32, 40])
@pytest.mark.parametrize("small", [-112, -140])
def test_update_by_few_rows_of_small_beside_large_values(n, small):
    """Every second gradient and every third hidden state in units of 2^small, beside others in the same tile that are 2^40 and 2^30:
    elements are no less exact for it, also where a factor is below the smallest normal float.  Within (n + 10) roundings of the
    terms' magnitudes as below (weights too small to be normal floats are rounded by their sigmoids' factors at 2^-149: twelve
    times that)."""
    H, V = 4200, 4100   # more than 2^23 elements: the matrix pipe's form
    rng = np.random.default_rng(n)
    w = (rng.normal(size=V) * np.where(np.arange(V) % 2, 2.0 ** 40, 2.0 ** small)).astype(np.float32)
    h = (rng.normal(size=(n, H)) * np.where(np.arange(H) % 3, 2.0 ** 30, 2.0 ** small)).astype(np.float32)
    zero = np.zeros((n, V), np.float32)
    got, ds, w, h = _one_layer(n, H, V, w, np.float32(2.0), h, zero, zero, np.zeros((V, H), np.float32), 1.0)
    want = -w[:, None] * (ds @ h)
    rounded = (n + 10) * 2.0 ** -24 * np.abs(w)[:, None] * (np.abs(ds) @ np.abs(h)) + 12 * 2.0 ** -149 * (1 + np.abs(h).sum(0))
    assert (np.abs(got - want) <= rounded).all()


@pytest.mark.parametrize("rows", [1, 20, 32, 33, 48, 49, 100])
@pytest.mark.parametrize("gv,hv", [(1.998, 0.9999 * 2.0 ** 127), (1.3 * 2.0 ** 60, 1.7 * 2.0 ** 40), (1.3 * 2.0 ** 110, 1.7 * 2.0 ** -60)])
def test_update_near_overflow(rows, gv, hv):
    """Products of 0.998 of the largest float, whose first pieces alone, rounded up, are past it; products and factors that are
    not near it but would be past it times 2^48 and 2^24"""
    import torch
    import paper_2408_08146_amd as KO
    H = 200
    g, h = torch.zeros(rows, H, device="cuda"), torch.zeros(rows, H, device="cuda")
    g[-1], h[-1] = gv, hv
    w = torch.zeros(H, H, device="cuda")
    KO.MedusaHeadTrainer([w], 2 * torch.eye(H, device="cuda")).step(h, g, 1.0)
    want = -g[-1, 0].double() * h[-1, 0].double()
    assert ((w.double() / want - 1).abs() <= 2.0 ** -23).all()


@pytest.mark.parametrize("n", [1, 20, 32, 33])
def test_two_halves_of_a_gradient_where_pieces_do_not_hold(n):
    """Up to 32 positions the update of the mapping adds the draft's and the target's gradients itself.  Weights in units of 2^-112
    make gradients around 2^-118, where low bits are below the smallest normal bfloat16 but nothing is below the smallest normal
    float (a bias keeps the halves from cancelling); the hidden states in units of 2^60.  Each element within (n + 10) roundings
    of its terms' magnitudes: n + 2 as for other updates, eight for two sigmoids and their factors."""
    H, V, bias = 130, 70, np.float32(2.0)
    rng = np.random.default_rng(n)
    w = rng.normal(size=V).astype(np.float32) * np.float32(2.0 ** -112)
    h = rng.normal(size=(n, H)).astype(np.float32) * np.float32(2.0 ** 60)
    zero = np.zeros((n, V), np.float32)
    got, ds, w, h = _one_layer(n, H, V, w, bias, h, zero, zero, np.zeros((V, H), np.float32), 1.0)
    want = -w[:, None] * (ds @ h)
    assert (np.abs(got - want) <= (n + 10) * 2.0 ** -24 * np.abs(w)[:, None] * (np.abs(ds) @ np.abs(h))).all()


@pytest.mark.parametrize("n", [2, 20, 32, 33])
def test_two_halves_of_a_gradient_and_an_infinite_hidden_state(n):
    """One infinite element of h: the draft's row has a gradient (1 / n), the target's, whose score is infinite as well, none.
    That unit's column of the mapping goes to minus infinity, the rest is as without it."""
    H, V, j0 = 130, 70, 67
    rng = np.random.default_rng(n)
    pos = lambda *s: (np.abs(rng.normal(size=s)) + 0.1).astype(np.float32)
    h, w, w_lin = pos(n, H) * np.float32(0.05), pos(V) * np.float32(0.1), pos(V, H) * np.float32(0.1)
    q, d = (rng.normal(size=(n, V)).astype(np.float32) for _ in range(2))
    h[1, j0] = np.inf
    got, ds, w, h = _one_layer(n, H, V, w, np.float32(-2.0), h, q, d, w_lin, 1.0)
    assert ds[1] == 1.0 / n and (got[:, j0] == -np.inf).all()
    keep = np.arange(H) != j0
    change = -w[:, None] * (ds @ h[:, keep])
    off = np.abs(got[:, keep] - w_lin[:, keep] - change)
    # 2^-24 of the stored weight, and of the change 3e-6: a sum over 70 x 130 terms behind a sigmoid
    assert np.isfinite(got[:, keep]).all()
    assert (off <= 2.0 ** -24 * np.abs(got[:, keep]) + 3e-6 * np.abs(w)[:, None] * (np.abs(ds) @ h[:, keep])).all()


@pytest.mark.parametrize("V", [1, 1023, 1025, 32768, 33001])
def test_distillation_rows_of_every_length(V):
    import torch
    import paper_2408_08146_amd as KO
    n, H = 3, 8
    g = torch.Generator(device="cuda").manual_seed(V)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, d = rnd(n, V) * 3, rnd(n, V) * 3
    D = KO.Discriminator(rnd(V, H), [rnd(1, V)], [rnd(1)])
    loss, grad = torch.zeros(2, device="cuda"), torch.full((n, V), 7.0, device="cuda")
    D.gen_grad(rnd(n, H), q, d, 0.0, loss, grad)
    p, s = torch.softmax(q.double(), -1), torch.log_softmax(d.double(), -1)
    assert abs(loss[1].item() + (p * s).sum(-1).mean().item()) < 2e-6 * (1 + abs(loss[1].item()))
    assert (grad.double() - (s.exp() - p) / n).abs().max().item() < 1e-6


def _change_error(new, old, want):
    """Of a parameter's change against float64's, less what storing the parameter in fp32 rounds away (2^-24 / sqrt(12) of each
    parameter root mean square, three times that at the most over so many)."""
    err = (new.double() - old.double() - want).norm().item()
    return max(0.0, err - 3 * 2.0 ** -24 / 12 ** 0.5 * old.double().norm().item()) / want.norm().item()


def test_updates_at_the_benchmarked_size():
    """One step of each kind at 4096 x 32000 with a learning rate of 1e-3, where a whole update is 1e-4 of the parameters and
    less: the change itself is compared, so that a missing, wrong or partial one shows.  1e-3 of it: the gradients pass
    through five products and, in the discriminator, units within rounding of zero may switch."""
    import torch
    import paper_2408_08146_amd as KO
    H, V, W, lr = 4096, 32000, 1024, 1e-3
    g = torch.Generator(device="cuda").manual_seed(17)
    rnd = lambda *s, scale=1.0: torch.randn(*s, generator=g, device="cuda") * scale
    blocks, w_lm, h, grad = [rnd(H, H, scale=0.02) for _ in range(2)], rnd(V, H, scale=0.02), rnd(128, H), rnd(128, V, scale=1e-4)
    p = [b.double().requires_grad_() for b in blocks]
    x = h.double()
    for w in p:
        x = x + torch.nn.functional.silu(x @ w.T)
    x.backward((grad.double() @ w_lm.double()))
    new = [b.clone() for b in blocks]
    KO.MedusaHeadTrainer(new, w_lm).step(h, grad, lr)
    for k in range(2):
        assert _change_error(new[k], blocks[k], -lr * p[k].grad) < 1e-3, k
    del x, p, w_lm
    h, q = h[:20].contiguous(), rnd(20, V, scale=2.0)
    d = q + rnd(20, V)
    old = [rnd(V, H, scale=0.02), rnd(W, V, scale=0.02), rnd(1, W, scale=0.02), rnd(W, scale=30.0), rnd(1, scale=0.02)]
    p = [t.double().requires_grad_() for t in old]
    def score(logits):
        a = torch.relu((h.double() @ p[0].T + logits.double()) @ p[1].T + p[3])
        return (a @ p[2].T + p[4])[:, 0]
    (torch.nn.functional.softplus(score(d)).mean() + torch.nn.functional.softplus(-score(q)).mean()).backward()
    new = [t.clone() for t in old]
    KO.Discriminator(new[0], [new[1], new[2]], [new[3], new[4]], fc_hidden=W).step(h, q, d, lr, torch.zeros(1, device="cuda"))
    for k in range(5):
        assert _change_error(new[k], old[k], -lr * p[k].grad) < 1e-3, k
