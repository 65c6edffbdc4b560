"""Prediction over all output neurons (slide_predict mode 1) against the oracle, and the
prediction-quality loop on a task with planted structure: the hashed retrieval must find what the
dense evaluation finds."""
import numpy as np
import pytest

from paper_2201_12667_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from helpers import (FLOOR, REL, make_oracle, make_pair, planted_batch, planted_prototypes,  # noqa: E402
                     planted_workload)


def _say(*a):
    print(*a, flush=True)


def _dense_scores(orc, batch):
    """All N scores per sample in double precision, from the oracle's parameters."""
    h = orc.forward_hidden(batch).astype(np.float64)
    return h @ orc.p["W2"].astype(np.float64).T + orc.p["b2"].astype(np.float64)


def _check_topk(ids, sc, z, topk):
    """ids/sc [B][topk] from the GPU against the full score matrix z [B][N] of the oracle: the
    scores agree to the fp32 bar, every reported id carries the score reported for it, the list is
    the oracle's top-k up to the order of scores that differ by less than the bar, ties to the
    lower id are honoured where the oracle's scores are exactly equal, and the tail is padded."""
    B, N = z.shape
    k = min(topk, N)
    order = np.lexsort((np.broadcast_to(np.arange(N), z.shape), -z), axis=1)[:, :k]
    want = np.take_along_axis(z, order, axis=1)
    tol = REL * np.abs(want) + FLOOR * np.abs(z).max()
    assert np.all(ids[:, k:] == -1) and np.all(np.isneginf(sc[:, k:]))
    got_ids = ids[:, :k]
    assert got_ids.min() >= 0 and got_ids.max() < N
    assert all(len(set(r.tolist())) == k for r in got_ids)
    assert np.all(np.abs(sc[:, :k] - want) <= tol)                       # r-th best score
    assert np.all(np.abs(np.take_along_axis(z, got_ids, axis=1) - want) <= 2 * tol)   # carried by the reported id
    exact = float((got_ids == order).mean())
    return exact


@pytest.mark.parametrize("name,wl,topk", [
    ("dwta-small", synth.small(synth.HASH_DWTA), 5),
    ("dense-hidden-h200", synth.small(synth.HASH_DWTA, input_dim=0, hidden_dim=200, K=3, L=5, batch=70,
                                      num_classes=9973), 64),
    ("h1024-b130", synth.small(synth.HASH_DWTA, hidden_dim=1024, K=4, L=5, batch=130, num_classes=7001,
                               input_dim=2500, bucket_cap=64), 10),
    ("fewer-neurons-than-k", synth.small(synth.HASH_SIMHASH, hidden_dim=32, K=3, L=3, batch=9, num_classes=50,
                                         input_dim=100, nnz_mean=5.0, lab_mean=1.0), 64),
    # 2048 samples: eight row blocks of samples
    ("b2048", synth.small(synth.HASH_SIMHASH, hidden_dim=32, K=5, L=4, batch=2048, num_classes=20011,
                                       input_dim=0, bucket_cap=8), 7),
    ("h4", synth.small(synth.HASH_SIMHASH, hidden_dim=4, K=2, L=3, batch=3, num_classes=700,
                       input_dim=60, nnz_mean=4.0), 3),
])
def test_predict_over_all_neurons_matches_oracle(name, wl, topk):
    _say("dense predict", name)
    gen, model, orc = make_pair(wl)
    model.build_tables()
    b = gen.batch(0)
    ids, sc = model.predict(model.to_device(b), topk, mode=1)
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    exact = _check_topk(ids, sc, _dense_scores(orc, b), topk)
    _say("   positions identical to the oracle's order:", round(exact, 4))
    assert exact > 0.98
    want_ids, _ = orc.predict(b, topk, 1)
    assert float((ids == want_ids).mean()) > 0.98
    assert model.status() == 0
    model.destroy()


@pytest.mark.parametrize("slope", [0.01, -0.01])
def test_predict_when_every_or_no_later_neuron_beats_the_list(slope):
    """Scores that follow the neuron id: biases that grow with it put the whole list at the end of the layer, behind most
    of the sampled neurons, biases that fall with it at its start.  (One pass over the layer; several:
    test_predict_all_in_chunks.)"""
    _say("dense predict, bias slope", slope)
    wl = synth.small(synth.HASH_DWTA, num_classes=20011, batch=33)
    gen, model, orc = make_pair(wl)
    bias = (slope * np.arange(wl.num_classes)).astype(np.float32)
    orc.p["b2"][:] = bias
    model.p["b2"].copy_(torch.from_numpy(bias))
    model.build_tables()
    b = gen.batch(0)
    for topk in (1, 64):
        ids, sc = model.predict(model.to_device(b), topk, mode=1)
        ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
        exact = _check_topk(ids, sc, _dense_scores(orc, b), topk)
        _say("   topk", topk, "positions identical to the oracle's order:", round(exact, 4))
        assert exact > 0.9
        lo, hi = (wl.num_classes - 200, wl.num_classes) if slope > 0 else (0, 200)
        assert ids.min() >= lo and ids.max() < hi
    assert model.status() == 0
    model.destroy()


@pytest.mark.parametrize("N,H,batch", [(16384, 16, 33), (16640, 32, 32), (40009, 36, 65), (40009, 128, 129),
                                       (33001, 272, 40), (30011, 264, 200)])
def test_predict_all_when_the_sampled_neurons_mislead(N, H, batch):
    """The bar of the dense pass comes from every (N // 8192)-th neuron: here those are the worst of the layer,
    so that nearly every other neuron reaches the bar (more than a sample's candidate buffer holds for the
    larger N: that sample evaluates the layer itself), and a few neurons carry weights that are no ordinary numbers
    (infinite, or so large that their bf16 part is).  Row blocks, staged and resident h, ragged coordinates."""
    _say("misleading sample", N, H, batch)
    wl = synth.small(synth.HASH_SIMHASH, input_dim=0, hidden_dim=H, K=3, L=3, num_classes=N, batch=batch, bucket_cap=8)
    gen, model, orc = make_pair(wl)
    rng = np.random.default_rng(1)
    bias = (rng.standard_normal(N) * 0.01).astype(np.float32)
    bias[np.arange(N) % (N // 8192) != 0] += 10
    W2 = orc.p["W2"].copy()
    W2[N - 1, H - 1] = np.inf
    W2[7, 0] = -np.inf
    W2[N // 2, :4] = 3.4e38 * np.array([1, -1, 1, 0], np.float32)
    model.p["W2"].copy_(torch.from_numpy(W2))
    model.p["b2"].copy_(torch.from_numpy(bias))
    model.build_tables()
    b = gen.batch(0)
    b["hidden"][:, [0, H - 1]] = 0.5
    b["hidden"][:, 1:3] = 0.25
    for topk in (2, 64):
        ids, sc = (x.cpu().numpy() for x in model.predict(model.to_device(b), topk, mode=1))
        assert np.all(ids[:, 0] == N - 1) and np.all(np.isposinf(sc[:, 0]))
        assert np.all(ids[:, 1] == N // 2) and np.allclose(sc[:, 1], 1.7e38, rtol=1e-5)
        keep = np.ones(N, bool)
        keep[[N - 1, 7, N // 2]] = False
        z = b["hidden"].astype(np.float64) @ W2[keep].astype(np.float64).T + bias[keep].astype(np.float64)
        if topk > 2:
            back = np.cumsum(keep) - 1
            assert _check_topk(back[ids[:, 2:]], sc[:, 2:], z, topk - 2) > 0.97
    model.destroy()


@pytest.mark.parametrize("batch", [64, 65, 128, 129, 256, 257])
@pytest.mark.parametrize("H", [16, 124, 160, 164])
def test_predict_all_row_blocks(batch, H):
    """Edges of the row blocks, resident and staged activations, against 64-bit scores: the lists are the best by those
    up to near-ties, the scores within the six bf16 products' error (2e-6 of the largest is ten times what 1,024
    coordinates show)."""
    _row_blocks(17003, batch, H)


# around one tile of neurons and two rounds of them for every workgroup of a machine of 256 compute units
@pytest.mark.parametrize("N,batch,H", [(65003, 65, 128), (70003, 65, 128), (65003, 128, 96), (40003, 128, 64), (65003, 129, 128),
                                       (70003, 129, 128), (65003, 192, 64), (65003, 193, 64), (132003, 130, 128), (65003, 160, 112)])
def test_predict_all_row_blocks_of_few_tiles(N, batch, H):
    _row_blocks(N, batch, H)


# up to 32 samples and whole lines of W2: a stretch of neurons for every wave (at the size from which that is taken and one
# short of it, a last stretch that is short or missing, an odd number of coordinate blocks), and rows that are no whole lines
@pytest.mark.parametrize("N,batch,H", [(131071, 5, 32), (131072, 32, 32), (131072, 1, 96), (139001, 31, 160), (155649, 7, 256),
                                       (131072 + 4097, 32, 64), (140003, 9, 40)])
def test_predict_all_row_blocks_of_streamed_layers(N, batch, H):
    _row_blocks(N, batch, H)


def _row_blocks(N, batch, H):
    _say("dense predict blocks", N, batch, H)
    topk = 7
    wl = synth.small(synth.HASH_SIMHASH, input_dim=0, hidden_dim=H, K=3, L=3, num_classes=N, batch=batch, bucket_cap=8)
    gen, model, orc = make_pair(wl)
    model.build_tables()
    host = gen.batch(0)
    ids, scores = model.predict(model.to_device(host), topk, 1)
    z = host["hidden"].astype(np.float64) @ orc.p["W2"].astype(np.float64).T + orc.p["b2"].astype(np.float64)
    want = -np.sort(-z, axis=1)[:, :topk]
    ids, scores = ids.cpu().numpy(), scores.cpu().numpy()
    bar = 2e-6 * np.abs(z).max()
    assert np.abs(scores - want).max() <= bar
    assert np.abs(np.take_along_axis(z, ids.astype(np.int64), 1) - scores).max() <= bar
    assert all(len(set(r)) == topk for r in ids.tolist())
    model.destroy()


@pytest.mark.parametrize("batch,H", [(8, 32), (8, 40), (40, 32), (100, 32)])
@pytest.mark.parametrize("layout", ["falls", "falls-roughly", "log"])
def test_predict_all_costs_the_same_in_any_order_of_the_ids(layout, batch, H):
    """Scores that follow the neuron id, as where ids go by frequency: as few neurons as in random order reach the bar, so
    the call takes about as long.  (Where more reach it than a sample's candidate buffer holds, that sample reads the
    layer by itself, tens of milliseconds for a call of a tenth of one.)  The scores are the biases, the lists exact."""
    N = 670_091
    ids, rng = np.arange(N), np.random.default_rng(2)
    bias = {"falls": -1e-3 * ids, "falls-roughly": -1e-3 * ids + 0.02 * 1e-3 * N * rng.standard_normal(N),
            "log": -np.log(ids + 10) + 0.3 * rng.standard_normal(N)}[layout].astype(np.float32)
    _cost_of_scores("order " + layout, N, batch, H, bias)


@pytest.mark.parametrize("batch,H", [(8, 32), (8, 40), (100, 32)])
@pytest.mark.parametrize("layout", ["equal", "untouched", "two-values", "ten-values"])
def test_predict_all_costs_the_same_with_tied_scores(layout, batch, H):
    """Scores that many neurons share, as before training or for a sample whose activations are zero: ties go to the lower
    id, and of a tie at the bar only the lower ids pass it."""
    N = 670_091
    rng = np.random.default_rng(4)
    bias = np.zeros(N, np.float32)
    if layout == "untouched":
        bias[rng.integers(0, N, 5000)] = -1e-3 * rng.random(5000)
    elif layout == "two-values":
        bias[:] = rng.integers(0, 2, N)
    elif layout == "ten-values":
        bias[:] = rng.integers(0, 10, N)
    _cost_of_scores("ties " + layout, N, batch, H, bias)


def _cost_of_scores(name, N, batch, H, bias):
    """Lists and time of a prediction whose scores are the biases (W2 = 0), against the same scores in random order."""
    _say("dense predict cost", name, N, batch, H)
    wl = synth.small(synth.HASH_SIMHASH, input_dim=0, hidden_dim=H, K=3, L=3, num_classes=N, batch=batch, bucket_cap=8)
    gen, model, _ = make_pair(wl)
    model.p["W2"].zero_()
    model.build_tables()
    db = model.to_device(gen.batch(0))

    def timed(scores, topk):
        model.p["b2"].copy_(torch.from_numpy(scores))
        ms = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            got, sc = model.predict(db, topk, mode=1)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        want = np.lexsort((np.arange(N), -scores))[:topk]
        assert np.array_equal(got.cpu().numpy(), np.broadcast_to(want, got.shape))
        assert np.array_equal(sc.cpu().numpy(), np.broadcast_to(scores[want], sc.shape))
        return sorted(ms)[3]
    for topk in (10, 32):
        spread = timed(np.random.default_rng(3).standard_normal(N).astype(np.float32), topk)
        here = timed(bias, topk)
        _say("   topk", topk, "us: %.0f in random order, %.0f so" % (1e3 * spread, 1e3 * here))
        assert here < 5 * spread + 0.5                     # (an overflowing sample: 15 ms)
    model.destroy()


@pytest.mark.parametrize("layout", ["random", "second", "first", "second-misleads"])
def test_predict_all_in_chunks(layout):
    """A layer so large that the 64 best take two passes over it (1.2 M neurons each): the list of the first and its bar go
    on into the second.  Random scores; the second pass holds all winners; the first does; the second holds a
    quarter of a million neurons that reach the bar, because the sampled ones are the worst there, more than a
    sample's candidate buffer."""
    N, topk, batch = 1_500_007, 64, 5
    stride = N // 8192
    ns = -(-N // stride)
    most = int(ns * 16384 / (topk + 4 * topk ** 0.5 + 16)) // 256 * 256
    assert N // 2 < most < N
    _say("chunks", layout, most)
    wl = synth.small(synth.HASH_SIMHASH, input_dim=0, hidden_dim=16, K=3, L=3, num_classes=N, batch=batch, bucket_cap=8)
    gen, model, orc = make_pair(wl)
    ids = np.arange(N)
    bias = (np.random.default_rng(1).standard_normal(N) * 0.01).astype(np.float32)
    if layout == "second":
        bias[most:] += 10
    elif layout == "first":
        bias[:most] += 10
    elif layout == "second-misleads":
        bias[(ids >= most) & (ids % stride != 0)] += 10
    model.p["b2"].copy_(torch.from_numpy(bias))
    model.build_tables()
    b = gen.batch(0)
    z = b["hidden"].astype(np.float64) @ orc.p["W2"].astype(np.float64).T + bias.astype(np.float64)
    db = model.to_device(b)
    for _ in range(2):
        got, sc = (x.cpu().numpy() for x in model.predict(db, topk, mode=1))
        assert _check_topk(got, sc, z, topk) > 0.97
        if layout != "random":
            assert np.all(got < most) if layout == "first" else np.all(got >= most)
    model.destroy()


@pytest.mark.parametrize("batch,H,D", [(1, 32, 0), (33, 16, 300), (70, 128, 0), (129, 32, 0), (200, 136, 300)])
@pytest.mark.parametrize("weights", ["first-row-inf", "first-bias-nan", "first-bias-inf", "all-nan"])
def test_predict_all_writes_nothing_for_rows_past_the_batch(batch, H, D, weights):
    """A batch that fills max_batch but not its row block, and a neuron 0 (or a whole layer, as after divergence) whose
    score is no number for the zeros that fill the block: those rows have no candidate buffer, and the ones of the
    batch lose nothing.  The first sample's candidates and the activations that lie behind the scratch are whole."""
    _say("rows past the batch", batch, H, D, weights)
    wl = synth.small(synth.HASH_SIMHASH, input_dim=D, hidden_dim=H, K=3, L=3, num_classes=16411, batch=batch, bucket_cap=8,
                     nnz_mean=9.0)
    gen, model, orc = make_pair(wl)
    W2, bias = orc.p["W2"].copy(), orc.p["b2"].copy()
    if weights == "first-row-inf":
        W2[0] = np.inf
    elif weights == "first-bias-nan":
        bias[0] = np.nan
    elif weights == "first-bias-inf":
        bias[0] = np.inf
    else:
        W2[:] = np.nan
    model.p["W2"].copy_(torch.from_numpy(W2))
    model.p["b2"].copy_(torch.from_numpy(bias))
    model.build_tables()
    b = gen.batch(0)
    db = model.to_device(b)
    topk = 5
    ids, sc = (x.cpu().numpy() for x in model.predict(db, topk, mode=1))
    h = orc.forward_hidden(b).astype(np.float64)
    if D:
        assert np.allclose(model.debug_hidden(want_grad=False)[0], h, rtol=1e-6, atol=1e-7)
    assert all(len(set(r.tolist())) == topk and r.min() >= 0 and r.max() < wl.num_classes for r in ids)
    if weights == "all-nan":
        assert np.all(np.isnan(sc)) and np.array_equal(ids, np.broadcast_to(np.arange(topk), ids.shape))
    else:
        # neuron 0 is first or, where its score is a NaN with the sign bit (0 x inf), last; the rest of the layer is in order
        assert not np.any(np.isfinite(sc[ids == 0]))
        z = h @ W2[1:].astype(np.float64).T + bias[1:].astype(np.float64)
        first = ids[:, 0] == 0
        rest = np.where(first[:, None], ids[:, 1:], ids[:, :-1])
        got = np.where(first[:, None], sc[:, 1:], sc[:, :-1])
        assert np.all(rest > 0)
        assert _check_topk(rest - 1, got, z, topk - 1) > 0.97
    assert model.status() == 0
    model.destroy()


@pytest.mark.parametrize("topk", [1, 5])
def test_predict_all_fills_the_list_when_scores_leave_the_range(topk):
    """Scores of minus infinity everywhere but at one sampled neuron, whose sum is the lowest finite number when it is
    rounded after every term and minus infinity when it is not: whichever the kernels find, they have to agree
    on it, or the neuron sets a bar that nothing reaches and the list comes back short."""
    _say("scores out of range", topk)
    N, H, j = 16640, 32, 8000
    wl = synth.small(synth.HASH_SIMHASH, input_dim=0, hidden_dim=H, K=3, L=3, num_classes=N, batch=3, bucket_cap=8)
    gen, model, _ = make_pair(wl)
    W2, bias = np.zeros((N, H), np.float32), np.full(N, -np.inf, np.float32)
    bias[j] = 0
    big = np.float32(2.0 ** 128 * (1 - 2.0 ** -8))                        # the largest bf16 number
    W2[j, 0], W2[j, 1] = -big, np.float32(float(big) - float(np.finfo(np.float32).max))
    W2[j, 2:] = -0.4 * 2.0 ** 104                                         # 0.4 units in the last place of the sum
    model.p["W2"].copy_(torch.from_numpy(W2))
    model.p["b2"].copy_(torch.from_numpy(bias))
    model.build_tables()
    b = gen.batch(0)
    b["hidden"][:] = 1
    ids, sc = (x.cpu().numpy() for x in model.predict(model.to_device(b), topk, mode=1))
    assert ids.min() >= 0 and ids.max() < N and all(len(set(r.tolist())) == topk for r in ids)
    assert np.all(sc <= -np.finfo(np.float32).max) and np.all(np.isneginf(sc[ids != j]))
    model.destroy()


@pytest.mark.parametrize("topk", [1, 33, 64])
@pytest.mark.parametrize("layout", ["spread", "few-threads", "ties", "nan"])
def test_predict_retrieved_selection_edges(layout, topk):
    """The selection among thousands of retrieved neurons: best entries spread over the list; all of them in the
    shares of 63 of the 256 selecting threads (more than one gather holds reach the bar); every score the
    same (ties to the lower id); fewer comparable scores than topk.  The scores are the biases (W2 = 0), so the
    expected lists are exact."""
    _say("selection", layout, topk)
    wl = synth.small(synth.HASH_SIMHASH, input_dim=0, hidden_dim=32, K=1, L=16, num_classes=20011, batch=3,
                     bucket_cap=1024, lab_mean=1.0)
    gen, model, _ = make_pair(wl)
    model.build_tables()
    db = model.to_device(gen.batch(0))
    model.predict(db, topk, mode=0)
    as_ptr, ids, _, _, _ = model.debug_active()
    rng = np.random.default_rng(3)
    bias = rng.standard_normal(wl.num_classes).astype(np.float32)
    mine = ids[as_ptr[0]:as_ptr[1]]
    assert mine.size > 5000
    if layout == "few-threads":
        bias[mine[np.arange(mine.size) % 256 < 63]] += 100
    elif layout == "ties":
        bias[:] = 0
        bias[::2] = -0.0
    elif layout == "nan":
        bias[:] = np.nan
        bias[mine[::mine.size // 20]] = 1.5
        bias[mine[7]] = -np.inf
    model.p["W2"].zero_()
    model.p["b2"].copy_(torch.from_numpy(bias))
    got, sc = (x.cpu().numpy() for x in model.predict(db, topk, mode=0))
    for i in range(wl.batch):
        own = ids[as_ptr[i]:as_ptr[i + 1]]
        own = own[~np.isnan(bias[own])]
        own = own[np.lexsort((own, -bias[own]))][:topk]
        assert np.array_equal(got[i, :own.size], own)
        assert np.array_equal(sc[i, :own.size], bias[own])
        assert np.all(got[i, own.size:] == -1) and np.all(np.isneginf(sc[i, own.size:]))
    model.destroy()


def test_prediction_quality_on_a_planted_task():
    """300 training steps on the GPU, then top-1 over the retrieved set (mode 0) and over all neurons
    (mode 1): both find the planted class, and they agree."""
    wl = planted_workload()
    gen, model, orc = make_pair(wl)
    protos = planted_prototypes(wl)
    model.build_tables()
    first = last = None
    for s in range(300):
        b, _ = planted_batch(wl, protos, s)
        loss = model.train_step(model.to_device(b))
        if s == 0:
            first = float(loss.item())
    last = float(loss.item())
    _say("planted task: loss", first, "->", last)
    assert last < 0.1 < first
    hits = {0: 0, 1: 0}
    agree = total = 0
    for s in range(10_000, 10_004):
        b, labels = planted_batch(wl, protos, s)
        db = model.to_device(b)
        lsh = model.predict(db, 1, mode=0)[0].cpu().numpy()[:, 0]
        dense = model.predict(db, 1, mode=1)[0].cpu().numpy()[:, 0]
        hits[0] += int((lsh == labels).sum())
        hits[1] += int((dense == labels).sum())
        agree += int((lsh == dense).sum())
        total += labels.size
    _say("P@1 retrieved set", hits[0] / total, " P@1 all neurons", hits[1] / total, " agreement", agree / total)
    assert hits[1] / total >= 0.97 and hits[0] / total >= 0.9 and agree / total >= 0.9
    # the dense pass on the trained weights against the oracle evaluated on the same weights
    w = {k: v.cpu().numpy() for k, v in model.p.items()}
    ref = make_oracle(wl, w, gen.hash_params())
    b, _ = planted_batch(wl, protos, 20_000)
    ids, sc = model.predict(model.to_device(b), 5, mode=1)
    assert _check_topk(ids.cpu().numpy(), sc.cpu().numpy(), _dense_scores(ref, b), 5) > 0.98
    model.destroy()
