"""Embedding network, optimiser and learned k-NN on the GPU against the
FP64 oracle (oracle/cnn.py for the network, the TWED oracle for distances).

Tolerances.  The network runs its convolutions on BF16 operands (8
significant bits, relative rounding error at most 2^-9 = 1.95e-3) with FP32
accumulation.  A layer's output is a sum of K = 5 C_in products whose two
operands are each rounded once, so its relative error is about
sqrt(2) * 2^-9 = 2.8e-3 when the rounding errors are independent; four
layers compound to about 5.5e-3, and the segment means do not increase it.
The forward bar is therefore 2e-2 relative (norm over the embeddings, 3.6x
the estimate).  The backward pass rounds the incoming gradients to BF16 as
well and adds ReLU-mask flips where a pre-activation is within rounding of
zero, so gradients are held to 5e-2 relative norm error and cosine >= 0.998
per tensor.  AdamW is plain FP32 arithmetic: 1e-5 relative.  Distances
returned by the k-NN search are FP32 TWED values: 1e-5 relative, the bar of
every FP32 distance in this library.
"""
import os
import sys

import numpy as np
import pytest

import oracle
from oracle import cnn as ocnn
from paper_2007_16135_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2007_16135_amd import binding as B  # noqa: E402
from paper_2007_16135_amd import knn  # noqa: E402


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def threads():
    return min(os.cpu_count() or 1, 16)


def pack(series):
    off = np.zeros(len(series) + 1, dtype=np.int64)
    off[1:] = np.cumsum([len(s) for s in series])
    X = np.concatenate(series).astype(np.float32)
    return X, off


def ragged_series(seed=0):
    """Walks of lengths covering the degenerate segment cases (L < 4), tile
    edges and the workload's range."""
    rng = np.random.default_rng(seed)
    lengths = [1, 2, 3, 4, 5, 7, 13, 63, 64, 65, 100, 129, 300, 512]
    return [np.cumsum(rng.standard_normal(L)).astype(np.float32) for L in lengths]


def random_params(seed):
    p = ocnn.init_params(seed)
    rng = np.random.default_rng(seed + 100)
    for l in range(4):
        p["b"][l] = rng.normal(0, 0.1, p["b"][l].shape)
    vec = ocnn.flatten(p).astype(np.float32)
    return vec, ocnn.unflatten(vec.astype(np.float64))


def rel_norm(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def cosine(a, b):
    a, b = np.asarray(a, np.float64).ravel(), np.asarray(b, np.float64).ravel()
    return float(a @ b / max(np.linalg.norm(a) * np.linalg.norm(b), 1e-300))


def dev(a, dt=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def test_param_count():
    assert B.twed_embed_param_count() == ocnn.n_params()
    assert B.twed_embed_max_length() == 65535


@pytest.mark.parametrize("seed", [0, 1])
def test_forward_matches_oracle(seed):
    series = ragged_series(seed)
    vec, params = random_params(seed)
    X, off = pack(series)
    say(f"embed forward seed {seed}: {len(series)} series, {off[-1]} rows")
    emb = B.twed_embed_forward(dev(vec), dev(X), off)
    torch.cuda.synchronize()
    got = emb.cpu().numpy()
    ref = ocnn.embed(params, [s.astype(np.float64) for s in series])
    assert got.shape == ref.shape == (len(series), 128)
    err = rel_norm(got, ref)
    say(f"  relative norm error {err:.2e}")
    assert err < 2e-2
    for i in range(len(series)):
        assert rel_norm(got[i], ref[i]) < 3e-2, i


def test_forward_chunk_independence():
    # the same series embedded alone and inside a larger collection agree exactly
    series = ragged_series(3)
    vec, _ = random_params(3)
    X, off = pack(series)
    emb_all = B.twed_embed_forward(dev(vec), dev(X), off).cpu().numpy()
    for i in (0, 5, len(series) - 1):
        Xi, offi = pack([series[i]])
        emb_i = B.twed_embed_forward(dev(vec), dev(Xi), offi).cpu().numpy()
        np.testing.assert_array_equal(emb_i[0], emb_all[i])


@pytest.fixture
def limits():
    """Sets twed_embed_set_limits for one test and restores the defaults."""
    yield B.twed_embed_set_limits
    B.twed_embed_set_limits(0, 0)


def test_forward_many_chunks_bitwise(limits):
    # A collection embedded in many small chunks (each a run of whole series
    # from a nonzero base row) equals the single-chunk forward bit for bit.
    # Chunks after the first start at row_base > 0: a segment length or row
    # index taken relative to the wrong base would read outside the chunk's
    # activations here.
    c = synth.knn_collection(60, 5)
    X, off = c.X.reshape(-1).astype(np.float32), c.off
    vec, params = random_params(4)
    ref = B.twed_embed_forward(dev(vec), dev(X), off).cpu().numpy()
    for rows in (600, 1500):
        limits(rows, 0)
        say(f"forward in chunks of {rows} rows: {c.count} series, {off[-1]} rows")
        got = B.twed_embed_forward(dev(vec), dev(X), off).cpu().numpy()
        np.testing.assert_array_equal(got, ref)
    limits(0, 0)
    picks = [c.count - 1, c.count // 2]
    want = ocnn.embed(params, [X[off[i]:off[i + 1]].astype(np.float64) for i in picks])
    for j, i in enumerate(picks):
        assert rel_norm(ref[i], want[j]) < 3e-2, i


def test_forward_default_chunk_boundary():
    # At the default limit (2^22 samples per chunk) a collection of 4.6e6
    # samples is embedded in two chunks; series of the second chunk agree bit
    # for bit with the same series embedded alone, and with the FP64 oracle.
    rng = np.random.default_rng(11)
    lengths = rng.integers(384, 641, 9000)
    off = np.zeros(len(lengths) + 1, dtype=np.int64)
    off[1:] = np.cumsum(lengths)
    assert off[-1] > (1 << 22) + 100_000
    X = np.cumsum(rng.standard_normal(off[-1]).astype(np.float32)).astype(np.float32)
    X -= np.repeat(X[off[:-1]], lengths)  # every series starts near 0
    vec, params = random_params(5)
    say(f"forward at the default chunk: {len(lengths)} series, {off[-1]} rows")
    emb = B.twed_embed_forward(dev(vec), dev(X), off).cpu().numpy()
    first2 = int(np.searchsorted(off, 1 << 22, side="right"))  # a series of the second chunk
    picks = [0, first2 - 2, first2 - 1, first2, first2 + 1, len(lengths) - 1]
    for i in picks:
        Xi = X[off[i]:off[i + 1]]
        alone = B.twed_embed_forward(dev(vec), dev(Xi), np.array([0, len(Xi)], np.int64)).cpu().numpy()
        np.testing.assert_array_equal(alone[0], emb[i])
    want = ocnn.embed(params, [X[off[i]:off[i + 1]].astype(np.float64) for i in picks[-3:]])
    for j, i in enumerate(picks[-3:]):
        assert rel_norm(emb[i], want[j]) < 3e-2, i


@pytest.mark.parametrize("seed", [0, 1])
def test_loss_and_gradients_match_oracle(seed):
    series = ragged_series(seed + 10)
    vec, params = random_params(seed + 10)
    X, off = pack(series)
    rng = np.random.default_rng(seed)
    n = len(series)
    P = 60
    pairs = np.stack([rng.integers(0, n, P), rng.integers(0, n, P)], axis=1)
    targets = rng.uniform(0.0, 300.0, P)
    say(f"embed loss/grad seed {seed}: {n} series, {P} pairs")
    loss, grad, emb = B.twed_embed_loss_grad(dev(vec), dev(X), off, dev(pairs, torch.int32), dev(targets),
                                             emb=torch.empty((n, 128), dtype=torch.float32, device="cuda"))
    torch.cuda.synchronize()
    ref_loss, ref_g, ref_emb = ocnn.batch_loss_and_grads(params, [s.astype(np.float64) for s in series],
                                                         [tuple(p) for p in pairs], targets)
    say(f"  loss {float(loss.item()):.6f} vs {ref_loss:.6f}")
    assert abs(float(loss.item()) - ref_loss) <= 2e-2 * abs(ref_loss)
    assert rel_norm(emb.cpu().numpy(), ref_emb) < 2e-2
    got = ocnn.unflatten(grad.cpu().numpy().astype(np.float64))
    for l in range(4):
        for name in ("W", "b"):
            g, r = got[name][l], ref_g[name][l]
            e, c = rel_norm(g, r), cosine(g, r)
            say(f"  layer {l + 1} {name}: rel {e:.2e} cos {c:.6f}")
            assert e < 5e-2 and c > 0.998, (l, name)


@pytest.fixture
def generic_gemm():
    """Runs a block with TWED_CNN_GEMM=generic (the per-wave tile kernels)."""
    class Switch:
        def __enter__(self):
            os.environ["TWED_CNN_GEMM"] = "generic"

        def __exit__(self, *exc):
            os.environ.pop("TWED_CNN_GEMM", None)
    yield Switch()
    os.environ.pop("TWED_CNN_GEMM", None)


def test_staged_conv_kernels_match_tile_kernels(generic_gemm):
    # The LDS-staged convolutions against the per-wave tile GEMM on a batch of
    # more rows than 512 weight-gradient workgroups cover in one chunk each
    # (so workgroups loop over chunks), series of every length class.  The
    # forward and data-gradient kernels run the same MFMA steps in the same
    # order: embeddings agree bit for bit.  The loss and the embedding
    # gradient are summed over pairs with atomics, so from there on two runs
    # may differ in rounding; the weight gradients also differ in summation
    # order (the tile kernel adds split-K partials with atomics).
    rng = np.random.default_rng(77)
    lengths = np.concatenate([[1, 2, 3, 4, 5, 255, 256, 257], rng.integers(60, 1200, 300)])
    series = [np.cumsum(rng.standard_normal(int(L))).astype(np.float32) for L in lengths]
    vec, _ = random_params(77)
    X, off = pack(series)
    n = len(series)
    assert off[-1] > 512 * 256
    pairs = np.stack([rng.integers(0, n, 512), rng.integers(0, n, 512)], axis=1).astype(np.int32)
    targets = rng.uniform(0.0, 300.0, 512).astype(np.float32)
    say(f"staged vs tile conv kernels: {n} series, {off[-1]} rows")

    def run():
        loss, grad, emb = B.twed_embed_loss_grad(dev(vec), dev(X), off, dev(pairs, torch.int32), dev(targets),
                                                 emb=torch.empty((n, 128), dtype=torch.float32, device="cuda"))
        fwd = B.twed_embed_forward(dev(vec), dev(X), off)
        torch.cuda.synchronize()
        return float(loss.item()), grad.cpu().numpy(), emb.cpu().numpy(), fwd.cpu().numpy()

    l_s, g_s, e_s, f_s = run()
    l_s2, g_s2, _, _ = run()
    with generic_gemm:
        l_t, g_t, e_t, f_t = run()
    np.testing.assert_array_equal(f_s, f_t)
    np.testing.assert_array_equal(e_s, e_t)
    assert abs(l_s - l_t) <= 1e-6 * abs(l_t) and abs(l_s - l_s2) <= 1e-6 * abs(l_s)
    assert rel_norm(g_s, g_s2) < 1e-5
    got, ref = ocnn.unflatten(g_s.astype(np.float64)), ocnn.unflatten(g_t.astype(np.float64))
    for l in range(4):
        for name in ("W", "b"):
            e = rel_norm(got[name][l], ref[name][l])
            say(f"  layer {l + 1} {name}: rel {e:.2e}")
            assert e < 1e-4, (l, name)


def test_out_of_range_pairs_contribute_nothing():
    series = ragged_series(20)
    vec, _ = random_params(20)
    X, off = pack(series)
    n = len(series)
    pairs = np.array([[0, 5], [3, 9], [12, 1]], dtype=np.int32)
    t = np.array([10.0, 20.0, 30.0], dtype=np.float32)
    l1, g1, _ = B.twed_embed_loss_grad(dev(vec), dev(X), off, dev(pairs, torch.int32), dev(t))
    l1, g1 = float(l1.item()), g1.cpu().numpy()
    bad = np.concatenate([pairs, [[n, 0], [-1, 2]]]).astype(np.int32)
    tb = np.concatenate([t, [1.0, 1.0]]).astype(np.float32)
    l2, g2, _ = B.twed_embed_loss_grad(dev(vec), dev(X), off, dev(bad, torch.int32), dev(tb))
    # the mean still divides by every listed pair
    np.testing.assert_allclose(float(l2.item()), l1 * 3 / 5, rtol=1e-5)
    # the gradients pass through BF16 operands, whose rounding depends on the scale
    assert rel_norm(g2.cpu().numpy(), g1 * 3 / 5) < 1e-2


def test_adamw_matches_oracle():
    n = B.twed_embed_param_count()
    rng = np.random.default_rng(4)
    w = rng.standard_normal(n).astype(np.float32)
    m = (rng.standard_normal(n) * 0.01).astype(np.float32)
    v = (rng.uniform(0, 1e-3, n)).astype(np.float32)
    g = (rng.standard_normal(n) * 0.1).astype(np.float32)
    tw_, tm, tv = dev(w), dev(m), dev(v)
    B.twed_embed_adamw(tw_, tm, tv, dev(g), 7, 1e-3, 1e-2)
    torch.cuda.synchronize()
    rw, rm, rv = ocnn.adamw_step(w, m, v, g, 7, 1e-3, 1e-2)
    # FP32 moments: a few units in the last place of the two summed terms
    # (the sum itself may cancel, so a bar relative to it alone is too tight),
    # plus the FP32 representation error of beta1 = 0.9 (<= 2^-25) and
    # beta2 = 0.999 (<= 2^-24) times the terms they weigh
    u = 2.0 ** -24
    g64, m64, v64 = g.astype(np.float64), m.astype(np.float64), v.astype(np.float64)
    bm = 4 * u * (0.9 * np.abs(m64) + 0.1 * np.abs(g64)) + 2.0 ** -25 * (np.abs(m64) + np.abs(g64))
    bv = 4 * u * (0.999 * v64 + 0.001 * g64 * g64) + 2.0 ** -24 * (v64 + g64 * g64)
    assert np.all(np.abs(tm.cpu().numpy() - rm) <= bm)
    assert np.all(np.abs(tv.cpu().numpy() - rv) <= bv)
    np.testing.assert_allclose(tw_.cpu().numpy(), rw, rtol=1e-5, atol=1e-7)


# ---- learned k-NN ------------------------------------------------------------------

NU, LAM = 1e-3, 1.0


def collection(count, seed_base):
    c = synth.knn_collection(count, seed_base)
    X = c.X.reshape(-1).astype(np.float32)
    T = c.T.astype(np.float32)
    return c, X, T


def oracle_dists(Q, TQ, offQ, DB, TDB, offDB, pairs):
    return oracle.get().pairs(Q.astype(np.float64), TQ.astype(np.float64), offQ, DB.astype(np.float64),
                              TDB.astype(np.float64), offDB, pairs, NU, LAM, 1.0, threads=threads())


def bf16(x):
    u = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


def index_for(DB, TDB, offDB, vec):
    return B.KnnIndex(dev(DB), dev(TDB), offDB, dev(vec), NU, LAM)


def test_knn_exhaustive_is_exact():
    db, DB, TDB = collection(160, 3)
    qc, Q, TQ = collection(6, 4)
    vec = knn.init_params(1)
    ix = index_for(DB, TDB, db.off, vec)
    k = 10
    say(f"knn exhaustive: {db.count} db, {qc.count} queries")
    ids, dist = ix.query(dev(Q), dev(TQ), qc.off, k=k, n_cand=db.count)
    torch.cuda.synchronize()
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    pairs = np.array([(q, j) for q in range(qc.count) for j in range(db.count)], dtype=np.int64)
    D = oracle_dists(Q, TQ, qc.off, DB, TDB, db.off, pairs).reshape(qc.count, db.count)
    for q in range(qc.count):
        ref = np.sort(D[q])[:k]
        np.testing.assert_allclose(dist[q], ref, rtol=1e-5)
        np.testing.assert_allclose(D[q, ids[q]], dist[q], rtol=1e-5)
        assert len(set(ids[q].tolist())) == k
    ix.close()


def test_knn_many_chunks_matches_single(limits):
    # index build and queries forced through many forward chunks and score
    # chunks (three queries per score chunk) give the default-limit answer
    # bit for bit; the exhaustive form stays exact against the oracle
    db, DB, TDB = collection(300, 3)
    qc, Q, TQ = collection(10, 4)
    vec = knn.init_params(3)
    runs = {}
    for name, lim in (("default", (0, 0)), ("chunked", (900, 3 * db.count * 4))):
        limits(*lim)
        ix = index_for(DB, TDB, db.off, vec)
        for n_cand in (40, db.count):
            say(f"knn {name}: n_cand {n_cand}")
            ids, dist = ix.query(dev(Q), dev(TQ), qc.off, k=10, n_cand=n_cand)
            runs[name, n_cand] = (ids.cpu().numpy(), dist.cpu().numpy())
        ix.close()
    for n_cand in (40, db.count):
        np.testing.assert_array_equal(runs["chunked", n_cand][0], runs["default", n_cand][0])
        np.testing.assert_array_equal(runs["chunked", n_cand][1], runs["default", n_cand][1])
    ids, dist = runs["chunked", db.count]
    pairs = np.array([(q, j) for q in range(qc.count) for j in range(db.count)], dtype=np.int64)
    D = oracle_dists(Q, TQ, qc.off, DB, TDB, db.off, pairs).reshape(qc.count, db.count)
    for q in range(qc.count):
        np.testing.assert_allclose(dist[q], np.sort(D[q])[:10], rtol=1e-5)


def test_knn_pruned_candidates():
    db, DB, TDB = collection(300, 3)
    qc, Q, TQ = collection(8, 4)
    vec = knn.init_params(2)
    k, n_cand = 5, 24
    ix = index_for(DB, TDB, db.off, vec)
    say(f"knn pruned: {db.count} db, {qc.count} queries, n_cand {n_cand}")
    ids, dist = ix.query(dev(Q), dev(TQ), qc.off, k=k, n_cand=n_cand)
    torch.cuda.synchronize()
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    # host scores from the network's own embeddings, rounded as the index stores them
    eq = bf16(B.twed_embed_forward(dev(vec), dev(Q), qc.off).cpu().numpy()).astype(np.float64)
    ed = bf16(B.twed_embed_forward(dev(vec), dev(DB), db.off).cpu().numpy()).astype(np.float64)
    S = (eq ** 2).sum(1)[:, None] + (ed ** 2).sum(1)[None, :] - 2 * eq @ ed.T
    pairs = np.array([(q, j) for q in range(qc.count) for j in range(db.count)], dtype=np.int64)
    D = oracle_dists(Q, TQ, qc.off, DB, TDB, db.off, pairs).reshape(qc.count, db.count)
    for q in range(qc.count):
        thr = np.sort(S[q])[n_cand - 1]
        tol = 1e-3 * (abs(thr) + 1.0)
        assert np.all(S[q, ids[q]] <= thr + tol), q           # returned ids were candidates
        np.testing.assert_allclose(D[q, ids[q]], dist[q], rtol=1e-5)
        keys = list(zip(dist[q].tolist(), ids[q].tolist()))
        assert keys == sorted(keys)
        sure = np.where(S[q] < thr - tol)[0]                   # certainly among the candidates
        others = np.setdiff1d(sure, ids[q])
        assert np.all(D[q, others] >= dist[q, -1] * (1 - 1e-5)), q
    ix.close()


def test_training_lowers_loss_and_helps_recall():
    # What the trained network gains, at the 200-candidate budget of the
    # k-NN query: it finds clearly more of the exact neighbours than the
    # untrained network (measured gains on this seed and collection: +0.10
    # to +0.18), and the exact re-rank finds far more than the network's own
    # ranking (+0.4).  64 queries against 1,500 database series; recall is
    # taken against the FP64 oracle's exact neighbours.
    db, DB, TDB = collection(1500, 3)
    qc, Q, TQ = collection(64, 4)
    dbc = knn.Collection(dev(DB), dev(TDB), db.off)
    tr = knn.Trainer(dbc, NU, LAM, seed=0, batch_series=128, pairs_per_step=1024, n_anchors=512)
    first = float(tr.step().item())
    secs = tr.train(999)
    last = float(np.mean([float(tr.step().item()) for _ in range(5)]))
    say(f"training: loss {first:.4f} -> {last:.4f} in {secs:.1f} s (mining {tr.mine_s:.1f} s), "
        f"{tr.pairs_seen} pairs")
    assert last < 0.5 * first
    pairs = np.array([(q, j) for q in range(qc.count) for j in range(db.count)], dtype=np.int64)
    D = oracle_dists(Q, TQ, qc.off, DB, TDB, db.off, pairs).reshape(qc.count, db.count)
    truth = knn.exact_knn_from_matrix(D, 10)
    rec = {}
    for name, vec in (("trained", tr.params.cpu().numpy()), ("untrained", knn.init_params(0))):
        ix = index_for(DB, TDB, db.off, vec)
        ids, _ = ix.query(dev(Q), dev(TQ), qc.off, k=10, n_cand=200)
        rec[f"{name}@200"] = knn.recall_at(ids.cpu().numpy(), truth)
        ids_net, _ = ix.query(dev(Q), dev(TQ), qc.off, k=10, n_cand=10)
        rec[name + "_network_only"] = knn.recall_at(ids_net.cpu().numpy(), truth)
        ix.close()
    say(f"recall@10: {rec}")
    assert rec["trained@200"] >= rec["untrained@200"] + 0.05
    assert rec["trained@200"] >= rec["trained_network_only"] + 0.25


def test_knn_long_series_exhaustive():
    # queries and database series longer than one wave's strip (1,024
    # samples): their pairs run the single-pair sweep; the exhaustive answer
    # is exact against the oracle
    rng = np.random.default_rng(41)
    lens_db = [1030, 1200, 300, 1500, 1100, 900, 2000, 1025]
    lens_q = [1300, 200]
    mk = lambda L: np.cumsum(rng.standard_normal(L)).astype(np.float32)
    DBs, Qs = [mk(L) for L in lens_db], [mk(L) for L in lens_q]
    DB, offDB = pack(DBs)
    Q, offQ = pack(Qs)
    TDB = np.concatenate([np.arange(L, dtype=np.float32) for L in lens_db])
    TQ = np.concatenate([np.arange(L, dtype=np.float32) for L in lens_q])
    ix = index_for(DB, TDB, offDB, knn.init_params(5))
    say("knn long series: 8 db, 2 queries")
    ids, dist = ix.query(dev(Q), dev(TQ), offQ, k=4, n_cand=len(lens_db))
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    ix.close()
    pairs = np.array([(q, j) for q in range(len(lens_q)) for j in range(len(lens_db))], dtype=np.int64)
    D = oracle_dists(Q, TQ, offQ, DB, TDB, offDB, pairs).reshape(len(lens_q), len(lens_db))
    for q in range(len(lens_q)):
        np.testing.assert_allclose(dist[q], np.sort(D[q])[:4], rtol=1e-5)
        np.testing.assert_allclose(D[q, ids[q]], dist[q], rtol=1e-5)


@pytest.mark.parametrize("lens", [[1], [371], [372], [373], [744, 1], [370, 2, 3, 369], [1, 2, 3, 4, 5] * 160,
                                  [1500], [17] * 400, [372] * 60])
def test_forward_windows_match_layers_bitwise(lens, generic_gemm):
    # The one-launch forward pass stores 372 rows per window: collections that
    # end at, before and behind a window's edge, series across several windows,
    # series shorter than the kernel width, more windows than compute units.
    # The embeddings are the bits of the layers swept one by one.
    rng = np.random.default_rng(sum(lens))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    X = dev(np.cumsum(rng.standard_normal(off[-1])))
    vec = dev(knn.init_params(7) + 0.05 * rng.standard_normal(B.twed_embed_param_count()).astype(np.float32))
    say(f"embed windows: {len(lens)} series, {off[-1]} rows")
    got = B.twed_embed_forward(vec, X, off).cpu().numpy()
    with generic_gemm:
        want = B.twed_embed_forward(vec, X, off).cpu().numpy()
    assert np.isfinite(got).all() and np.array_equal(got, want)


@pytest.mark.parametrize("P", [1, 3, 4, 5, 16, 17, 65536, 65537, 70001])
def test_pair_loss_over_workgroups(P):
    # A wave takes several pairs, four waves add one sum, and above 65,536
    # pairs the waves loop: pairs in no full wave or workgroup, and the loop.
    # The loss is compared with its FP64 value at the returned embeddings; the
    # sums of P / 16 workgroups round once per addition, each r to a few ulp of
    # its two logarithms.  The gradient of tiled pairs is that of the first 16.
    series = ragged_series(33)
    vec, _ = random_params(33)
    X, off = pack(series)
    rng = np.random.default_rng(P)
    base = np.stack([rng.integers(0, len(series), 16), rng.integers(0, len(series), 16)], axis=1)
    pairs, t = np.resize(base, (P, 2)), np.resize(rng.uniform(0.0, 300.0, 16), P).astype(np.float32)
    say(f"pair loss: {P} pairs")

    def run(p, tt):
        emb = torch.empty((len(series), 128), dtype=torch.float32, device="cuda")
        loss, grad, _ = B.twed_embed_loss_grad(dev(vec), dev(X), off, dev(p, torch.int32), dev(tt), emb=emb)
        return float(loss.item()), grad.cpu().numpy(), emb.cpu().numpy().astype(np.float64)

    loss, grad, emb = run(pairs, t)
    p = np.sqrt(((emb[pairs[:, 0]] - emb[pairs[:, 1]]) ** 2).sum(axis=1) + ocnn.EPS)
    lp, lt = np.log1p(p), np.log1p(t.astype(np.float64))
    r = lp - lt
    u = 2.0 ** -24
    bound = (2 * np.abs(r) * 8 * u * (lp + lt + 1)).mean() + (r * r).mean() * (20 + min(P // 16 + 1, 4096)) * u
    assert abs(loss - (r * r).mean()) <= bound
    if P % 16 == 0:
        # scaled by 16 / P before BF16 operands, as a power of two: only the
        # order of the atomic additions differs
        _, g16, _ = run(base, t[:16])
        assert rel_norm(grad, g16) < 1e-2


@pytest.mark.parametrize("n_db,n_cand", [(1, 1), (3, 2), (4095, 40), (4096, 4096), (4097, 33), (4099, 1000),
                                         (12293, 64), (12293, 5000)])
def test_candidate_selection_rounds_and_ties(n_db, n_cand):
    # The selection reads 4,096 scores per round, four per thread, and takes the
    # smallest scores, ties by the lowest id.  Seven distinct series repeated in
    # a random order give seven groups of exactly equal scores, so the
    # candidates follow from the order of the groups and the ids; with k = n_cand
    # (at most 64 of them) the query returns the nearest of them.
    rng = np.random.default_rng(n_db + n_cand)
    kinds = [np.cumsum(rng.standard_normal(8 + 3 * i)).astype(np.float32) + 4 * i for i in range(7)]
    which = rng.integers(0, len(kinds), n_db)
    DB, offDB = pack([kinds[w] for w in which])
    TDB = np.concatenate([np.arange(len(kinds[w]), dtype=np.float32) for w in which])
    vec = knn.init_params(3)
    Xk, offk = pack(kinds)
    Q = kinds[2] + 0.5
    both, off_both = pack(kinds + [Q])
    emb = bf16(B.twed_embed_forward(dev(vec), dev(both), off_both).cpu().numpy()).astype(np.float64)
    score = ((emb[:-1] - emb[-1]) ** 2).sum(axis=1)
    gaps = np.diff(np.sort(score))
    assert gaps.min() > 1e-3 * score.max()  # groups apart by far more than FP32 scores round
    chosen = np.lexsort((np.arange(n_db), score[which]))[:n_cand]
    D = oracle_dists(np.tile(Q, 1), np.arange(len(Q), dtype=np.float32), np.array([0, len(Q)]), Xk,
                     np.concatenate([np.arange(len(s), dtype=np.float32) for s in kinds]), offk,
                     np.array([(0, j) for j in range(len(kinds))]))
    want = chosen[np.lexsort((chosen, D[which[chosen]]))]
    k = min(n_cand, 64)
    say(f"candidate selection: {n_cand} of {n_db}")
    ix = index_for(DB, TDB, offDB, vec)
    ids, _ = ix.query(dev(Q), dev(np.arange(len(Q), dtype=np.float32)), np.array([0, len(Q)], dtype=np.int64), k=k,
                      n_cand=n_cand)
    ids = ids.cpu().numpy()[0]
    ix.close()
    assert np.array_equal(ids, want[:k])


def test_pair_count_at_its_limit():
    """2^31 - 1 pairs, the most the call takes, all of them outside the
    collection: accepted, zero loss and gradient."""
    vec, _ = random_params(3)
    X, off = pack(ragged_series(4)[:3])
    P = 2 ** 31 - 1
    say(f"loss and gradient of {P} pairs outside the collection")
    pairs = torch.full((P, 2), -1, dtype=torch.int32, device="cuda")
    target = torch.zeros(P, dtype=torch.float32, device="cuda")
    loss, grad, _ = B.twed_embed_loss_grad(dev(vec), dev(X), off, pairs, target)
    torch.cuda.synchronize()
    assert float(loss.item()) == 0.0
    assert float(grad.abs().max().item()) == 0.0
