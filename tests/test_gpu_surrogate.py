"""The surrogate's kernels against its FP64 twin (same BF16 rounding points),
the top-k selection against a brute-force order, training, and the
retrieval test: recall@10 of surrogate-pruned NNS-EMD against exhaustive
NNS-EMD, and what training gains over the untrained network."""
import numpy as np
import pytest

from oracle import surrogate_oracle as SO
from paper_2401_07378_amd import surrogate as SG
from paper_2401_07378_amd import workloads as W
from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


def _theta(seed, bias=0.05):
    th = SG.init_params(seed).astype(np.float64)
    r = np.random.default_rng(seed + 1)
    for name, o, shp in SG.param_layout()[0]:
        if name.startswith("b"):
            th[o:o + int(np.prod(shp))] = r.normal(0.0, bias, int(np.prod(shp)))
    return th.astype(np.float32)


def _sets(seed, sizes):
    r = np.random.default_rng(seed)
    off = np.zeros(len(sizes) + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    X = W.to_f32(r.random((off[-1], 3)))
    a = np.concatenate([W.dirichlet_masses(r, k) for k in sizes]).astype(np.float32)
    return X, a, off


def _close_blockwise(got, want, rel):
    for name, o, shp in SG.param_layout()[0]:
        n = int(np.prod(shp))
        g, w = got[o:o + n].astype(np.float64), want[o:o + n]
        err = np.linalg.norm(g - w) / max(np.linalg.norm(w), 1e-30)
        assert err <= rel, (name, err)


def _close_elementwise(got, want, rtol, atol_frac, label=""):
    """Every gradient element: |g - w| <= rtol |w| + atol_frac max|w| of its
    parameter block.  The twin rounds to BF16 at the kernels' points, so the
    two differ by FP32 accumulation and by an occasional BF16 rounding that
    an FP32 intermediate takes the other way (one BF16 step, 2^-8 relative,
    in that intermediate); rtol and the block-scaled floor cover those,
    while a wrong sign, a dropped chunk or a swapped index on any element
    above the floor does not pass."""
    for name, o, shp in SG.param_layout()[0]:
        n = int(np.prod(shp))
        g, w = got[o:o + n].astype(np.float64), want[o:o + n]
        scale = max(float(np.abs(w).max()), 1e-30)
        bad = np.abs(g - w) > rtol * np.abs(w) + atol_frac * scale
        assert not bad.any(), (label, name, int(bad.sum()), n, float(np.abs(g - w).max() / scale))


def test_embed_matches_twin():
    from paper_2401_07378_amd import binding
    # ragged chunks of 64 points, an empty set (zero row) and a 16-chunk set
    sizes = [1, 2, 63, 64, 65, 0, 128, 129, 200, 256, 300, 1000, 7]
    X, a, off = _sets(1, sizes)
    th = _theta(2)
    E = binding.sg_embed(to_dev(th), to_dev(X), to_dev(a), to_dev(off)).cpu().numpy()
    want = SO.embed(th, X, a, off, rounding=True)
    assert np.abs(want).max() > 0.1
    np.testing.assert_allclose(E, want, rtol=1e-3, atol=1e-4 * np.abs(want).max())


def test_predict_matches_twin_and_flags_bad_indices():
    import torch
    from paper_2401_07378_amd import binding
    r = np.random.default_rng(3)
    th = _theta(4)
    Eq = W.to_f32(np.abs(r.normal(0, 0.5, (3, 256))))
    Ec = W.to_f32(np.abs(r.normal(0, 0.5, (130, 256))))
    got = binding.sg_predict(to_dev(th), to_dev(Eq), to_dev(Ec)).cpu().numpy()
    want = SO.head(th, np.repeat(Eq[:1], 130, 0), Ec, rounding=True)
    np.testing.assert_allclose(got, want, rtol=1e-3)
    qi = r.integers(0, 3, 77).astype(np.int32)
    ci = r.integers(0, 130, 77).astype(np.int32)
    got = binding.sg_predict(to_dev(th), to_dev(Eq), to_dev(Ec), to_dev(qi), to_dev(ci)).cpu().numpy()
    np.testing.assert_allclose(got, SO.head(th, Eq[qi], Ec[ci], rounding=True), rtol=1e-3)
    ci[5] = 130
    qi[9] = -1
    got = binding.sg_predict(to_dev(th), to_dev(Eq), to_dev(Ec), to_dev(qi), to_dev(ci)).cpu().numpy()
    assert np.isnan(got[5]) and np.isnan(got[9]) and np.isfinite(np.delete(got, [5, 9])).all()


def test_predict_unaligned_tables_take_the_general_path():
    """Embedding tables that start off a 16-byte boundary (a view one float
    in) go through the unfused head; same values as the aligned call."""
    import torch
    from paper_2401_07378_amd import binding
    r = np.random.default_rng(31)
    th = _theta(32)
    Eq = W.to_f32(np.abs(r.normal(0, 0.5, (2, 256))))
    Ec = W.to_f32(np.abs(r.normal(0, 0.5, (200, 256))))
    qi = r.integers(0, 2, 150).astype(np.int32)
    ci = r.integers(0, 200, 150).astype(np.int32)
    flat = torch.zeros(1 + Ec.size, dtype=torch.float32, device="cuda")
    flat[1:] = to_dev(Ec).reshape(-1)
    Ec_off = flat[1:].view(200, 256)
    assert Ec_off.data_ptr() % 16 != 0
    a = binding.sg_predict(to_dev(th), to_dev(Eq), to_dev(Ec), to_dev(qi), to_dev(ci)).cpu().numpy()
    b = binding.sg_predict(to_dev(th), to_dev(Eq), Ec_off, to_dev(qi), to_dev(ci)).cpu().numpy()
    want = SO.head(th, Eq[qi], Ec[ci], rounding=True)
    np.testing.assert_allclose(a, want, rtol=1e-3)
    np.testing.assert_allclose(b, want, rtol=1e-3)
    torch.cuda.synchronize()


@pytest.mark.parametrize("pairs,lo,hi", [(37, 1, 200), (64, 256, 256), (3, 1, 3)])
def test_loss_grad_matches_twin(pairs, lo, hi):
    from paper_2401_07378_amd import binding
    r = np.random.default_rng(pairs)
    sizes = r.integers(lo, hi + 1, 2 * pairs)
    X, a, off = _sets(pairs + 100, sizes)
    th = _theta(pairs + 200)
    y = W.to_f32(r.uniform(0.05, 0.8, pairs))
    loss, grad = binding.sg_loss_grad(to_dev(th), to_dev(X), to_dev(a), to_dev(off), to_dev(y))
    want_loss, want_grad = SO.loss_and_grad(th, X, a, off, y, rounding=True)
    assert float(loss.item()) == pytest.approx(want_loss, rel=1e-3)
    g = grad.cpu().numpy()
    _close_blockwise(g, want_grad, 1e-2)
    _close_elementwise(g, want_grad, 3e-2, 3e-3, label=f"{pairs}-{lo}-{hi}")


def test_loss_is_nan_for_bad_offsets():
    from paper_2401_07378_amd import binding
    X, a, off = _sets(5, [10, 12, 9, 11])
    bad = off.copy()
    bad[-1] -= 3
    loss, _ = binding.sg_loss_grad(to_dev(_theta(6)), to_dev(X), to_dev(a), to_dev(bad),
                                   to_dev(np.ones(2, np.float32)))
    assert np.isnan(float(loss.item()))


def test_adam_step_matches_twin():
    import torch
    from paper_2401_07378_amd import binding
    X, a, off = _sets(7, [30, 40, 25, 33])
    th = _theta(8)
    r = np.random.default_rng(9)
    m0 = W.to_f32(r.normal(0, 1e-3, th.size))
    v0 = W.to_f32(np.abs(r.normal(0, 1e-5, th.size)))
    y = np.array([0.3, 0.2], np.float32)
    t, m, v = to_dev(th), to_dev(m0), to_dev(v0)
    grad = torch.empty_like(t)
    binding.sg_train_step(t, m, v, 3, 1e-3, to_dev(X), to_dev(a), to_dev(off), to_dev(y), grad=grad)
    g = grad.cpu().numpy().astype(np.float64)
    want_t, want_m, want_v = SO.adam(th.astype(np.float64), m0.astype(np.float64), v0.astype(np.float64), g, 3, 1e-3)
    # FP32 rounding of each term (not of the possibly cancelled sum) bounds the error.
    tm = 0.9 * np.abs(m0) + 0.1 * np.abs(g)
    tv = 0.999 * v0 + 0.001 * g * g
    assert np.all(np.abs(m.cpu().numpy() - want_m) <= 1e-6 * tm + 1e-30)
    assert np.all(np.abs(v.cpu().numpy() - want_v) <= 1e-6 * tv + 1e-30)
    np.testing.assert_allclose(t.cpu().numpy(), want_t, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("n,k", [(1, 1), (5, 3), (1000, 1000), (1025, 1024), (100000, 1000), (100000, 10),
                                 (70001, 257)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_topk_matches_brute_force(n, k, dtype):
    import torch
    from paper_2401_07378_amd import binding
    r = np.random.default_rng(n + k)
    v = r.integers(-50, 50, n).astype(np.float64) / 7.0  # many ties
    if n > 10:
        v[r.choice(n, 3, replace=False)] = np.nan
        v[r.choice(n, 3, replace=False)] = -0.0
        v[r.choice(n, 2, replace=False)] = np.inf
    v = v.astype(np.float32) if dtype == "f32" else v
    got = binding.topk_smallest(to_dev(v), k).cpu().numpy()
    np.testing.assert_array_equal(got, SO.topk_smallest(v, k))
    torch.cuda.synchronize()


@pytest.mark.parametrize("case", ["continuous", "sampled_positions_small", "all_equal", "narrow"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_topk_large_inputs_threshold_pass(case, dtype):
    """Above 32768 values a sampled threshold narrows the input first; the
    answer must still be the exact (value, index) order: continuous values,
    the smallest values placed exactly at the sampled positions, every value
    equal (the candidates overflow and the direct pass runs), and a narrow
    band with heavy ties at the threshold."""
    import torch
    from paper_2401_07378_amd import binding
    r = np.random.default_rng(77)
    n, k = 200003, 1000
    v = r.random(n)
    if case == "sampled_positions_small":
        pos = (np.arange(4096, dtype=np.int64) * n) // 4096
        v[pos] = -1.0 - r.random(4096)
    elif case == "all_equal":
        v[:] = 0.25
    elif case == "narrow":
        v = np.round(r.random(n) * 300) / 300
    v[r.choice(n, 5, replace=False)] = np.nan
    v[r.choice(n, 3, replace=False)] = -0.0
    v = v.astype(np.float32) if dtype == "f32" else v
    got = binding.topk_smallest(to_dev(v), k).cpu().numpy()
    np.testing.assert_array_equal(got, SO.topk_smallest(v, k))
    torch.cuda.synchronize()


def _train(num_pairs, epochs, seed=11):
    import torch
    X, a, off = W.surrogate_training_pairs(num_pairs, seed=3100 + seed)
    Xd, ad, offd = to_dev(X), to_dev(a), to_dev(off)
    labels, st = SG.nnsemd_labels(Xd, ad, offd, num_pairs, 256)
    assert np.all(st["status"] == 0)
    tr = SG.Trainer(SG.init_params(seed), torch.device("cuda:0"))
    hist = tr.fit(Xd, ad, off, labels, batch=512, epochs=epochs, lr=2e-3)
    return tr, hist


def test_training_reduces_loss_and_ranks_held_out_pairs():
    from paper_2401_07378_amd import binding
    tr, hist = _train(8192, 12)
    assert hist[-1] < 0.2 * hist[0], hist
    X, a, off = W.surrogate_training_pairs(2048, seed=4242)
    Xd, ad, offd = to_dev(X), to_dev(a), to_dev(off)
    labels, _ = SG.nnsemd_labels(Xd, ad, offd, 2048, 256)
    E = binding.sg_embed(tr.theta, Xd, ad, offd)
    import torch
    idx = torch.arange(2048, dtype=torch.int32, device=Xd.device) * 2
    pred = binding.sg_predict(tr.theta, E, E, idx, idx + 1).cpu().numpy()
    y = labels.cpu().numpy()
    rank = lambda v: np.argsort(np.argsort(v))
    rho = np.corrcoef(rank(pred), rank(y))[0, 1]
    assert rho > 0.9, rho


def test_retrieval_recall_and_gain():
    """The retrieval configuration as stated: the surrogate trained on 200000
    NNS-EMD labels; 100 queries against 100000 candidates: the trained
    surrogate keeps 1000 (1 % of the NNS-EMD work) and NNS-EMD re-ranks them; the top-10
    must match exhaustive NNS-EMD with recall >= 0.99, every returned cost
    must be the exhaustive NNS-EMD value, and the untrained network must do
    clearly worse (what training gains)."""
    import torch
    from paper_2401_07378_amd import binding
    tr, _ = _train(200000, 16)
    ps = W.retrieval_3d(100000)
    Y, b, yo = to_dev(ps.Y), to_dev(ps.b), to_dev(ps.y_off)
    E_tr = SG.build_index(tr.theta, Y, b, yo)
    th0 = to_dev(SG.init_params(11))
    E_0 = SG.build_index(th0, Y, b, yo)
    aq = to_dev(W.uniform_masses(256))
    xo = to_dev(np.array([0, 256], np.int64))
    zeros = torch.zeros(100000, dtype=torch.int32, device=Y.device)
    cand = torch.arange(100000, dtype=torch.int32, device=Y.device)
    rec_tr, rec_0 = [], []
    for q in range(100):
        Xq = to_dev(W.retrieval_query(q))
        ex = binding.emd_approx_batched(Xq, aq, xo, Y, b, yo, pair_x=zeros, pair_y=cand, max_m=256, max_n=256)
        truth = binding.topk_smallest(ex["costs"][:100000], 10).cpu().numpy()
        costs = ex["costs"][:100000].cpu().numpy()
        got = SG.retrieve(tr.theta, E_tr, Xq, aq, Y, b, yo, 256)
        gi, gc = got["idx"].cpu().numpy(), got["cost"].cpu().numpy()
        np.testing.assert_array_equal(gc, costs[gi])
        rec_tr.append(len(set(gi) & set(truth)) / 10)
        g0 = SG.retrieve(th0, E_0, Xq, aq, Y, b, yo, 256)["idx"].cpu().numpy()
        rec_0.append(len(set(g0) & set(truth)) / 10)
    r_tr, r_0 = float(np.mean(rec_tr)), float(np.mean(rec_0))
    print(f"recall@10 trained {r_tr:.4f}, untrained {r_0:.4f}")
    assert r_tr >= 0.99, (r_tr, r_0)
    assert r_tr - r_0 >= 0.1, (r_tr, r_0)


@pytest.mark.parametrize("sizes", [[1, 0, 64], [63, 65, 128, 129], [0, 0, 200] + [7] * 600 + [0]],
                         ids=["edges", "chunks", "many"])
def test_embed_chunk_edges(sizes):
    """Sets that end at, before and after a 64-point chunk, empty ones (zero
    rows, whatever the biases), and more sets than resident workgroups.
    Bound: FP32 accumulation, and layer-1 values that round to BF16 the other
    way (2^-8 of one of 256 products)."""
    from paper_2401_07378_amd import binding
    r = np.random.default_rng(len(sizes))
    off = np.zeros(len(sizes) + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    X = W.to_f32(r.random((off[-1], 3)))
    a = np.concatenate([W.dirichlet_masses(r, k) for k in sizes if k]).astype(np.float32)
    th = _theta(3, bias=0.3)
    E = binding.sg_embed(to_dev(th), to_dev(X), to_dev(a), to_dev(off)).cpu().numpy()
    want = SO.embed(th, X, a, off, rounding=True)
    assert np.abs(E - want).max() <= 1e-3 * np.abs(want).max()
    for s, k in enumerate(sizes):
        assert k > 0 or not E[s].any()


@pytest.mark.parametrize("pairs,sizes", [(1, [1, 65]), (2, [64, 63, 128, 1]), (130, [3, 66, 64])],
                         ids=["one", "edges", "many-sets"])
def test_gradient_chunk_edges(pairs, sizes):
    """Sets that end around the 64-point chunks, fewer and more sets than
    resident workgroups: the gradient against the twin (tolerance as in the
    ragged-batch gradient test)."""
    from paper_2401_07378_amd import binding
    X, a, off = _sets(pairs, [sizes[k % len(sizes)] for k in range(2 * pairs)])
    th = _theta(5)
    y = W.to_f32(np.random.default_rng(pairs).uniform(0.1, 1.0, pairs))
    loss, grad = binding.sg_loss_grad(to_dev(th), to_dev(X), to_dev(a), to_dev(off), to_dev(y))
    wl, wg = SO.loss_and_grad(th, X, a, off, y, rounding=True)
    assert float(loss.item()) == pytest.approx(float(wl), rel=1e-3)
    _close_blockwise(grad.cpu().numpy(), wg, 2e-2)


@pytest.mark.parametrize("pairs,sizes", [(2, [1, 0, 2, 1]), (40, [0, 1, 2, 7, 0, 30]), (32, [64, 1, 63, 65]),
                                         (4097, [2]), (2, [9000, 7400, 1, 3])],
                         ids=["tiny", "empty", "straddling", "past-one-round", "few-large"])
def test_gradient_chunks_across_sets(pairs, sizes):
    """The backward's 64-point chunks hold points of several sets, empty sets
    lie between them, and a workgroup takes a second chunk (more than 256 x 64
    points); two calls give the same bits."""
    from paper_2401_07378_amd import binding
    X, a, off = _sets(pairs, [sizes[k % len(sizes)] for k in range(2 * pairs)])
    th = _theta(6)
    y = W.to_f32(np.random.default_rng(pairs).uniform(0.1, 1.0, pairs))
    loss, grad = binding.sg_loss_grad(to_dev(th), to_dev(X), to_dev(a), to_dev(off), to_dev(y))
    wl, wg = SO.loss_and_grad(th, X, a, off, y, rounding=True)
    assert float(loss.item()) == pytest.approx(float(wl), rel=1e-3)
    _close_blockwise(grad.cpu().numpy(), wg, 2e-2)
    again = binding.sg_loss_grad(to_dev(th), to_dev(X), to_dev(a), to_dev(off), to_dev(y))[1]
    assert np.array_equal(grad.cpu().numpy(), again.cpu().numpy())
