"""Edges of the bucket-major round phases of the point and given-D paths:
active counts at the wavefront and workgroup-chunk boundaries, one supplier
with every consumer in its bucket, exact ties inside buckets (packed and
unpacked order keys), partial serves, and the lattice test on coordinates
that the centring would round.  Plans and counters must equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2401_07378_amd import workloads as W
from tests.gpu_helpers import assert_pair_matches, gpu_pair, oracle_pair, to_dev

pytestmark = pytest.mark.gpu

EDGES = [(1, 1), (1, 300), (300, 1), (63, 65), (64, 64), (65, 63), (255, 257), (256, 256), (257, 255), (512, 513),
         (769, 1023), (1024, 1024), (1025, 900)]


@pytest.mark.parametrize("mn", EDGES, ids=lambda v: "%dx%d" % v)
@pytest.mark.parametrize("lattice", [0, 5])
@pytest.mark.parametrize("protocol", ["greedy", "random"])
def test_chunk_edges(mn, lattice, protocol):
    m, n = mn
    X, a, Y, b = W.random_pair(900 + m + 3 * n + lattice, m, n, 3, masses="integer" if lattice else "dirichlet",
                               lattice=lattice)
    for threads in (256, 512):
        g = gpu_pair(X, a, Y, b, protocol=protocol, seed=3, threads=threads)
        assert_pair_matches(g, oracle_pair(X, a, Y, b, protocol=protocol, seed=3), label=f"{mn}-{lattice}-{threads}")


@pytest.mark.parametrize("mn", [(1025, 1024), (1300, 2048), (2049, 700), (2300, 2560), (3072, 400), (3073, 64),
                                (300, 4096)], ids=lambda v: "%dx%d" % v)
@pytest.mark.parametrize("metric,protocol,lattice", [("l2", "greedy", 0), ("l2", "random", 40), ("l1", "greedy", 40),
                                                     ("l1", "random", 0)])
def test_points_per_thread(mn, metric, protocol, lattice):
    """Sides around the capacities of the workgroup's variants (4, 8, 12 and
    16 points per thread of 256; 2, 4 and 8 of 512), beyond one per thread."""
    m, n = mn
    X, a, Y, b = W.random_pair(500 + m + 3 * n + lattice, m, n, 2, masses="integer" if lattice else "dirichlet",
                               lattice=lattice)
    ref = oracle_pair(X, a, Y, b, metric, protocol=protocol, seed=4)
    for threads in (256, 512):
        g = gpu_pair(X, a, Y, b, metric, protocol=protocol, seed=4, threads=threads, path="on_chip")
        assert_pair_matches(g, ref, label=f"{mn}-{threads}")


@pytest.mark.parametrize("metric", ["l2", "sqeuclidean", "l1"])
def test_one_hub_supplier(metric):
    """Every consumer's nearest supplier is the same one, on an integer ring
    of equal distances: one bucket holds all claimants, tied."""
    rng = np.random.default_rng(17)
    Y = np.concatenate([rng.integers(0, 3, size=(700, 2)), [[1, 1]]]).astype(np.float32)
    X = np.concatenate([[[1, 1]], 60 + rng.integers(0, 9, size=(200, 2))]).astype(np.float32)
    b = np.full(len(Y), 1.0 / len(Y), np.float32)
    a = np.full(len(X), 1.0 / len(X), np.float32)
    assert_pair_matches(gpu_pair(X, a, Y, b, metric), oracle_pair(X, a, Y, b, metric), label=metric)


def test_centre_that_hides_low_bits():
    """Points at 0 and 2^-30 next to points at 1: both centre to -0.5 in
    FP32, so the pair looks like a lattice but its keys are not exact."""
    t = np.float32(2.0 ** -30)
    X = np.array([[0.0], [t], [1.0]] * 20, np.float32)
    Y = np.array([[t], [0.0], [1.0]] * 20, np.float32)
    a = np.full(60, 1.0 / 60, np.float32)
    g = gpu_pair(X, a, Y, a, "l1")
    assert_pair_matches(g, oracle_pair(X, a, Y, a, "l1"), label="l1")
    g = gpu_pair(X, a, Y, a, "l2")
    assert_pair_matches(g, oracle_pair(X, a, Y, a, "l2"), label="l2")


@pytest.mark.parametrize("protocol", ["greedy", "random"])
@pytest.mark.parametrize("y", [1.0, 2.0, -1.0])
@pytest.mark.parametrize("d", [1, 3])
def test_centre_below_the_coordinates_last_fp64_bit(d, y, protocol):
    """Two coincident suppliers at +-2^-53 (so that is the centre) and six
    consumers at y: y - c needs more bits than FP64 has, so the pair must not
    pass for a lattice.  The keys have all 53 bits; equal ones are served by
    consumer index."""
    X = np.full((2, d), np.sign(y) * 2.0 ** -53, np.float32)
    Y = np.full((6, d), y, np.float32)
    a = np.full(2, 0.5, np.float32)
    b = np.array([0.25, 0.125, 0.25, 0.125, 0.125, 0.125], np.float32)
    for metric in ("l2", "sqeuclidean"):
        g = gpu_pair(X, a, Y, b, metric, protocol=protocol, seed=9)
        assert_pair_matches(g, oracle_pair(X, a, Y, b, metric, protocol=protocol, seed=9), label=f"{metric}-{y}")


@pytest.mark.parametrize("kind", ["unit", "mixed", "tiny", "large"])
@pytest.mark.parametrize("d", [1, 3, 4, 7])
def test_matrix_core_keys_are_the_vector_keys(d, kind):
    """The matrix-core search (32 consumers and more) finds its slot by the
    equality of its keys with the fused multiply-add chain's; a key without an
    equal is re-scored.  One round of 128 consumers must therefore re-score as
    many as the vector search of the same consumers in eight calls of 16, also
    where products and norms are subnormal or span many binades."""
    rng = np.random.default_rng(40 + d)
    m, n = 301, 128

    def points(k):
        p = rng.uniform(-1, 1, size=(k, d))
        if kind == "mixed":
            p *= 10.0 ** rng.uniform(-22, 0, size=(k, d))
        return W.to_f32(p * {"tiny": 1e-20, "large": 1e15}.get(kind, 1.0))

    X, Y = points(m), points(n)
    a, b = np.full(m, 1.0 / m, np.float32), np.full(n, 1.0 / n, np.float32)
    whole = int(gpu_pair(X, a, Y, b, max_rounds=1)["stats"]["rescored"])
    b8 = np.full(16, 1.0 / 16, np.float32)
    parts = [int(gpu_pair(X, a, Y[k:k + 16], b8, max_rounds=1)["stats"]["rescored"]) for k in range(0, n, 16)]
    assert whole == sum(parts)
    assert whole < n or kind in ("tiny", "mixed")
    assert_pair_matches(gpu_pair(X, a, Y, b), oracle_pair(X, a, Y, b), label=kind)


@pytest.mark.parametrize("mn", [(300, 31), (300, 32), (15, 33), (1000, 48), (17, 49)], ids=lambda v: "%dx%d" % v)
@pytest.mark.parametrize("d", [1, 3, 4, 7])
def test_few_consumers(mn, d):
    """Consumer counts around the line between the vector search and two or
    three matrix-core tiles, with and without ties."""
    m, n = mn
    for lattice in (0, 6):
        X, a, Y, b = W.random_pair(m + 7 * n + d, m, n, d, masses="integer" if lattice else "dirichlet", lattice=lattice)
        for threads in (256, 512):
            assert_pair_matches(gpu_pair(X, a, Y, b, threads=threads), oracle_pair(X, a, Y, b), label=f"{mn}-{lattice}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("mn", [(1, 400), (257, 255), (513, 1024), (1500, 1300)], ids=lambda v: "%dx%d" % v)
def test_given_d_ties(mn, dtype):
    """Small integer distances (zeros of both signs among them): ties in
    every bucket, order keys packed for FP32 and compared in full for FP64."""
    import torch
    from paper_2401_07378_amd import binding
    m, n = mn
    rng = np.random.default_rng(m + n)
    D = rng.integers(0, 6, size=(m, n)).astype(dtype)
    D[(D == 0) & (rng.random((m, n)) < 0.5)] = -0.0
    a = W.dirichlet_masses(rng, m)
    b = W.dirichlet_masses(rng, n)
    r = binding.emd_approx_cost(to_dev(D), to_dev(a), to_dev(b))
    torch.cuda.synchronize()
    st = binding.stats_numpy(r["stats"])[0]
    ref = oracle.solve_cost(np.abs(D), a, b)
    k = int(st["nnz"])
    assert st["status"] == 0 and k == ref["nnz"] and int(st["rounds"]) == ref["rounds"]
    assert np.array_equal(r["plan_src"][:k].cpu().numpy(), ref["src"])
    assert np.array_equal(r["plan_dst"][:k].cpu().numpy(), ref["dst"])
    assert np.array_equal(r["plan_flow"][:k].cpu().numpy(), ref["flow"])
    assert int(st["near_ties_nn"]) == ref["near_ties_nn"]
    assert int(st["near_ties_order"]) == ref["near_ties_order"]
    assert float(r["cost"].item()) == pytest.approx(ref["cost"], rel=1e-12)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("protocol", ["greedy", "random"])
@pytest.mark.parametrize("mn", [(1, 1), (7, 256), (16, 64), (19, 130), (256, 31), (256, 256), (257, 40)],
                         ids=lambda v: "%dx%d" % v)
def test_given_d_scan_steps(mn, protocol, dtype):
    """Supplier counts around the steps of the search (8 or 16 entries per lane,
    4, 1) and sides around the one-point-per-thread variant."""
    import torch
    from paper_2401_07378_amd import binding
    m, n = mn
    rng = np.random.default_rng(3 * m + n)
    D = (rng.random((m, n)) * 4).astype(dtype)
    a, b = W.dirichlet_masses(rng, m), W.dirichlet_masses(rng, n)
    r = binding.emd_approx_cost(to_dev(D), to_dev(a), to_dev(b), protocol=protocol, seed=6)
    torch.cuda.synchronize()
    st = binding.stats_numpy(r["stats"])[0]
    ref = oracle.solve_cost(D, a, b, protocol=protocol, seed=6)
    k = int(st["nnz"])
    assert st["status"] == 0 and k == ref["nnz"] and int(st["rounds"]) == ref["rounds"]
    assert np.array_equal(r["plan_src"][:k].cpu().numpy(), ref["src"])
    assert np.array_equal(r["plan_dst"][:k].cpu().numpy(), ref["dst"])
    assert np.array_equal(r["plan_flow"][:k].cpu().numpy(), ref["flow"])
    assert float(r["cost"].item()) == pytest.approx(ref["cost"], rel=1e-12)
