"""Launch shapes of the multinomial draw: every position of a launch is drawn once whatever the number of tasks is -
less than a wave's worth, one share per workgroup exactly used or one task over, halving shares with tickets, ragged
ends.  Counts against the oracle, element by element (whole numbers, so no tolerance)."""
import numpy as np
import pytest

import oracle
from paper_1409_5402_amd import binding

pytestmark = pytest.mark.gpu


def matrix(n_tasks, V, seed):
    """n_tasks nonzeros with counts 1 or 2, V per document (the last document ragged), words in ascending order."""
    rng = np.random.default_rng(seed)
    full, rest = divmod(n_tasks, V)
    lens = [V] * full + ([rest] if rest else [])
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rowidx = np.concatenate([np.arange(n, dtype=np.int32) for n in lens])
    val = rng.integers(1, 3, size=n_tasks).astype(np.float32)
    return oracle.CSC(len(lens), V, colptr, rowidx, val)


# workgroups at once at K = 4: at most 256 * 20 (five waves per SIMD), at least 256 * 16; shares of up to 128 positions
# are handed out without tickets
@pytest.mark.parametrize("n", [1, 63, 64, 65, 4096 * 64 + 1, 4608 * 128, 4608 * 128 + 1, 5120 * 128 + 1, 5120 * 200 + 77])
def test_every_position_is_drawn_once(n):
    X = matrix(n, V=min(n, 251), seed=n % 1000)
    K, m = 4, 3
    o = oracle.OracleLDA(X, K, 0.3, 0.05, seed=5, m0=1, G=8)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.3, 0.05, 5, 1, 8)
    assert np.array_equal(g.get(binding.NDK), o.ndk) and np.array_equal(g.get(binding.NWK), o.nwk)
    for _ in range(2):
        o.sweep(m)
        g.sweep(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
    g.close()


@pytest.mark.parametrize("form", ["multinomial", "poisson"])
@pytest.mark.parametrize("limit", [-1, 0, 7, 300])
def test_pairs_beyond_a_slot(form, limit):
    """Tasks of zero to some forty pairs: three fit a slot, the rest goes on in chunks of 15 (chains of up to three) or,
    where the pool is used up or lowered to nothing, to the word rows - hot words' copies among them (twelve words)."""
    rng = np.random.default_rng(31)
    counts = rng.integers(0, 9, size=(300, 12))
    cols = [np.flatnonzero(r) for r in counts]
    X = oracle.CSC(300, 12, np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32),
                   np.concatenate(cols).astype(np.int32), counts[counts > 0].astype(np.float32))
    K = 40
    o = oracle.OracleLDA(X, K, 0.4, 0.05, seed=9, m0=1, G=3)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.4, 0.05, 9, 1, 3)
    g.debug_chunk_limit(limit)
    for m in (60, 1, 20):
        if form == "poisson":
            o.sweep_poisson(m * 0.7)
            g.sweep_poisson(m * 0.7)
        else:
            o.sweep(m)
            g.sweep(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
        np.testing.assert_allclose(g.get(binding.PHI), o.phi, rtol=1e-6)
    g.close()


@pytest.mark.parametrize("K,G", [(4, 1), (4, 3), (4, 1000), (130, 8)])
def test_heavy_tasks_are_drawn_once(K, G):
    """Counts of one to two for most words and up to 40 for a few, in a matrix large enough for a list of heavy tasks
    (more than 128 positions for each of 3072 workgroups): the largest groups are drawn first and passed over later.  Groups
    smaller than a count, of exactly a count, and no heavy group at all (G = 1); an empty document."""
    rng = np.random.default_rng(8)
    D, V = 1500, 400
    counts = rng.integers(1, 3, size=(D, V))
    counts[rng.integers(0, D, 1500), rng.integers(0, V, 1500)] = rng.integers(3, 41, 1500)
    counts[7, :] = 0
    cols = [np.flatnonzero(r) for r in counts]
    X = oracle.CSC(D, V, np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32),
                   np.concatenate(cols).astype(np.int32), counts[counts > 0].astype(np.float32))
    o = oracle.OracleLDA(X, K, 0.2, 0.05, seed=13, m0=2, G=G)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.2, 0.05, 13, 2, G)
    assert np.array_equal(g.get(binding.NDK), o.ndk) and np.array_equal(g.get(binding.NWK), o.nwk)
    for m in (1, 11):
        o.sweep(m)
        g.sweep(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
    g.close()


@pytest.mark.parametrize("extra", [1, 777])
def test_full_shares_where_phi_is_large(extra):
    """1024 topics and 33,000 words (135 MB of phi), 6.3 million tasks: shares by tickets round after round.  Every
    document and word keeps exactly m copies of each token."""
    X = matrix(3072 * 512 * 4 + extra, V=33000, seed=3)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, 1024, 0.1, 0.05, 5, 1, 8)
    m = 2
    g.sweep(m)
    docs = np.add.reduceat(X.val.astype(np.int64), X.colptr[:-1])
    words = np.bincount(X.rowidx, weights=X.val, minlength=X.V).astype(np.int64)
    assert np.array_equal(np.asarray(g.get(binding.NDK)).reshape(X.D, 1024).sum(1, dtype=np.int64), m * docs)
    assert np.array_equal(np.asarray(g.get(binding.NWK)).reshape(X.V, 1024).sum(1, dtype=np.int64), m * words)
    g.close()


@pytest.mark.parametrize("K,m", [(16, 2.5), (128, 40.5), (144, 2.5), (144, 40.5), (240, 12.25), (272, 40.5), (528, 2.5)])
def test_poisson_at_any_multiple_of_16(K, m):
    """Both occupancies of the Poisson kernel for a multiple of 16 topics, at the ends of their ranges: four waves up to 128
    topics and, from ten copies on, up to 256; three beyond.  Counts against the oracle."""
    rng = np.random.default_rng(K)
    counts = rng.integers(1, 9, size=(60, 90)) * (rng.uniform(size=(60, 90)) < 0.4)
    cols = [np.flatnonzero(r) for r in counts]
    X = oracle.CSC(60, 90, np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32),
                   np.concatenate(cols).astype(np.int32), counts[counts > 0].astype(np.float32))
    o = oracle.OracleLDA(X, K, 0.2, 0.05, seed=17, m0=1, G=4)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.2, 0.05, 17, 1, 4)
    for _ in range(2):
        o.sweep_poisson(m)
        g.sweep_poisson(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
    g.close()


# One number of topics and more for every form of the draw kernel that the other tests leave out: blocks that fill the row but are
# fewer than 32 (136, 200, 1200: the last word's and the last document's rows end the matrices), one batch of three to
# seven loads per block, aligned (388, 770, 896) and not (259, 333, 509, 641, 701, 893, 895), the contiguous scan with a ragged
# end (897, 1001, 1023), and several batches of one, two and four loads (1028 and 1283, 1156, 1200 and 1795, 1540).
@pytest.mark.parametrize("K", [136, 200, 259, 333, 388, 509, 641, 701, 770, 893, 895, 896, 897, 1001, 1023, 1028, 1156, 1200, 1283, 1540, 1795])
def test_every_form_of_the_draw_kernel(K):
    """Sweeps in full and single tasks through the debug hook, which draws with the same form, against the oracle."""
    rng = np.random.default_rng(K)
    counts = rng.integers(1, 13, size=(37, 53)) * (rng.uniform(size=(37, 53)) < 0.35)
    counts[2, :] = 0
    counts[:, 52] = counts[36, :] = 1
    cols = [np.flatnonzero(r) for r in counts]
    X = oracle.CSC(37, 53, np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32),
                   np.concatenate(cols).astype(np.int32), counts[counts > 0].astype(np.float32))
    m, G, seed = 7, 4, 99
    o = oracle.OracleLDA(X, K, 0.2, 0.01, seed=seed, m0=m, G=G)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.2, 0.01, seed, m, G)
    ids = np.unique(np.concatenate([rng.choice(g.task_count, 70, replace=False), [0, g.task_count - 1]]))
    for _ in range(2):
        assert np.array_equal(g.debug_draw(m, ids), oracle.draw_tasks(X, K, G, m, seed, oracle.pass_word(g.pass_index), o.theta, o.phi, ids))
        o.sweep(m)
        g.sweep(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
        assert np.array_equal(g.get(binding.THETA), o.theta) and np.array_equal(g.get(binding.PHI), o.phi)
    g.close()


# the ends of the ranges in which a document's theta row is in LDS (288 to 896), aligned and not, whole blocks and not, and their
# neighbours
@pytest.mark.parametrize("K", [284, 287, 288, 291, 292, 384, 385, 448, 500, 512, 516, 640, 641, 701, 768, 769, 892, 895, 896, 900])
def test_theta_rows_beside_the_counts(K):
    """Documents of one to 120 words, so that waves hold tasks of one, of two and of dozens of documents: lanes whose document
    has a row in LDS, lanes whose row went to another document, lanes that never had one.  Counts against the oracle."""
    rng = np.random.default_rng(K)
    lens = np.concatenate([rng.integers(1, 4, 90), rng.integers(20, 121, 60)])
    rng.shuffle(lens)
    rowidx = np.concatenate([np.sort(rng.choice(130, n, replace=False)) for n in lens]).astype(np.int32)
    val = rng.integers(1, 5, size=len(rowidx)).astype(np.float32)
    X = oracle.CSC(len(lens), 130, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), rowidx, val)
    o = oracle.OracleLDA(X, K, 0.2, 0.05, seed=23, m0=1, G=3)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.2, 0.05, 23, 1, 3)
    for m in (1, 30, 4):
        o.sweep(m)
        g.sweep(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
    g.close()


# every form of the normaliser kernel, at both ends of its range and off multiples of four; sliced: words shared out among
# workgroups (more than 176 topics, at least 3 million entries of phi, 65,536 nonzeros, 64 per document)
@pytest.mark.parametrize("K,V,D,most", [
    *[(K, 90, 70, 60) for K in (1, 3, 4, 5, 15, 16, 17, 50, 63, 64, 65, 100, 127, 128, 129, 177, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048)],
    *[(K, V, 500, 300) for K, V in ((177, 17000), (256, 12000), (257, 12000), (509, 6000), (512, 6000), (1001, 3000), (1024, 3000), (2045, 1500), (2048, 1500))]])
def test_normaliser_in_every_form(K, V, D, most):
    """mu against sums in double: documents from empty to `most` words, one topic of one word infinite.  Products of one sign
    in a chain of 4 ceil(K / 256) and a tree of six: an error of half an ulp per step."""
    rng = np.random.default_rng(K + V)
    lens = rng.integers(0, most + 1, size=D)
    lens[[0, D // 2, D - 1]] = 0, most, 1
    rowidx = np.concatenate([np.sort(rng.choice(V, n, replace=False)) for n in lens]).astype(np.int32)
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    g = binding.SameLDA(D, V, colptr, rowidx, np.ones(len(rowidx), np.float32), K, 0.1, 0.05, 1, 1)
    theta = rng.gamma(0.5, size=(D, K)).astype(np.float32) + np.float32(0.01)
    phi = (rng.gamma(0.5, size=(V, K)) / V).astype(np.float32)
    phi[rowidx[-1], K - 1] = np.inf
    g.set(binding.THETA, theta)
    g.set(binding.PHI, phi)
    doc = np.repeat(np.arange(D), lens)
    want = np.concatenate([(theta[doc[i:i + 4096]].astype(np.float64) * phi[rowidx[i:i + 4096]]).sum(1) for i in range(0, len(doc), 4096)])
    np.testing.assert_allclose(g.sddmm(), want, rtol=(4 * -(-K // 256) + 8) * 2.0 ** -24, atol=0)
    g.close()


# one, two, four and eight copies of the topic totals, at the ends of their ranges; more documents than workgroups that add them up
@pytest.mark.parametrize("K", [1, 3, 128, 129, 256, 257, 512, 513])
def test_topic_totals_are_the_counts(K):
    """n_k against both count matrices after every form of a sweep (whole numbers, so no tolerance)."""
    X = matrix(9000, V=3, seed=K)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.3, 0.05, 5, 1, 8)
    for sweep in (None, lambda: g.sweep(3), lambda: g.sweep_poisson(2.5), lambda: g.sweep_sampled(2), lambda: g.sweep(1, 0.5)):
        if sweep:
            sweep()
        nk = np.asarray(g.get(binding.NK)).astype(np.int64)
        assert np.array_equal(nk, np.asarray(g.get(binding.NDK)).reshape(X.D, K).sum(0, dtype=np.int64))
        assert np.array_equal(nk, np.asarray(g.get(binding.NWK)).reshape(X.V, K).sum(0, dtype=np.int64))
    g.close()


# numbers of topics that are no multiple of 16: rows that end inside a block of loads at every remainder, fewer than four topics,
# few copies and many
@pytest.mark.parametrize("K,m", [(1, 3.5), (3, 3.5), (4, 3.5), (5, 40.5), (15, 2.5), (17, 40.5), (30, 2.5), (50, 40.5), (100, 2.5), (127, 40.5), (150, 2.5), (200, 40.5),
                                 (255, 2.5), (257, 2.5), (333, 40.5), (1001, 2.5)])
def test_poisson_at_any_number_of_topics(K, m):
    """Counts against the oracle; the last word and the last document, whose rows end the matrices, are drawn for as well."""
    rng = np.random.default_rng(K)
    counts = rng.integers(1, 9, size=(50, 70)) * (rng.uniform(size=(50, 70)) < 0.4)
    counts[:, 69] = counts[49, :] = 1
    cols = [np.flatnonzero(r) for r in counts]
    X = oracle.CSC(50, 70, np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32),
                   np.concatenate(cols).astype(np.int32), counts[counts > 0].astype(np.float32))
    o = oracle.OracleLDA(X, K, 0.2, 0.05, seed=19, m0=1, G=4)
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.2, 0.05, 19, 1, 4)
    for _ in range(2):
        o.sweep_poisson(m)
        g.sweep_poisson(m)
        assert np.array_equal(g.get(binding.NDK), o.ndk)
        assert np.array_equal(g.get(binding.NWK), o.nwk)
    g.close()


# n_dk in rows of one, two or four documents: fewer documents than a row, one row and a rest, several
@pytest.mark.parametrize("K", [1, 2, 3, 4, 50, 129, 257, 258, 1001, 1026, 2047])
@pytest.mark.parametrize("D", [1, 2, 3, 5, 6, 23])
def test_theta_and_totals_of_few_documents(D, K):
    """theta is n_dk / m + alpha in binary32, element by element, and n_k the sum over either matrix, collapsed and sampled."""
    rng = np.random.default_rng(D)
    lens = rng.integers(1, 8, size=D)
    rowidx = np.concatenate([np.sort(rng.choice(7, n, replace=False)) for n in lens]).astype(np.int32)
    X = oracle.CSC(D, 7, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), rowidx, rng.integers(1, 4, size=len(rowidx)).astype(np.float32))
    g = binding.SameLDA(X.D, X.V, X.colptr, X.rowidx, X.val, K, 0.3, 0.05, 5, 1, 8)
    for sweep, m in ((lambda: g.sweep(7), 7), (lambda: g.sweep_sampled(2), 0), (lambda: g.sweep_poisson(2.5), 2.5)):
        sweep()
        ndk = np.asarray(g.get(binding.NDK)).reshape(D, K)
        nk = np.asarray(g.get(binding.NK)).astype(np.int64)
        assert np.array_equal(nk, ndk.sum(0, dtype=np.int64))
        assert np.array_equal(nk, np.asarray(g.get(binding.NWK)).reshape(X.V, K).sum(0, dtype=np.int64))
        if m:
            assert np.array_equal(g.get(binding.THETA), ndk.astype(np.float32) / np.float32(m) + np.float32(0.3))
    g.close()
