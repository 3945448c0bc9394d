"""Fusion on proxies whose rows are nearly full, nearly empty, in between and
mixed, so that every kind of node (lists of left-out nodes, lists of kept
nodes, tables) and the choice between them meets the oracle, bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2307_04890_amd as tn  # noqa: E402


def _proxies(n, H, K, density, seed, diagonal=True):
    g = np.random.default_rng(seed)
    bucket = g.integers(0, K, (H, n)).astype(np.uint32)
    count = np.stack([np.bincount(bucket[j], minlength=K) for j in range(H)]).astype(np.int32)
    row = g.choice(np.asarray(density), size=(H, K, 1))
    bits = g.random((H, K, K)) < row
    if diagonal:
        bits |= np.eye(K, dtype=bool)
    kw = (K + 63) // 64
    packed = np.zeros((H, K, kw * 8), dtype=np.uint8)
    packed[:, :, :(K + 7) // 8] = np.packbits(bits, axis=2, bitorder="little")
    return bucket, count, packed.view(np.uint64)


def _check(n, bucket, count, P, pad=0, us=None):
    H, K, kw = P.shape
    wide = np.zeros((H, K, kw + pad), dtype=np.uint64)
    wide[:, :, :kw] = P
    args = (torch.from_numpy(wide.view(np.int64)).cuda(), torch.from_numpy(bucket.view(np.int32)).cuda(),
            torch.from_numpy(count).cuda(), n)
    est, lifted = tn.recombine(*args)
    us = np.arange(n) if us is None else us
    we, wl = oracle.recombine(n, P, bucket, us)
    assert (est.cpu().numpy()[us] == we).all()
    assert (lifted.cpu().numpy()[:, us] == wl).all()
    alone, none = tn.recombine(*args, lifted=False)
    assert none is None and torch.equal(alone, est)
    return we


KINDS = {
    "full": [1.0],
    "left_out": [0.995, 1.0],          # union of short lists
    "long_left_out": [0.9],            # ... of lists longer than a wavefront
    "kept": [0.01],                    # intersection of short lists
    "mixed": [0.02, 0.6, 0.98, 1.0],   # every kind in one call
    "between": [0.4, 0.6],
    "empty": [0.0],
}


@pytest.mark.parametrize("kind", sorted(KINDS))
# (tables, and lists where they fit: up to 16 hashes, from 24,576 nodes on)
@pytest.mark.parametrize("n,H,K", [(1, 1, 1), (1029, 16, 65), (5003, 2, 900), (8191, 3, 64), (8192, 3, 64),
                                   (8200, 16, 63), (9001, 5, 130), (10_000, 2, 1100), (9000, 17, 70)])
def test_every_kind_of_row(kind, n, H, K):
    bucket, count, P = _proxies(n, H, K, KINDS[kind], seed=n + H)
    us = np.random.default_rng(n).integers(0, n, 400) if n > 8000 else None
    _check(n, bucket, count, P, pad=n % 3, us=us)


def test_rows_that_lift_to_no_node():
    # without their own bit some rows keep nothing: est = 0
    bucket, count, P = _proxies(8700, 4, 40, [0.0, 0.03, 1.0], seed=5, diagonal=False)
    assert (_check(8700, bucket, count, P, us=np.arange(500)) == 0).any()


def test_buckets_without_nodes_and_one_bucket_with_all():
    n = 9000
    bucket, count, P = _proxies(n, 3, 200, [0.97, 0.05], seed=6)
    bucket[0] = 7
    bucket[1] = np.minimum(bucket[1], 20)
    count = np.stack([np.bincount(bucket[j], minlength=200) for j in range(3)]).astype(np.int32)
    _check(n, bucket, count, P, us=np.arange(600))


def test_estimates_do_not_depend_on_the_counts():
    # the counts enter the lifted sizes; the estimates are the proxies' alone
    n, us = 9000, np.arange(500)
    bucket, count, P = _proxies(n, 4, 50, [0.98], seed=7)
    want = oracle.recombine(n, P, bucket, us)[0]
    for other in (np.zeros_like(count), count + 1, count[:, ::-1].copy(), np.full_like(count, n)):
        est, _ = tn.recombine(torch.from_numpy(P.view(np.int64)).cuda(),
                              torch.from_numpy(bucket.view(np.int32)).cuda(), torch.from_numpy(other).cuda(), n)
        assert (est.cpu().numpy()[us] == want).all()


def _rows(P, density, seed):
    """The rows of every super-node redrawn at the given densities."""
    g = np.random.default_rng(seed)
    H, K, kw = P.shape
    bits = g.random((H, K, K)) < np.asarray(density)[:, :, None]
    bits |= np.eye(K, dtype=bool)
    packed = np.zeros((H, K, kw * 8), dtype=np.uint8)
    packed[:, :, :(K + 7) // 8] = np.packbits(bits, axis=2, bitorder="little")
    return packed.view(np.uint64)


# up to 65,536 nodes a small node is marked in a bitmap, past that in a hash
# table of at most 1024 entries; lists hold n / 64 left-out or 1024 kept nodes,
# other rows are bitmaps
@pytest.mark.parametrize("n,H,K", [(20_000, 16, 400), (65_536, 3, 700), (65_537, 3, 700), (150_001, 16, 2000),
                                   (90_000, 16, 90)])
def test_lists_bitmaps_and_both_tables(n, H, K):
    bucket, count, P = _proxies(n, H, K, [1.0], seed=n)
    g = np.random.default_rng(n + 1)
    # most rows leave out a few nodes, some about as many as a list may hold,
    # some many, some keep few
    level = g.choice([0.9995, 1 - 1 / 64, 0.5, 200 / n], size=(H, K), p=[0.9, 0.06, 0.02, 0.02])
    P = _rows(P, level, n + 2)
    _check(n, bucket, count, P, us=g.integers(0, n, 300))


def test_rows_at_the_bounds_of_the_lists():
    # one node per super-node: rows that leave out exactly n / 64 nodes or one
    # more, and that keep exactly 1024 nodes or one more
    n = K = 8192
    bucket = np.arange(n, dtype=np.uint32)[None]
    count = np.ones((1, n), dtype=np.int32)
    bits = np.ones((1, K, K), dtype=bool)
    g = np.random.default_rng(3)
    for r, zeros in [(0, 128), (1, 129), (2, n - 1024), (3, n - 1025), (4, 1), (5, n - 1), (6, n)]:
        bits[0, r, g.permutation(K)[:zeros]] = False
    P = np.packbits(bits, axis=2, bitorder="little").view(np.uint64)
    est = _check(n, bucket, count, P, us=np.arange(64))
    assert est[:8].tolist() == [n - 128, n - 129, 1024, 1025, n - 1, 1, 0, n]


# from the first n that takes lists on; about the last n whose nodes mark a bitmap of n bits, below it the last few
# sizes of a bitmap in 16-byte steps; lists of none, one to several chunks of 64
# entries, nodes of up to 16 chunks, more, and past 2560 entries
@pytest.mark.parametrize("n,K,H,density", [
    (24_575, 300, 16, [0.995, 1.0]), (24_576, 300, 16, [0.97, 1.0]), (24_577, 192, 3, [0.994]),
    (24_700, 300, 16, [0.02, 0.98, 1.0]), (30_001, 130, 5, [0.01]), (26_000, 260, 4, [0.4, 1.0]),
    (65_537, 1024, 9, [0.9992, 1.0]), (65_600, 512, 16, [0.994, 0.999]),
    (327_680, 1024, 4, [0.998]), (327_680, 1024, 4, [0.9997, 1.0]), (327_681, 1024, 4, [0.9997]),
])
def test_marked_and_hashed_nodes(n, K, H, density):
    bucket, count, P = _proxies(n, H, K, density, seed=n + K)
    us = np.concatenate([np.random.default_rng(n).integers(0, n, 250), [0, n - 1]])
    _check(n, bucket, count, P, us=us)


def test_lists_of_whole_chunks():
    # every bucket holds 64 nodes, so a list ends where a chunk does
    n, H, K = 32_768, 8, 512
    _, _, P = _proxies(n, H, K, [0.98, 1.0], seed=11)
    bucket = np.stack([np.random.default_rng(j).permutation(n) % K for j in range(H)]).astype(np.uint32)
    count = np.full((H, K), 64, np.int32)
    _check(n, bucket, count, P, us=np.arange(0, n, 37))


@pytest.mark.parametrize("n,K,H", [(60_000, 1024, 16), (24_576, 400, 9), (100_003, 1500, 12)])
def test_lists_with_some_intersections_and_bitmaps(n, K, H):
    # mostly nearly full rows, so that lists are the cheaper way, with a few rows
    # that keep little and a few in between: nodes of every kind
    bucket, count, P = _proxies(n, H, K, [0.01] * 2 + [0.5] * 5 + [1.0] * 600 + [0.999] * 393, seed=n)
    kept = np.bitwise_count(P).sum(axis=2)
    of = np.stack([kept[j][bucket[j]] for j in range(H)])  # by node
    pick = np.random.default_rng(n)
    us = np.unique(np.concatenate([
        pick.choice(np.flatnonzero(m), min(int(m.sum()), 120), replace=False)
        for m in ((of < 0.05 * K).any(0), ((of > 0.3 * K) & (of < 0.7 * K)).any(0), (of > 0.9 * K).all(0))]))
    _check(n, bucket, count, P, us=us)
