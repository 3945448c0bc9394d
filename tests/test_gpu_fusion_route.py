"""Fusion by lists, each case with the route that it takes: rows, buckets and
counts where the lists' code can go wrong, at sizes and with enough full rows
that lists are taken, against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2307_04890_amd as tn  # noqa: E402


def full_rows(H, K):
    P = np.full((H, K, (K + 63) // 64), ~np.uint64(0))
    if K % 64:
        P[:, :, -1] = np.uint64((1 << (K % 64)) - 1)
    return P


def set_row(P, j, r, kept):
    """Row r of proxy j keeps the super-nodes where `kept` (K bools)."""
    bits = np.zeros(64 * P.shape[2], dtype=bool)
    bits[:kept.size] = kept
    P[j, r] = np.packbits(bits, bitorder="little").view(np.uint64)


def counts(bucket, K):
    return np.stack([np.bincount(b, minlength=K) for b in bucket]).astype(np.int32)


def fuse(n, bucket, count, P, route):
    """Estimates and lifted sizes, after checking the route by the kernels the
    call launched: the tables are transposed and built before the estimates."""
    ctx = tn.get_context()
    args = (torch.from_numpy(P.view(np.int64)).cuda(), torch.from_numpy(bucket.view(np.int32)).cuda(),
            torch.from_numpy(count).cuda(), n)
    ctx.profile(True)
    try:
        est, lifted = tn.recombine(*args)
        names = [k for k, _ in ctx.profile_take()]
    finally:
        ctx.profile(False)
    if route == "lists":
        assert names == ["aux", "recombine"]
    else:
        assert names[:3] == ["aux"] * 3 and names[3] == "recombine"
    return est.cpu().numpy(), lifted.cpu().numpy()


def check(n, bucket, count, P, us, route="lists"):
    est, lifted = fuse(n, bucket, count, P, route)
    we, wl = oracle.recombine(n, P, bucket, us)
    assert (est[us] == we).all()
    if route == "lists":
        assert (lifted[:, us] == wl).all()
    return we


def open_nodes(bucket, P, most, seed):
    """Nodes some row of which is not full."""
    full = (P == full_rows(1, P.shape[1])[:1, :1]).all(axis=2)
    us = np.flatnonzero(~np.stack([full[j][bucket[j]] for j in range(len(bucket))]).all(axis=0))
    return us if len(us) <= most else np.sort(np.random.default_rng(seed).choice(us, most, replace=False))


@pytest.mark.parametrize("n", [24_576, 24_577, 24_639])
@pytest.mark.parametrize("H", [1, 2])
def test_rows_at_the_bounds_of_the_lists(n, H):
    # a node a super-node: rows that leave out n / 64 nodes, one fewer or one more,
    # that keep 1,024 or one fewer or more, 1, none, or all but one
    K, g = n, np.random.default_rng(n)
    bucket = np.stack([np.arange(n), g.permutation(n)][:H]).astype(np.uint32)
    P = full_rows(H, K)
    lengths = [n // 64 - 1, n // 64, n // 64 + 1, n - 1023, n - 1024, n - 1025, 1, n - 1, n]
    for j in range(H):
        for r, zeros in enumerate(lengths):
            kept = np.ones(K, dtype=bool)
            kept[g.permutation(K)[:zeros]] = False
            set_row(P, j, r if j == 0 else bucket[1][len(lengths) - 1 - r], kept)
    est = check(n, bucket, counts(bucket, K), P, np.arange(32))
    if H == 1:
        assert est[:len(lengths)].tolist() == [n - z for z in lengths]


@pytest.mark.parametrize("n,H,K,route", [
    (24_576, 4, 700, "tables"), (30_001, 3, 1500, "lists"), (24_600, 16, 640, "tables"),
    (24_576, 4, 2500, "lists"), (24_600, 16, 3000, "lists")])
def test_rows_that_lift_to_few_or_no_nodes(n, H, K, route):
    g = np.random.default_rng(n + K)
    bucket = g.integers(0, K, (H, n)).astype(np.uint32)
    P = full_rows(H, K)
    for j in range(H):
        for k, r in enumerate(g.permutation(K)[:6]):
            kept = np.zeros(K, dtype=bool)
            kept[g.permutation(K)[:(0, 0, 1, 3, 20, 25)[k]]] = True
            set_row(P, j, r, kept)
    us = open_nodes(bucket, P, 400, n)
    est = check(n, bucket, counts(bucket, K), P, us, route)
    assert (est == 0).any() and (est > 0).any()


def test_buckets_without_nodes_and_one_bucket_with_all():
    n, H, K = 26_000, 4, 900
    g = np.random.default_rng(8)
    bucket = g.integers(0, K, (H, n)).astype(np.uint32)
    bucket[0] = 7  # its row leaves out buckets without nodes only
    bucket[1] = np.minimum(bucket[1], 300)
    P = full_rows(H, K)
    level = [0.0, 0.5, 0.995, 0.999]
    for j in range(H):
        for r in [7] if j == 0 else g.permutation(K)[:40]:
            kept = g.random(K) < level[int(g.integers(len(level)))]
            kept[7 if j == 0 else r] = True
            if j == 0:
                kept[g.integers(0, 7, 3)] = False
            set_row(P, j, r, kept)
    us = open_nodes(bucket, P, n, 0)
    assert len(us) == n  # the one row is not full
    check(n, bucket, counts(bucket, K), P, g.integers(0, n, 500))


@pytest.mark.parametrize("wrong", ["none", "zero", "one more", "reversed", "moved", "n"])
@pytest.mark.parametrize("K,some,route", [(800, 60, "tables"), (5000, 12, "lists")])
def test_counts_that_are_not_the_buckets_own_keep_lists_off(wrong, K, some, route):
    # the lists' lengths come from the counts; the estimates are the proxies' alone
    n, H = 25_000, 3
    g = np.random.default_rng(9)
    bucket = g.integers(0, K, (H, n)).astype(np.uint32)
    P = full_rows(H, K)
    for j in range(H):
        for r in g.permutation(K)[:some]:
            set_row(P, j, r, g.random(K) < g.choice([0.01, 0.997]))
    own = counts(bucket, K)
    moved = own.copy()
    moved[1, 5] += 1
    moved[1, 6] -= 1
    count = {"none": own, "zero": np.zeros_like(own), "one more": own + 1, "moved": moved,
             "reversed": own[:, ::-1].copy(), "n": np.full_like(own, n)}[wrong]
    check(n, bucket, count, P, open_nodes(bucket, P, 400, 1), route if wrong == "none" else "tables")


@pytest.mark.parametrize("each", [63, 64, 65, 128])
def test_lists_of_whole_chunks(each):
    # `each` nodes a bucket: lists of one, two or four buckets end where a chunk of
    # 64 entries does, one before or one after
    H, K = 6, 512
    n = each * K
    bucket = np.stack([np.random.default_rng(j).permutation(n) % K for j in range(H)]).astype(np.uint32)
    P = full_rows(H, K)
    g = np.random.default_rng(12)
    for j in range(H):
        for k, r in enumerate(g.permutation(K)[:120]):
            kept = np.ones(K, dtype=bool)
            kept[g.permutation(K)[:(1, 1, 2, 4)[k % 4]]] = False
            set_row(P, j, r, kept)
    check(n, bucket, counts(bucket, K), P, open_nodes(bucket, P, 500, 2))


# marked in a bitmap up to 327,680 nodes, in a hash table past that; nodes of few
# entries and of more than a small node may have (2,560 marked, 1,024 hashed), rows
# held as bitmaps among them
@pytest.mark.parametrize("n,H,K,route", [
    (24_576, 16, 400, "lists"), (24_577, 9, 2000, "lists"), (24_704, 16, 129, "lists"), (65_536, 3, 700, "tables"),
    (65_536, 6, 700, "lists"), (90_000, 16, 1000, "lists"), (327_680, 5, 1024, "lists"),
    (327_681, 5, 1024, "lists")])
def test_union_nodes_of_every_size(n, H, K, route):
    g = np.random.default_rng(n + H)
    bucket = g.integers(0, K, (H, n)).astype(np.uint32)
    P = full_rows(H, K)
    most = max(1, K // 64)
    for j in range(H):
        rows = g.permutation(K)
        for k, r in enumerate(rows[:K // 3]):
            kept = np.ones(K, dtype=bool)
            kept[g.permutation(K)[:g.integers(1, most + 1) if k else K // 2]] = False
            set_row(P, j, r, kept)
    check(n, bucket, counts(bucket, K), P, open_nodes(bucket, P, 300, 3), route)
