"""The two register streams of a TN_HLL plan (register columns in LDS, one
launch per level) against the row-OR kernel's register stream of an ops plan,
on networks at the bounds of the columns: one and four registers a workgroup,
several workgroups a CU, several rounds, levels wider than a window, levels
of gathers only, saturation inside a run of levels."""
import numpy as np
import pytest

import tn_inputs as T

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2307_04890_amd as tn  # noqa: E402


def _both(n, ev, b, flags, saturation=True):
    h = T.hll_node_hashes(n, seed=n + b)
    ctx = tn.get_context()
    ref = tn.Plan(n, *ev, flags)
    want, we = ref.hll(h, b)
    p = tn.Plan(n, *ev, flags | tn.HLL)
    try:
        ctx.saturation(saturation)
        for _ in range(2):  # a second pass starts from the hashes again
            M, est = p.hll(h, b)
            assert torch.equal(M, want)
            assert torch.equal(est, we)
    finally:
        ctx.saturation(True)
        ref.close()
        p.close()


# 40,000 nodes: the last sizes with four registers a workgroup are below,
# 160,000 the last with one; a launch per level past four rounds of
# workgroups (2^11 registers at one a workgroup) and past 163,000 nodes
@pytest.mark.parametrize("n,b", [(37, 4), (1000, 12), (5000, 8), (30_000, 12), (40_650, 5), (41_000, 5),
                                 (50_000, 10), (50_000, 11), (163_000, 4), (170_000, 4)])
@pytest.mark.parametrize("flags", [0, tn.DIRECTED | tn.FORWARD])
def test_columns_and_levels_match_the_ops_stream(n, b, flags):
    _both(n, T.activity_driven(n, 4 * n, max(1, n // 3), seed=n), b, flags)


@pytest.mark.parametrize("saturation", [True, False])
@pytest.mark.parametrize("n,m,steps", [(300, 30_000, 15_000), (2000, 60_000, 30_000), (44_000, 1_500_000, 200_000)])
def test_streams_that_saturate(n, m, steps, saturation):
    _both(n, T.uniform_pairs(n, m, steps, seed=m), 6, 0, saturation)


@pytest.mark.parametrize("flags", [0, tn.FORWARD, tn.TIES_SEQUENTIAL])
def test_levels_of_gathers(flags):
    # stars: levels with many gathers and sources, some with no pair
    for n, steps, k in [(200, 500, 30), (5000, 300, 200), (45_000, 100, 1500)]:
        _both(n, T.star_steps(n, steps, k, seed=n), 5, flags)
    # one time step of everything: levels wider than a turn of every wavefront
    _both(3000, T.uniform_pairs(3000, 9000, 1, seed=3), 7, flags)
    _both(60_000, T.uniform_pairs(60_000, 30_000, 1, seed=4), 4, flags)


def test_networks_without_pairs():
    _both(100, (np.zeros(0, np.uint32), np.zeros(0, np.uint32), np.zeros(0, np.int64)), 5, 0)
    # every step a path of three nodes: gathers only
    t = np.repeat(np.arange(50, dtype=np.int64), 2)
    mid = np.arange(50, dtype=np.uint32) * 3 + 1
    src = np.stack([mid - 1, mid], 1).ravel()
    dst = np.stack([mid, mid + 1], 1).ravel()
    _both(151, (src, dst, t), 6, 0)


@pytest.mark.parametrize("n,b", [(1, 11), (2, 16), (200, 14), (170_000, 4)])
def test_rows_that_start_saturated(n, b):
    # a launch per level counts the rows not yet saturated: with one register
    # between all nodes some are from the start
    ev = T.activity_driven(max(n, 2), 5 * n, n, seed=n) if n > 2 else (
        np.zeros(1, np.uint32), np.full(1, n - 1, np.uint32), np.zeros(1, np.int64))
    top = np.uint64(3) << np.uint64(64 - b)
    h = (T.hll_node_hashes(n, seed=b) >> np.uint64(b)) | top  # every node in register 3
    for hashes in (h, np.full(n, h[0])):
        ref, p = tn.Plan(n, *ev), tn.Plan(n, *ev, tn.HLL)
        want, we = ref.hll(hashes, b)
        M, est = p.hll(hashes, b)
        assert torch.equal(M, want) and torch.equal(est, we)
        ref.close()
        p.close()


@pytest.mark.parametrize("flags", [0, tn.DIRECTED])
@pytest.mark.parametrize("m", [0, 1, 63, 64, 65, 959, 960, 961, 20_000])
def test_blocks_of_pairs(m, flags):
    # no pair, the last block's padding, blocks about the wavefronts' first
    # turns: one wide level, then levels of one pair each
    u = np.arange(0, 2 * m, 2, dtype=np.uint32)
    _both(2 * m + 2, (u, u + 1, np.zeros(m, np.int64)), 5, flags)
    k = np.arange(m, dtype=np.uint32)
    _both(m + 1, (k, k + 1, k.astype(np.int64)), 5, flags)


@pytest.mark.parametrize("flags", [0, tn.DIRECTED | tn.FORWARD])
@pytest.mark.parametrize("n", [700, 45_000])
@pytest.mark.parametrize("leaves,stars", [(2, 1), (2, 21), (2, 22), (3, 16), (3, 17), (4, 3), (63, 1)])
def test_levels_of_small_gathers(leaves, stars, n, flags):
    # stars of 3 to 64 nodes, side by side in a step: centres of 3, 4, 5 and 64
    # sources, levels of up to 64 gathers and of more, blocks of 64 that end
    # within a step and between steps, pairs beside them
    g = np.random.default_rng(n + leaves + stars)
    src, dst, t = [], [], []
    for step in range(200):
        at = g.permutation(n)[:stars * (leaves + 1) + 2]
        for c in range(stars if step % 7 else 1):
            star = at[c * (leaves + 1):(c + 1) * (leaves + 1)]
            src += [star[0]] * leaves
            dst += list(star[1:])
        src.append(at[-2])
        dst.append(at[-1])
        t += [step] * (len(src) - len(t))
    _both(n, (np.asarray(src, np.uint32), np.asarray(dst, np.uint32), np.asarray(t, np.int64)), 6, flags)
