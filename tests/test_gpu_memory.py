"""GPU memory that calls need: with little of it left they take the way that
needs less, and the context gives back what it keeps between calls."""
import contextlib
import gc

import numpy as np
import pytest
import torch

import oracle
import tn_inputs as T
from gpu_util import host

pytestmark = pytest.mark.gpu

tn = pytest.importorskip("paper_2307_04890_amd")

MB = 1 << 20


def free_bytes():
    torch.cuda.synchronize()
    gc.collect()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


@contextlib.contextmanager
def only(left):
    """All but about `left` bytes of the device's free memory taken."""
    hold, free = [], free_bytes()
    try:
        # (a large allocation leaves more than was reported before it)
        for _ in range(4):
            if free > left + 4 * MB:
                hold.append(torch.empty(free - left, dtype=torch.uint8, device="cuda"))
            free = torch.cuda.mem_get_info()[0]
        assert abs(free - left) < 8 * MB
        yield
    finally:
        hold.clear()
        torch.cuda.empty_cache()


def test_kept_stream_buffers_are_given_back():
    # a stream of large chunks leaves its ring (4 slots of 12 MB and more) with the
    # context; a plan that does not fit beside it takes that memory
    n, m = 40_000, 2_400_000
    s, d, t = T.uniform_pairs(4000, m, m // 8, seed=1)  # 36,000 rows never fill
    few = tuple(a[:2_000_000] for a in (s, d, t))
    ctx = tn.Context()
    p = tn.Plan(n, *few, ctx=ctx)
    want = host(p.execute())
    p.close()
    st = tn.build_component_matrix_streamed(n, s, d, t, chunk_events=600_000, ctx=ctx)[1]
    assert st["chunks_run"] >= 4
    with only(16 * len(few[0]) - 16 * MB):
        p = tn.Plan(n, *few, ctx=ctx)
    assert (host(p.execute()) == want).all()
    p.close()
    ctx.close()


def test_hll_columns_without_room_for_their_scratch():
    # register columns of 50,000 nodes, 2,048 registers, need 102 MB beside the
    # registers; a launch per level needs a few rows
    n, b = 50_000, 11
    s, d, t = T.activity_driven(n, 60_000, 60_000, seed=3)
    h = np.random.default_rng(4).integers(0, 2**64, size=n, dtype=np.uint64)
    p = tn.Plan(n, s, d, t, tn.HLL)
    ctx = p.ctx = tn.Context()
    want = torch.empty((n, 1 << b), dtype=torch.uint8, device="cuda")
    west = torch.empty(n, dtype=torch.float64, device="cuda")
    M, est = torch.empty_like(want), torch.empty_like(west)
    before = free_bytes()
    p.hll(h, b, M=want, est=west)
    assert before - free_bytes() > 90 * MB  # on columns
    ctx.close()
    ctx = p.ctx = tn.Context()
    with only(60 * MB):
        p.hll(h, b, M=M, est=est)
        torch.cuda.synchronize()
    assert torch.equal(M, want) and torch.equal(est, west)
    p.ctx = tn.get_context()
    p.close()
    ctx.close()


def test_fusion_without_room_for_lists():
    # the lists' set-up takes 83 MB more than the tables' 1.1 GB; either gives the
    # oracle's estimates
    n, H, K = 1_000_000, 16, 8192
    g = np.random.default_rng(5)
    bucket = g.integers(0, K, (H, n)).astype(np.uint32)
    count = np.stack([np.bincount(b, minlength=K) for b in bucket]).astype(np.int32)
    P = np.full((H, K, K // 64), ~np.uint64(0))
    for j in range(H):
        for r in g.integers(0, K, 40):  # all but a few of the others
            for c in g.integers(0, K, 5):
                if c != r:
                    P[j, r, c // 64] &= ~(np.uint64(1) << np.uint64(c % 64))
    args = (torch.from_numpy(P.view(np.int64)).cuda(), torch.from_numpy(bucket.view(np.int32)).cuda(),
            torch.from_numpy(count).cuda(), n)
    ctx = tn.Context()
    before = free_bytes()
    want, _ = tn.recombine(*args, lifted=False, ctx=ctx)
    need = before - free_bytes()
    ctx.close()
    full = (P == ~np.uint64(0)).all(axis=2)
    us = np.flatnonzero(~np.stack([full[j][bucket[j]] for j in range(H)]).all(axis=0))[:300]
    we, _ = oracle.recombine(n, P, bucket, us)
    assert (want.cpu().numpy()[us] == we).all() and (we < n).any()
    ctx = tn.Context()
    with only(need - 40 * MB):
        est, _ = tn.recombine(*args, lifted=False, ctx=ctx)
        torch.cuda.synchronize()
    assert torch.equal(est, want)
    ctx.close()


@pytest.mark.parametrize("hll", [False, True])
def test_plans_without_room_for_their_column_form(hll):
    # the columns' forms of a plan take half as much again as its schedule; it runs
    # without them too
    n = 20_000
    s, d, t = T.uniform_pairs(n, 3_000_000, 750_000, seed=6)
    flags = tn.HLL if hll else 0
    h = np.random.default_rng(7).integers(0, 2**64, size=n, dtype=np.uint64)
    p = tn.Plan(n, s, d, t, flags)
    size, base = p.stats["device_bytes"], (8 if hll else 16) * len(s)
    assert size > 1.3 * base
    want = p.hll(h, 6)[0].cpu() if hll else host(p.execute())
    p.close()
    ctx = tn.Context()
    before = free_bytes()
    p = tn.Plan(n, s, d, t, flags, ctx=ctx)
    assert abs(before - free_bytes() - size) < 6 * MB
    p.close()
    with only((size + base) // 2):
        p = tn.Plan(n, s, d, t, flags, ctx=ctx)
    assert base <= p.stats["device_bytes"] < (size + base) // 2
    got = p.hll(h, 6)[0].cpu() if hll else host(p.execute())
    assert (got == want).all()
    p.close()
    ctx.close()
