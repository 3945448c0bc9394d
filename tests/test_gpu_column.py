"""GPU parity of the row-OR stream on one workgroup per word column: networks
whose columns fit in LDS, at the edges of the sizes and level widths where it
is taken, against the slices of the matrix in memory (an explicit slice width
selects them) and the oracle's words."""
import numpy as np
import pytest
import torch

import oracle
import tn_inputs as T
from gpu_util import host
from test_gpu_exact import _partial_network

pytestmark = pytest.mark.gpu

tn = pytest.importorskip("paper_2307_04890_amd")

def case(kind, n, per_node, seed):
    m = int(n * per_node)
    if kind == "uniform":
        return T.uniform_pairs(n, m, max(2, m // n), seed=seed)
    if kind == "random":
        return T.random_tiny(n, m, max(2, m // 300), seed=seed, allow_self=True)
    if kind == "stars":
        return T.star_steps(n, m // 25, 90, seed=seed)
    return T.activity_driven(n, m, max(2, m // 5), seed=seed)


# sizes about a word column, level widths about the thread counts, and the LDS
# (20,472 rows: 1,024 of scratch to 19,447 nodes, fewer to 20,407)
SIZES = [(2, "random", 5), (63, "random", 60), (64, "random", 60), (65, "uniform", 40), (513, "uniform", 30),
         (1025, "uniform", 12), (3000, "random", 20), (7167, "activity", 6), (7168, "activity", 6),
         (8193, "uniform", 5), (10_000, "random", 12), (10_001, "stars", 1), (16_385, "uniform", 4),
         (19_447, "activity", 3), (19_448, "uniform", 4), (20_407, "activity", 3),
         (20_408, "activity", 3)]


@pytest.mark.parametrize("flags", [0, tn.DIRECTED | tn.FORWARD, tn.TIES_SEQUENTIAL])
@pytest.mark.parametrize("n,kind,per_node", SIZES)
def test_word_columns_in_lds_match_slices_in_memory(n, kind, per_node, flags):
    s, d, t = case(kind, n, per_node, 9100 + n)
    nw = oracle.words(n)
    p = tn.Plan(n, s, d, t, flags)
    want = p.execute(slice_words=1).clone()
    wout, winn = tn.component_sizes(want, n)
    # row padding of more than the matrix itself, left dirty by an earlier use
    C = torch.full((n, 2 * nw + 3), -1, dtype=torch.int64, device="cuda")
    ctx = tn.get_context()
    try:
        for sat in (True, False, True):
            ctx.saturation(sat)
            p.execute(C=C)
            assert (host(C) == host(want)).all(), sat
            # the sizes that come with the columns
            E, out, inn = p.execute_sizes(C)
            assert (host(E) == host(want)).all(), sat
            assert torch.equal(out, wout) and torch.equal(inn, winn), sat
            S, _ = tn.build_component_matrix_streamed(n, s, d, t, flags,
                                                      chunk_events=max(1, len(s) // 5))
            assert (host(S) == host(want)).all(), sat
    finally:
        ctx.saturation(True)
        p.close()
    ref = oracle.forward_matrix if flags & tn.FORWARD else oracle.reverse_matrix
    for w0 in (0, nw - 1):
        got = ref(n, s, d, t, directed=bool(flags & tn.DIRECTED),
                  sequential=bool(flags & tn.TIES_SEQUENTIAL), w0=w0, nw=1)
        assert (host(want)[:, w0:w0 + 1] == got).all(), w0


# half columns: their tail bits, the row ids (32,767 with the scratch rows) and
# the counters (32,512 nodes), and too few ops for them
@pytest.mark.parametrize("sat", [True, False])
@pytest.mark.parametrize("n,kind,per_node", [
    (20_416, "random", 3), (20_449, "uniform", 3), (25_001, "stars", 2), (31_743, "activity", 3),
    (31_744, "activity", 3), (32_511, "uniform", 2), (32_512, "random", 2), (32_513, "random", 2),
    (25_000, "uniform", 0.5)])
def test_half_columns_match_slices_in_memory(n, kind, per_node, sat):
    s, d, t = case(kind, n, per_node, 9700 + n)
    p = tn.Plan(n, s, d, t)
    ctx = tn.get_context()
    want = host(p.execute(slice_words=1))
    wout, winn = tn.component_sizes(p.execute(slice_words=1), n)
    C = torch.full((n, oracle.words(n) + 3), -1, dtype=torch.int64, device="cuda")
    try:
        ctx.saturation(sat)
        p.execute(C=C)
        assert (host(C) == want).all()
        C.fill_(-1)
        E, out, inn = p.execute_sizes(C)
        assert (host(E) == want).all()
        assert torch.equal(out, wout) and torch.equal(inn, winn)
    finally:
        ctx.saturation(True)
        p.close()


def test_full_half_columns_reach_every_counter_plane():
    # one op a level takes the fewest threads, so a lane counts 127 rows
    n = 32_512
    spokes = np.random.default_rng(9800).permutation(np.arange(1, n, dtype=np.uint32))
    d = np.concatenate([spokes, spokes])
    s, t = np.zeros_like(d), np.arange(len(d), dtype=np.int64)
    p = tn.Plan(n, s, d, t)
    C, out, inn = p.execute_sizes()
    assert (host(C) == np.uint64(2**64 - 1)).all()  # 32,512 = 508 words
    assert (out == n).all() and (inn == n).all()
    p.close()


@pytest.mark.parametrize("n", [1000, 9000])
def test_full_columns_stop_and_are_counted(n):
    # every row fills up long before the earliest events: plans give the full
    # matrix, a stream ends early, and a plan's traffic is one pass over it
    s, d, t = T.uniform_pairs(n, 40 * n, 40, seed=9200)
    nw = oracle.words(n)
    p = tn.Plan(n, s, d, t)
    C = p.execute()
    assert tn.get_context().last_traffic() == (n * nw, n * nw)
    p.close()
    full = np.full((n, nw), ~np.uint64(0))
    if n % 64:
        full[:, -1] = np.uint64((1 << (n % 64)) - 1)
    assert (host(C) == full).all()
    S, st = tn.build_component_matrix_streamed(n, s, d, t, chunk_events=2 * n)
    assert (host(S) == full).all()
    assert st["saturated"] == 1 and st["chunks_run"] < st["chunks"]


@pytest.mark.parametrize("K", [65, 1000, 4096])
@pytest.mark.parametrize("sat", [True, False])
def test_hashed_proxies_of_wide_and_narrow_levels(K, sat):
    # proxies of narrow and of wide levels by chunk size, against the mapped
    # networks' matrices
    n, H = 12_000, 3
    s, d, t = T.uniform_pairs(n, 60_000, 60, seed=9300)
    A = T.hash_coefficients(H, seed=9301)
    ctx = tn.get_context()
    try:
        ctx.saturation(sat)
        # chunks of one time step have narrow levels, of many steps wide ones
        outs = [tn.hash_build_proxies(n, s, d, t, A, K, chunk_events=c) for c in (0, 300, 20_000)]
    finally:
        ctx.saturation(True)
    bucket = outs[0][0].cpu().numpy()
    for h in range(H):
        want = oracle.reverse_matrix(K, bucket[h][s], bucket[h][d], t)
        for o in outs:
            assert (host(o[2][h]) == want).all(), h


def test_streams_of_one_context_keep_their_matrices():
    # two contexts on streams of their own, each with its own size
    rng = np.random.default_rng(9400)
    made = []
    for n in (900, 8200):
        s, d, t = T.uniform_pairs(n, 12 * n, 12, seed=int(rng.integers(1 << 30)))
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            p = tn.Plan(n, s, d, t)
            C = p.execute()
            made.append((n, s, d, t, p, C, st))
    torch.cuda.synchronize()
    for n, s, d, t, p, C, st in made:
        assert torch.equal(C, p.execute(slice_words=2)), n
        p.close()


# rows about eight, four, three, two and one column to a compute unit, past the
# last that fits, a lone node, no events
BATCH = [(1, 0), (64, 500), (700, 0), (2558, 9000), (2559, 9000), (5117, 9000), (5118, 9000),
         (6823, 9000), (6824, 9000), (10_235, 9000), (10_236, 30_000), (20_407, 30_000),
         (20_480, 9000)]


@pytest.mark.parametrize("flags", [0, tn.DIRECTED | tn.FORWARD, tn.TIES_SEQUENTIAL])
@pytest.mark.parametrize("last", [len(BATCH), len(BATCH) - 1, 3])
def test_batches_of_word_columns_match_single_plans(last, flags):
    nets = []
    for k, (n, m) in enumerate(BATCH[:last]):
        ev = T.uniform_pairs(n, m, max(2, m // 40), seed=9500 + k) if n > 1 and m else \
            (np.zeros(0, np.uint32), np.zeros(0, np.uint32), np.zeros(0, np.int64))
        nets.append((n, *ev))
    want = []
    for net in nets:
        p = tn.Plan(*net, flags)
        want.append(p.execute(slice_words=1).clone())
        p.close()
    b = tn.Batch(nets, flags=flags)
    ctx = tn.get_context()
    try:
        for sat in (True, False, True):
            ctx.saturation(sat)
            for lead in (0, 3):  # a second set of outputs, with row padding left dirty
                Cs = [torch.full((n, oracle.words(n) + lead), -1, dtype=torch.int64, device="cuda")
                      for n, *_ in nets]
                for _ in range(2):  # captured, then replayed
                    b.execute(Cs)
                    for k, (C, w) in enumerate(zip(Cs, want)):
                        assert (host(C) == host(w)).all(), (BATCH[k], sat, lead)
    finally:
        ctx.saturation(True)
        b.close()


@pytest.mark.parametrize("n", [500, 9000, 20_407, 21_000])
def test_saturation_switched_within_a_stream(n):
    # batches with saturation off leave no slice state; those after it must not
    # take the rows for the identity's
    s, d, t = T.uniform_pairs(n, 900, 90, seed=9600 + n)
    cut = np.searchsorted(t, [30, 60])
    ctx = tn.get_context()
    live = tn.Online(n, flags=tn.FORWARD)
    try:
        for k, on in enumerate((False, True, True)):
            part = slice(*([0, *cut, len(t)][k:k + 2]))
            ctx.saturation(on)
            live.insert(s[part], d[part], t[part])
        got = host(live.C)
    finally:
        ctx.saturation(True)
        live.close()
    p = tn.Plan(n, s, d, t, tn.FORWARD)
    assert (got == host(p.execute(slice_words=1))).all()
    p.close()


def test_sizes_of_plans_on_two_streams_of_one_context():
    # a long execution on one stream while short ones run on another: nothing of
    # the context's may pass between them
    made = []
    for n, per_node in ((16_000, 6), (1000, 3)):
        p = tn.Plan(n, *case("uniform", n, per_node, 9900 + n))
        C, out, inn = p.execute_sizes(slice_words=2)
        # a set of outputs for each of several executions
        outs = [(torch.empty_like(C), torch.empty_like(out), torch.empty_like(inn)) for _ in range(6)]
        made.append((p, C, out, inn, outs, torch.cuda.Stream()))
    for _, _, _, _, _, st in made:
        st.wait_stream(torch.cuda.current_stream())
    for i in range(6):
        for p, _, _, _, outs, st in made:
            with torch.cuda.stream(st):
                for _ in range(1 if p.n > 1000 else 20):
                    E, o, x = outs[i]
                    p.execute_sizes(E, out=o, inn=x)
    torch.cuda.synchronize()
    for p, C, out, inn, outs, _ in made:
        for E, o, x in outs:
            assert torch.equal(E, C) and torch.equal(o, out) and torch.equal(x, inn), p.n
        p.close()


@pytest.mark.parametrize("n", [700, 12_000, 25_000])
def test_captured_sizes_replay_after_other_calls(n):
    # a graph holds the launches of a plan and nothing of the context's scratch,
    # which later calls replace
    p = tn.Plan(n, *case("uniform", n, 3, 9950 + n))
    other = tn.Plan(40_000, *T.uniform_pairs(40_000, 40_000, 400, seed=9960))
    wC, wout, winn = (a.clone() for a in p.execute_sizes(slice_words=1))
    C, out, inn = p.execute_sizes()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        p.execute_sizes(C, out=out, inn=inn)
    for sw in (1, 4, 16):  # larger scratch each time
        other.execute_sizes(slice_words=sw)
        for a in (C, out, inn):
            a.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert (host(C) == host(wC)).all()
        assert torch.equal(out, wout) and torch.equal(inn, winn)
    p.close()
    other.close()


@pytest.mark.parametrize("n", [64, 9000, 21_000])
def test_chunks_without_ops(n):
    # self-loops leave nothing to run or to upload, in every chunk or in some
    a = np.arange(60, dtype=np.uint32) % n
    s, d, t = a, a.copy(), np.arange(60, dtype=np.int64)
    for moved in (0, 25):  # events that join two nodes, at the end of the list
        d[60 - moved:] = (a[60 - moved:] + 7) % n
        C, st = tn.build_component_matrix_streamed(n, s, d, t, chunk_events=5)
        assert (host(C) == oracle.reverse_matrix(n, s, d, t)).all() and st["chunks_run"] == 12
        live = tn.Online(n, flags=tn.FORWARD)
        for k in range(0, 60, 20):
            live.insert(s[k:k + 20], d[k:k + 20], t[k:k + 20])
        assert (host(live.C) == oracle.forward_matrix(n, s, d, t)).all()
        live.close()


@pytest.mark.parametrize("first", ["small", "large"])
@pytest.mark.parametrize("off", [None, 1, 4])
@pytest.mark.parametrize("n", [8192, 10_240, 10_241, 16_384, 16_385, 20_407])
def test_streams_of_small_and_large_chunks(n, off, first):
    # batches of few events run on slices in memory, larger ones on word columns,
    # about the number of events that decides, one of them without saturation; the
    # first batch of a network of more than 16,384 nodes decides on the slices
    edge = -(-n // (80 if n <= 16_384 else 48))
    sizes = [1 if first == "small" else -(-n // 12), edge, 3, edge - 1, 4 * n, 2, edge, 7]
    s, d, t = T.uniform_pairs(n, sum(sizes), 3 * sum(sizes), seed=10_000 + n)
    t = np.arange(len(t), dtype=np.int64)
    ctx = tn.get_context()
    live = tn.Online(n, flags=tn.FORWARD)
    try:
        at = 0
        for k, m in enumerate(sizes):
            ctx.saturation(k != off)
            st = live.insert(s[at:at + m], d[at:at + m], t[at:at + m])
            assert st["slice_words"] == (1 if n <= 16_384 or first == "large" else 2)
            at += m
        got = host(live.C)
    finally:
        ctx.saturation(True)
        live.close()
    p = tn.Plan(n, s, d, t, tn.FORWARD)
    assert (got == host(p.execute(slice_words=1))).all()
    p.close()


@pytest.mark.parametrize("n", [4096, 4097, 10_240, 10_241, 16_384, 16_385, 20_407])
def test_plans_of_few_ops(n):
    # about the number of ops from which on a matrix alone is built on word columns;
    # its sizes always come with them
    edge = -(-n * (1 if n <= 16_384 else 2) // 64)
    for m in (0, 1, edge - 1, edge):
        s, d, t = T.uniform_pairs(n, m, max(1, m), seed=10_100 + n + m) if m else \
            (np.zeros(0, np.uint32), np.zeros(0, np.uint32), np.zeros(0, np.int64))
        t = np.arange(m, dtype=np.int64)
        p = tn.Plan(n, s, d, t)
        want = host(p.execute(slice_words=1))
        C = torch.full((n, oracle.words(n) + 3), -1, dtype=torch.int64, device="cuda")
        p.execute(C)
        assert (host(C) == want).all(), m
        wout, winn = tn.component_sizes(C, n)
        C.fill_(-1)
        _, out, inn = p.execute_sizes(C)
        assert (host(C) == want).all() and torch.equal(out, wout) and torch.equal(inn, winn), m
        p.close()


@pytest.mark.parametrize("which", [
    [(4096, 0), (4096, 100), (4097, 0), (4097, 2048), (4097, 2049), (9000, 4499), (9000, 4500), (20_407, 10),
     (20_407, 10_204), (60, 3), (60, 40)],
    [(4096, 0), (4097, 2049), (60, 3), (9000, 4500)], [(4096, 5), (60, 0)], [(60, 3), (4097, 2048)]])
def test_batches_of_few_events(which):
    # about the size and the number of events from which on a network runs on word
    # columns, others as tiles beside them in one launch
    nets = []
    for k, (n, m) in enumerate(which):
        ev = T.uniform_pairs(n, m, max(2, m // 40), seed=10_200 + k) if m else \
            (np.zeros(0, np.uint32), np.zeros(0, np.uint32), np.zeros(0, np.int64))
        nets.append((n, *ev))
    want = []
    for net in nets:
        p = tn.Plan(*net)
        want.append(host(p.execute(slice_words=1)))
        p.close()
    b = tn.Batch(nets)
    ctx = tn.get_context()
    try:
        for sat in (True, False, True):
            ctx.saturation(sat)
            for lead in (0, 5):
                Cs = [torch.full((n, oracle.words(n) + lead), -1, dtype=torch.int64, device="cuda")
                      for n, *_ in nets]
                for _ in range(3):
                    b.execute(Cs)
                    for k, (C, w) in enumerate(zip(Cs, want)):
                        assert (host(C) == w).all(), (k, sat, lead)
                        C.fill_(-1)
    finally:
        ctx.saturation(True)
        b.close()


def test_columns_full_before_a_chunk_move_nothing():
    # node 0 collects nodes 1 to 63 and gives them to all: word column 0 is full,
    # column 1 never; chunks before that in time move column 1 alone
    n = 128
    give = np.tile(np.arange(1, n), 3)
    s = np.concatenate([give, np.arange(1, n), np.zeros(63, int)]).astype(np.uint32)
    d = np.concatenate([np.zeros(4 * (n - 1), int), np.arange(1, 64)]).astype(np.uint32)
    t = np.arange(len(s), dtype=np.int64)
    live = tn.Online(n, flags=tn.DIRECTED)
    ctx = tn.get_context()
    cuts = [len(s), 3 * (n - 1), 2 * (n - 1), n - 1, 0]
    for k, (hi, lo) in enumerate(zip(cuts, cuts[1:])):
        live.insert(s[lo:hi], d[lo:hi], t[lo:hi])
        assert ctx.last_traffic() == ((2 + k) * n,) * 2
    assert (host(live.C) == oracle.reverse_matrix(n, s, d, t, directed=True)).all()
    live.close()


@pytest.mark.parametrize("n,per_node", [(700, 4), (20_000, 0.01), (25_000, 2), (33_000, 1)])
def test_either_sizes_alone(n, per_node):
    # word columns, half columns and slices: out-sizes, in-sizes or none
    p = tn.Plan(n, *case("uniform", n, per_node, 10_300 + n))
    C, out, inn = p.execute_sizes()
    want = host(C).copy()
    ctx, dp = tn.get_context(), tn.api._dp
    for o, i in ((True, False), (False, True), (False, False)):
        C.fill_(-1)
        a, b = torch.full_like(out, -7), torch.full_like(inn, -7)
        rc = tn.lib.tn_plan_execute_sizes(ctx.bind_stream(), p.h, dp(C), C.stride(0), 0, dp(a if o else None),
                                          dp(b if i else None))
        assert rc == 0 and (host(C) == want).all()
        assert torch.equal(a, out) if o else (a == -7).all()
        assert torch.equal(b, inn) if i else (b == -7).all()
    p.close()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 4097, 10_000])
def test_out_sizes_alone_of_any_words(n):
    # lines that end in a part of a word, rows wider than the matrix, whatever was in
    # the array before
    rng = np.random.default_rng(10_400 + n)
    nw = oracle.words(n)
    C = rng.integers(0, 2**64, (n, nw + n % 3), dtype=np.uint64)
    C[:: 3, :nw] = 2**64 - 1
    if n % 64:
        C[:, nw - 1] &= np.uint64(2 ** (n % 64) - 1)
    want = np.bitwise_count(C[:, :nw]).sum(axis=1)
    dev = torch.from_numpy(C.view(np.int64)).cuda()
    for _ in range(2):
        assert (tn.component_sizes(dev, n, inn=False)[0].cpu().numpy() == want).all()
    assert (tn.component_sizes(dev, n)[0].cpu().numpy() == want).all()


@pytest.mark.parametrize("n,m,steps,seed", [(8001, 400_000, 50, 8430), (16_385, 500_000, 100, 8420)])
def test_out_sizes_alone_from_the_slice_state(n, m, steps, seed):
    # slices left all ones beside one that is not, and a plan's own choice
    n, s, d, t, flags = _partial_network(n, m, steps, seed)
    p = tn.Plan(n, s, d, t, flags)
    ctx, dp = tn.get_context(), tn.api._dp
    for sw in (0, 1, 2, 4):
        C, want, _ = p.execute_sizes(slice_words=sw)
        out = torch.full_like(want, -7)
        assert tn.lib.tn_plan_execute_sizes(ctx.bind_stream(), p.h, dp(C), C.stride(0), sw, dp(out), None) == 0
        assert torch.equal(out, want)
    p.close()


@pytest.mark.parametrize("n,per_op", [(4096, 64), (4097, 64), (5120, 64), (5121, 64), (8064, 64), (8065, 32),
                                      (9217, 128), (10_000, 32), (10_240, 128), (10_241, 32), (16_385, 16)])
def test_plans_of_few_ops_without_saturation(n, per_op):
    # about the number of ops from which on a matrix alone is built on word columns,
    # with and without the saturation of full rows
    ctx = tn.get_context()
    edge = -(-n // per_op)
    for m in (0, 1, edge - 1, edge):
        s, d, _ = T.uniform_pairs(n, max(1, m), max(1, m), seed=10_500 + n + m)
        p = tn.Plan(n, s[:m], d[:m], np.arange(m, dtype=np.int64))
        want = host(p.execute(slice_words=1))
        C = torch.empty((n, oracle.words(n) + 3), dtype=torch.int64, device="cuda")
        try:
            for saturation in (True, False):
                ctx.saturation(saturation)
                C.fill_(-1)
                p.execute(C)
                assert (host(C) == want).all(), (m, saturation)
                C.fill_(-1)
                _, out, inn = p.execute_sizes(C)
                assert (host(C) == want).all(), (m, saturation)
                assert torch.equal(out, tn.component_sizes(C, n, inn=False)[0]), (m, saturation)
        finally:
            ctx.saturation(True)
            p.close()
