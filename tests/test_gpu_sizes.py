"""Component sizes (row and column popcounts of a bit matrix, one pass) at the
edges of the kernel's lane groups, rounds and column blocks, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2307_04890_amd as tn  # noqa: E402


def _random_matrix(n, ld, seed):
    """An (n, ld) bit matrix with its padding bits 0, and its dense bits."""
    g = np.random.default_rng(seed)
    dense = g.random((n, n)) < g.random(n)[None, :]
    dense[:, g.integers(0, n)] = True
    packed = np.zeros((n, ld * 8), dtype=np.uint8)
    packed[:, :(n + 7) // 8] = np.packbits(dense, axis=1, bitorder="little")
    return packed.view(np.int64), dense


# lane groups of 8 lanes up to 512 columns, 16 to 1024, 32 to 2048, 64 above;
# rounds of 16 steps x 64 / lanes rows; two column blocks from 4097
@pytest.mark.parametrize("n,pad", [(1, 0), (63, 1), (64, 0), (65, 3), (127, 0), (128, 5), (512, 0), (513, 0),
                                   (1000, 7), (1024, 0), (1025, 0), (2049, 2), (4096, 0), (4097, 0), (5003, 1)])
def test_sizes_match_numpy(n, pad):
    host, dense = _random_matrix(n, (n + 63) // 64 + pad, seed=n)
    C = torch.from_numpy(host).cuda()
    want_out, want_in = dense.sum(axis=1), dense.sum(axis=0)
    out, inn = tn.component_sizes(C, n)
    assert (out.cpu().numpy() == want_out).all() and (inn.cpu().numpy() == want_in).all()
    # each alone
    out, none = tn.component_sizes(C, n, inn=False)
    assert none is None and (out.cpu().numpy() == want_out).all()
    none, inn = tn.component_sizes(C, n, out=False)
    assert none is None and (inn.cpu().numpy() == want_in).all()


def test_sizes_of_a_full_matrix_reach_every_counter_plane():
    # every column counter ends at the rows of its wavefront, the largest
    # value its bit planes take
    n = 70_001
    nw = (n + 63) // 64
    C = torch.full((n, nw), -1, dtype=torch.int64, device="cuda")
    C[:, nw - 1] = (1 << (n % 64)) - 1
    C[5] = 0
    out, inn = tn.component_sizes(C, n)
    assert (inn == n - 1).all()
    assert out[5] == 0 and (out[:5] == n).all() and (out[6:] == n).all()
