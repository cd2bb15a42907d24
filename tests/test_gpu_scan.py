"""The window scan at its edges: read counts around its blocks of 8192 reads and
its rows of 64, and batches whose graphs share a wavefront's reads, a row of them
or a block.  All graphs equal the oracle's, bit for bit."""

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K = 21
BLOCK, ROW = 8192, 64
MODES = {"direct": 0, "binned": dbg.F_BINNED}


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def read_set(n, seed):
    """n reads of 0 to 40 bases out of one short genome; one of 3000 among many."""
    rng = np.random.default_rng(seed)
    genome = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, 4000)]
    lens = rng.integers(0, 41, n)
    if n > 1000:
        lens[n // 2] = 3000
    at = rng.integers(0, 1000, n)
    return readsim.reads_from_strings([genome[a:a + l].tobytes() for a, l in zip(at, lens)], K)


def assert_graph(g, rs):
    records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, K), g.extract(), "%d reads" % (len(rs.offsets) - 1))


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("n", [1, ROW, ROW + 1, BLOCK - 1, BLOCK, BLOCK + 1, 2 * BLOCK, 3 * BLOCK + 65])
def test_read_counts(n, mode):
    rs = read_set(n, n)
    with dbg.Graph(expected_vertices=20_000, flags=MODES[mode]) as g:
        print("[case] %d reads, %s" % (n, mode), flush=True)
        g.build(rs.reads, rs.offsets, K)
        assert_graph(g, rs)


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("sizes", [
    (1,) * 70,                            # more graphs than lanes
    (ROW, ROW - 1, ROW + 1, 2, 3, 8 * ROW),
    (BLOCK, 1, BLOCK - 1, 5, 2 * BLOCK + 7),
], ids=["one read each", "rows", "blocks"])
def test_batches(sizes, mode):
    sets = [read_set(n, 1000 + i) for i, n in enumerate(sizes)]
    print("[case] batch of %s reads, %s" % (sizes, mode), flush=True)
    graphs = [dbg.Graph(expected_vertices=20_000, flags=MODES[mode]) for _ in sets]
    assert dbg.build_batch(graphs, [(s.reads, s.offsets, K) for s in sets]) == [0] * len(sets)
    for g, s in zip(graphs, sets):
        assert_graph(g, s)
        g.close()
