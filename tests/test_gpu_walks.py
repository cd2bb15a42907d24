"""Contigs whose walks end around the letters that the first pass keeps (32 to a
word, 64 in all), loops entered and closed around there, and contigs longer than
what a workgroup puts together, among short ones.  Exact on the sorted strings."""

import numpy as np
import pytest

import oracle
import readsim
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = (1, 2, 31, 32, 33, 34, 63, 64, 65, 66, 67, 97, 130)


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def sequence(rng, n):
    return np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, n)].tobytes()


def lines(rng, k):
    return [sequence(rng, k - 1 + e) for e in EDGES for _ in range(60)]


def loops(rng, k):
    """A tail of `a` edges into a loop of `b`."""
    out = []
    for a in (1, 2, 31, 33, 64, 65):
        for b in (1 + k, 31 + k, 64, 65, 90):
            tail, ring = sequence(rng, a + k), sequence(rng, b)
            out.append(tail + ring + ring[:k])
    return out


def long_ones(rng, k):
    """A contig longer than a workgroup's room, alone and between short ones."""
    return [sequence(rng, 30_000)] + [sequence(rng, k + 40) for _ in range(700)] + [sequence(rng, 26_000)]


@pytest.mark.parametrize("k,flags", [(21, dbg.F_BINNED), (31, dbg.F_BINNED), (31, dbg.F_BINNED | dbg.F_ENTRY32),
                                     (31, 0), (32, 0)])
@pytest.mark.parametrize("make", [lines, loops, long_ones], ids=lambda f: f.__name__)
def test_walks(make, k, flags):
    print("[case] %s, k=%d, flags %d" % (make.__name__, k, flags), flush=True)
    rs = readsim.reads_from_strings(make(np.random.default_rng(k), k), k)
    keys, counts = oracle.build_graph(rs.reads, rs.offsets, k)
    want = oracle.contig_strings(*oracle.contigs(keys, counts, k))
    assert len(want) > 20 or make is long_ones
    with dbg.Graph(flags=flags) as g:
        g.build(rs.reads, rs.offsets, k)
        assert oracle.contig_strings(*g.contigs()) == want
