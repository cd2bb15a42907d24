"""Level-2 tiles with more pieces than their table in LDS has entries (2048):
one bucket gets a few records from each of some thousand level-1 tiles.  The
bucket arithmetic of the kernels is repeated here, so that the test cannot stop
reaching the case unnoticed."""

import math

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CODE = {"A": 0, "C": 1, "T": 2, "G": 3}
M64 = (1 << 64) - 1


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def mix64(z):
    z ^= z >> 30
    z = z * 0xBF58476D1CE4E5B9 & M64
    z ^= z >> 27
    z = z * 0x94D049BB133111EB & M64
    return z ^ z >> 31


def bucket(text, d1):
    """The level-1 bucket of a window's (k-1)-mer."""
    key = 0
    for c in text:
        key = key << 2 | CODE[c]
    if len(text) < 32:
        x = key * 0x0E3779B97F4A7C15 & (1 << 60) - 1
        x ^= x >> 30
    else:
        hi, lo = key >> 64, key & M64
        x = hi ^ ((lo ^ mix64(hi)) * 0xD1B54A32D192ED03 & M64) >> 4
    return (x >> 28 & 0xFFFFFFFF) * d1 >> 32


@pytest.mark.parametrize("k,tile1,tile2,a_tile", [(21, 8192, 16384, 3), (21, 8192, 16384, 7), (45, 4096, 8192, 3)])
def test_more_pieces_than_lds_holds(k, tile1, tile2, a_tile):
    rng = np.random.default_rng([k, a_tile])
    rare = "".join("ACGT"[i] for i in rng.integers(0, 4, k))  # one k-mer, two windows
    n_tiles = 2600
    between = tile1 // a_tile - 2  # windows between two of the rare read
    reads = [b"A" * (between + k - 2), rare.encode()] * (n_tiles * a_tile)
    rs = readsim.reads_from_strings(reads, k)
    with dbg.Graph(expected_vertices=1_200_000, flags=dbg.F_BINNED) as g:
        parts = g.stats()["capacity"] // 2048
        fan = -(-parts // math.ceil(math.sqrt(parts)))
        d1 = -(-parts // fan)
        assert d1 * fan == parts and parts > 1024
        # the rare read's first window, and where it lies among the windows
        first = np.arange(n_tiles * a_tile) * (between + 2) + between
        b = bucket(rare[:-1], d1)
        assert b not in (bucket("A" * (k - 1), d1), bucket(rare[1:], d1))
        tiles = first // tile1
        most = max(np.unique(tiles[i:i + tile2]).size for i in range(0, tiles.size, tile2))
        print("[case] k=%d, %d windows, %d buckets, %d pieces in a tile" % (k, 2 * tiles.size + tiles.size * between, d1, most),
              flush=True)
        assert most > 2048
        g.build(rs.reads, rs.offsets, k)
        st = g.stats()
        assert (st["sort_tiles"] & 0xffff, st["sort_tiles"] >> 16) == (tile1, tile2)
        if k > 32:
            hi, lo, counts = oracle.build_graph_wide(rs.reads, rs.offsets, k)
            keys, got = g.extract_sorted()
            keys = keys.reshape(-1, 2)
            assert np.array_equal(keys[:, 0], hi) and np.array_equal(keys[:, 1], lo) and np.array_equal(got, counts)
        else:
            records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, k), g.extract(), "many pieces")
