"""The tiles that a build by sorted tiles takes (dbg_stats sort_tiles), by the
input's size and the table's, and the edges of each: tiles filled to within one
window, reads that meet at a tile's end, windowless reads between, one letter.
All graphs equal the oracle's, bit for bit."""

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# name, slots of the table, least bases of the input, tiles for one- and two-word records
SHAPES = [
    ("small", 300 * 2048, 0, {21: (2048, 0), 45: (2048, 0)}),
    ("small-two-level", 2000 * 2048, 0, {21: (2048, 16384), 45: (2048, 8192)}),
    ("mid", 1000 * 2048, 2_200_000, {21: (8192, 0), 45: (4096, 0)}),
    ("mid-two-level", 5000 * 2048, 2_200_000, {21: (8192, 16384), 45: (4096, 8192)}),
    # more than 384 buckets of the first level: from 384 * 384 segments on
    ("large", 200_000 * 2048, 2_200_000, {21: (16384, 16384), 45: (8192, 8192)}),
]


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def letters(rng, n):
    return np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, int(n))].tobytes()


@pytest.mark.parametrize("k", [21, 45])
@pytest.mark.parametrize("name,slots,least,tiles", SHAPES, ids=[s[0] for s in SHAPES])
def test_tile_edges(name, slots, least, tiles, k):
    rng = np.random.default_rng([slots, k])
    t = tiles[k][0]

    def of(windows):
        return letters(rng, windows + k - 2)

    # whole tiles of one read first (few vertices: they have to fit the table), so
    # that what follows starts at a tile's first window
    fill = [of(t)] * -(-least // t)
    edges = {
        "one window short": [of(t - 1)], "full": [of(t)], "one window more": [of(t + 1)],
        "meeting at the end": [of(t - 7), of(7), of(t)],
        "two windows": [of(2)],
        "windowless between": [of(t // 2)] + [letters(rng, k - 1)] * 50 + [of(t // 2 - 1)] + [letters(rng, 3)] * 50 + [of(40)],
        "windowless at the end": [of(t - 1)] + [letters(rng, k - 1)] * (t // 2 + 9),
        "exactly k": [letters(rng, k) for _ in range(t // 2 + 3)],
        "one letter": [b"A" * (3 * t + 5), letters(rng, 500)],
    }
    with dbg.Graph(capacity=slots, flags=dbg.F_BINNED) as g:
        for what, reads in edges.items():
            rs = readsim.reads_from_strings(fill + reads, k)
            print("[case] %s tiles, %s, k=%d, %d bases" % (name, what, k, rs.total_bases), flush=True)
            g.reset()
            g.build(rs.reads, rs.offsets, k)
            st = g.stats()
            assert (st["sort_tiles"] & 0xffff, st["sort_tiles"] >> 16) == tiles[k], st
            if k > 32:
                hi, lo, counts = oracle.build_graph_wide(rs.reads, rs.offsets, k)
                keys, got = g.extract_sorted()
                keys = keys.reshape(-1, 2)
                assert np.array_equal(keys[:, 0], hi) and np.array_equal(keys[:, 1], lo) and np.array_equal(got, counts), what
            else:
                records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, k), g.extract(), what)


def test_shaped_builds_report_no_tiles():
    rs = readsim.make_config(1)
    with dbg.Graph(expected_vertices=200_000, flags=dbg.F_BINNED, bin_shape1=3, bin_shape2=3) as g:
        g.build(rs.reads, rs.offsets, rs.k)
        assert g.stats()["sort_tiles"] == 0
    with dbg.Graph(expected_vertices=900 * 1024, flags=dbg.F_BINNED) as g:  # one level, whose 900 buckets are not a scatter's
        g.build(rs.reads, rs.offsets, rs.k)
        st = g.stats()
        assert st["sort_tiles"] == 2048 and (st["bin_shape1"], st["bin_shape2"]) == (dbg.SHAPE_BIG, dbg.SHAPE_BIG)
