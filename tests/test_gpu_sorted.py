"""The partition by sorted tiles (automatic scatter shapes) at the sizes where
it can go wrong: tiles filled to within one window, tiles whose reads or bases
overflow their LDS room, reads too short for a window between tiles, bytes
checked that no window covers, one-level and two-level tables, segments fed by
one long piece or by thousands of one-record pieces.  All graphs equal the
oracle's, bit for bit."""

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RNG = np.random.default_rng(0x50F7)
K = 21
ONE_LEVEL, TWO_LEVEL = 200_000, 1_200_000  # expected vertices: 196 segments, 1172 segments


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def letters(n):
    return np.frombuffer(b"ACGT", np.uint8)[RNG.integers(0, 4, int(n))].tobytes()


def tiled(windows):
    """One read with that many windows."""
    return [letters(windows + K - 2)]


def short_between(n):
    """Reads of a few hundred bases, each followed by reads without a window."""
    out = []
    for _ in range(n):
        out.append(letters(RNG.integers(K, 400)))
        out += [letters(RNG.integers(0, K)) for _ in range(int(RNG.integers(0, 9)))]
    return out


def cases():
    t = 2048  # records of a small input's tile
    for w in (2, t - 1, t, t + 1, 2 * t, 3 * t + 5):
        yield "one read of %d windows" % w, tiled(w)
    yield "two reads meeting at a tile's end", tiled(t - 7) + tiled(7) + tiled(t)
    yield "reads of exactly k", [letters(K) for _ in range(5000)]  # more reads a tile than are staged
    yield "short reads between", short_between(600)
    # more bases a tile than are staged: thousands of windowless reads inside one
    yield "a tile of windowless reads", tiled(500) + [letters(K - 1) for _ in range(9000)] + tiled(900)
    yield "one letter", [b"A" * 40_000, letters(3000)]  # every record of a tile in one piece
    yield "two letters", [b"AC" * 9000, b"acgt" * 2000]


CASES = list(cases())


@pytest.mark.parametrize("vertices", [ONE_LEVEL, TWO_LEVEL], ids=["one-level", "two-level"])
@pytest.mark.parametrize("name,reads", CASES, ids=[c[0].replace(" ", "-") for c in CASES])
def test_tiles_and_reads(name, reads, vertices):
    for k in (K, 45):
        rs = readsim.reads_from_strings(reads, k)
        if k > 32:
            hi, lo, counts = oracle.build_graph_wide(rs.reads, rs.offsets, k)
        else:
            ref = oracle.build_graph(rs.reads, rs.offsets, k)
        for rep in range(2):
            print("[case] %s, k=%d, %d vertices expected, build %d" % (name, k, vertices, rep), flush=True)
            with dbg.Graph(expected_vertices=vertices, flags=dbg.F_BINNED) as g:
                # unaligned reads: the slice starts at an odd byte of the buffer
                buf = torch.from_numpy(np.concatenate([np.full(5, 78, np.uint8), rs.reads])).cuda()
                off = torch.from_numpy(rs.offsets.astype(np.int64)).cuda()
                g.build_device(buf[5:] if rep else torch.from_numpy(rs.reads).cuda(), off, k)
                g.sync()
                if k > 32:
                    keys, got = g.extract_sorted()
                    assert np.array_equal(keys.reshape(-1, 2)[:, 0], hi) and np.array_equal(keys.reshape(-1, 2)[:, 1], lo)
                    assert np.array_equal(got, counts)
                else:
                    records.assert_exact(ref, g.extract(), name)


@pytest.mark.parametrize("vertices", [ONE_LEVEL, TWO_LEVEL], ids=["one-level", "two-level"])
def test_every_byte_is_checked(vertices):
    """A bad byte is found wherever it is: in a window, in a read without one
    (before, between and after the tiles), and where no read has a window; the
    graph stays as it was."""
    inner = tiled(2048) + [letters(K - 2)] * 3 + tiled(3000) + [letters(5)] * 3
    sets = [([letters(7)] + inner, i) for i in range(len(inner) + 1)]
    sets += [([letters(9)] * 50, i) for i in (0, 31, 49)]
    ok = readsim.reads_from_strings(inner, K)
    ref = oracle.build_graph(ok.reads, ok.offsets, K)
    with dbg.Graph(expected_vertices=vertices, flags=dbg.F_BINNED) as g:
        g.build(ok.reads, ok.offsets, K)
        for reads, i in sets:
            for at in (0, len(reads[i]) // 2, len(reads[i]) - 1):
                bad = list(reads)
                bad[i] = bad[i][:at] + b"N" + bad[i][at + 1:]
                rs = readsim.reads_from_strings(bad, K)
                with pytest.raises(dbg.DbgError) as e:
                    g.build(rs.reads, rs.offsets, K)
                assert e.value.code == dbg.E_BASE, (i, at)
        records.assert_exact(ref, g.extract(), "after rejected builds")


def test_thousands_of_small_pieces():
    """A two-level bucket whose records come one or two to a tile: its level-2
    tiles have more pieces than fit in LDS."""
    rare = [letters(K + 1) for _ in range(40)]
    reads = []
    for _ in range(2400):
        reads += [b"A" * 8000] + [rare[int(x)] for x in RNG.integers(0, len(rare), 3)]
    rs = readsim.reads_from_strings(reads, K)
    ref = oracle.build_graph(rs.reads, rs.offsets, K)
    with dbg.Graph(expected_vertices=TWO_LEVEL, flags=dbg.F_BINNED) as g:
        g.build(rs.reads, rs.offsets, K)
        records.assert_exact(ref, g.extract(), "rare records")


def test_batch_of_both_kinds():
    """One- and two-level tables, an instance without a window and a rejected
    one in one pass."""
    sets = [short_between(40), tiled(9000), [letters(6)] * 20, tiled(100) + [b"ACGTNACGT" * 5], tiled(70_000)]
    sizes = [ONE_LEVEL, TWO_LEVEL, ONE_LEVEL, ONE_LEVEL, TWO_LEVEL]
    gs = [dbg.Graph(expected_vertices=v, flags=dbg.F_BINNED) for v in sizes]
    rs = [readsim.reads_from_strings(s, K) for s in sets]
    for rep in range(2):  # the second build adds to the first
        st = dbg.build_batch(gs, [(x.reads, x.offsets, K) for x in rs])
        assert st == [0, 0, 0, dbg.E_BASE, 0]
        for j, (g, x) in enumerate(zip(gs, rs)):
            if j == 3:
                assert g.vertex_count() == 0
                continue
            keys, counts = oracle.build_graph(x.reads, x.offsets, K)
            records.assert_exact((keys, counts * (rep + 1)), g.extract(), "set %d, build %d" % (j, rep))
    for g in gs:
        g.close()


@pytest.mark.parametrize("want,slots", [(3, 4), (5, 6), (10, 12), (21, 25), (993, 1024)])
def test_small_tables_round_up_as_large_ones(want, slots):
    """A one-level table has the segments that two levels would give it, so that
    an estimate which was just too low still fits."""
    n = int(want * 2048 * 1.02) if want < 900 else int(want * 2048 * 0.9)
    read = letters(n + K - 2)
    rs = readsim.reads_from_strings([read], K)
    print("[case] %d segments asked for, %d vertices" % (want, n), flush=True)
    with dbg.Graph(capacity=want * 2048, flags=dbg.F_BINNED) as g:
        assert g.stats()["capacity"] == slots * 2048
        g.build(rs.reads, rs.offsets, K)
        records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, K), g.extract(), "capacity")


@pytest.mark.parametrize("segments", [1, 2, 6, 25, 56, 110])
@pytest.mark.parametrize("k", [21, 45])
def test_few_segments_read_deeply(k, segments):
    """Many tiles over few segments: long pieces are read in rows of 64 records
    (up to 64 segments of one-word keys, 32 of two-word ones).  Built twice, the
    second time into a table that holds the vertices."""
    rng = np.random.default_rng([k, segments])
    n = segments * 900
    genome = letters(n + k)
    reads = [genome]
    for _ in range(22_000):
        m = int(rng.integers(k - 3, 200))
        at = int(rng.integers(0, max(1, n - m)))
        reads.append(genome[at:at + m])
    rs = readsim.reads_from_strings(reads, k)
    for flags in (0, dbg.F_STATS):
        print("[case] k=%d, %d segments, flags %d" % (k, segments, flags), flush=True)
        with dbg.Graph(capacity=segments * 2048, flags=dbg.F_BINNED | flags) as g:
            for rep in (1, 2):
                g.build(rs.reads, rs.offsets, k)
                if k > 32:
                    hi, lo, counts = oracle.build_graph_wide(rs.reads, rs.offsets, k)
                    keys, got = g.extract_sorted()
                    keys = keys.reshape(-1, 2)
                    assert np.array_equal(keys[:, 0], hi) and np.array_equal(keys[:, 1], lo)
                    assert np.array_equal(got, rep * counts)
                else:
                    keys, counts = oracle.build_graph(rs.reads, rs.offsets, k)
                    records.assert_exact((keys, counts * rep), g.extract(), "build %d" % rep)
            if flags:
                st = g.probe_stats()
                assert st["cas_attempts"] - st["cas_lost"] == g.vertex_count() and st["lookups"] == g.stats()["windows"]


@pytest.mark.parametrize("windows", [0.3, 3, 40, 700, 1700, 2600])
@pytest.mark.parametrize("k", [21, 45])
@pytest.mark.parametrize("vertices", [ONE_LEVEL, TWO_LEVEL], ids=["one-level", "two-level"])
def test_segments_of_few_records(vertices, k, windows):
    """From nearly empty segments, planned four together, to those of two units;
    the second part is added to what the first left in them."""
    total = int(windows * -(-2 * vertices // 2048))
    rng = np.random.default_rng([vertices, k, total])
    genome = letters(max(k + 50, min(total, vertices) // 2))
    parts = []
    for _ in range(2):
        reads, left = [], total
        while left > 0:
            n = int(rng.integers(2, 120))
            at = int(rng.integers(0, len(genome) - k))
            reads.append(genome[at:at + min(n, left) + k - 2])
            left -= n
        parts.append(reads)
    first, both = (readsim.reads_from_strings(p, k) for p in (parts[0], parts[0] + parts[1]))
    second = readsim.reads_from_strings(parts[1], k)
    print("[case] k=%d, %d vertices, %g windows a segment" % (k, vertices, windows), flush=True)
    with dbg.Graph(expected_vertices=vertices, flags=dbg.F_BINNED) as g:
        for new, rs in ((first, first), (second, both)):
            g.build(new.reads, new.offsets, k)
            if k > 32:
                hi, lo, counts = oracle.build_graph_wide(rs.reads, rs.offsets, k)
                keys, got = g.extract_sorted()
                keys = keys.reshape(-1, 2)
                assert np.array_equal(keys[:, 0], hi) and np.array_equal(keys[:, 1], lo) and np.array_equal(got, counts)
            else:
                records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, k), g.extract(), "build")
