"""Tiles of the first partition whose reads or bases do not fit their LDS room:
reads of one or two windows, and windowless reads between them.  Their windows
are taken from the ASCII reads directly, sixteen bytes at a time; the reads here
end at the buffer's last byte, start at odd addresses, and leave tiles of 2048
records (small inputs) and of 64 KB (above 2 MB).  All graphs equal the
oracle's, bit for bit."""

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SMALL, MID = 300_000, 2_300_000  # bases


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def reads_of(lengths, seed):
    rng = np.random.default_rng(seed)
    text = np.frombuffer(b"ACGTacgt", np.uint8)[rng.integers(0, 8, int(np.sum(lengths)))].tobytes()
    ends = np.cumsum(lengths)
    return [text[e - n:e] for n, e in zip(lengths, ends)]


def exact(k, bases, rng):
    return np.full(bases // k, k)


def mixed(k, bases, rng):
    return rng.integers(max(1, k // 3), k + 5, 2 * bases // (k + 5 + max(1, k // 3)))


def sparse(k, bases, rng):  # seldom a window, then a few; long runs without
    n = 2 * bases // k
    out = rng.integers(0, k, n)
    out[rng.random(n) < 0.02] = k + 20
    out[n // 3:n // 2] = k - 1
    return out


def check(rs, k, what, at=0):
    buf = torch.from_numpy(np.concatenate([np.full(at, 78, np.uint8), rs.reads])).cuda()
    off = torch.from_numpy(rs.offsets.astype(np.int64)).cuda()
    print("[case] %s, k=%d, %d reads, at byte %d" % (what, k, rs.n_reads, at), flush=True)
    with dbg.Graph(expected_vertices=max(1000, rs.total_bases), flags=dbg.F_BINNED) as g:
        g.build_device(buf[at:], off, k)
        g.sync()
        if k > 32:
            hi, lo, counts = oracle.build_graph_wide(rs.reads, rs.offsets, k)
            keys, got = g.extract_sorted()
            keys = keys.reshape(-1, 2)
            assert np.array_equal(keys[:, 0], hi) and np.array_equal(keys[:, 1], lo) and np.array_equal(got, counts)
        else:
            records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, k), g.extract(), what)


@pytest.mark.parametrize("bases", [SMALL, MID], ids=["small", "mid"])
@pytest.mark.parametrize("lengths", [exact, mixed, sparse])
@pytest.mark.parametrize("k", [2, 16, 17, 21, 31, 33, 45, 63])
def test_few_windows_a_read(k, lengths, bases):
    rng = np.random.default_rng([k, bases])
    rs = readsim.reads_from_strings(reads_of(lengths(k, bases, rng), k), k)
    check(rs, k, lengths.__name__, at=0 if bases == SMALL else 5)


@pytest.mark.parametrize("k", [21, 63])
def test_bad_bytes_are_found(k):
    """In the first and last byte of reads at the start, inside and end of such
    tiles, with and without a window; and only there: the bytes behind the last
    read are not looked at."""
    rng = np.random.default_rng(k)
    reads = reads_of(mixed(k, 200_000, rng), 3)
    ok = readsim.reads_from_strings(reads, k)
    n = len(reads)
    with dbg.Graph(expected_vertices=ok.total_bases, flags=dbg.F_BINNED) as g:
        off = torch.from_numpy(ok.offsets.astype(np.int64)).cuda()
        for r in (0, 1, n // 2, n // 2 + 1, n // 2 + 2, n - 2, n - 1):
            for at in {0, len(reads[r]) - 1}:
                print("[case] k=%d, read %d of %d bases, byte %d" % (k, r, len(reads[r]), at), flush=True)
                bad = ok.reads.copy()
                bad[int(ok.offsets[r]) + at] = ord("N")
                g.build_device(torch.from_numpy(bad).cuda(), off, k)
                with pytest.raises(dbg.DbgError) as e:
                    g.sync()
                assert e.value.code == dbg.E_BASE
        assert g.vertex_count() == 0
        buf = torch.full((ok.total_bases + 64,), 78, dtype=torch.uint8, device="cuda")
        buf[32:32 + ok.total_bases] = torch.from_numpy(ok.reads).cuda()
        g.build_device(buf[32:32 + ok.total_bases], off, k)
        g.sync()
        assert g.stats()["inserts"] == int(np.maximum(ok.lengths() - k + 1, 0).sum())
