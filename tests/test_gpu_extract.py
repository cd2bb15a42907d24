"""Extraction of binned tables of one segment, of one group of segments (1024),
of one segment more and of several groups, short keys and long: the oracle's
vertices, each once, the same order twice, and not one word behind the last."""

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


@pytest.mark.parametrize("k", [21, 45])
@pytest.mark.parametrize("segments", [1, 2, 1024, 1025, 2500])
def test_segments(segments, k):
    print("[case] %d segments, k=%d" % (segments, k), flush=True)
    rng = np.random.default_rng(segments)
    genome = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, min(700 * segments, 150_000))].tobytes()
    rs = readsim.reads_from_strings([genome], k)
    with dbg.Graph(capacity=2048 * segments, flags=dbg.F_BINNED) as g:
        g.build(rs.reads, rs.offsets, k)
        n = g.vertex_count()
        words = 1 if k < 32 else 2
        outs = []
        for _ in range(2):
            keys = torch.full(((n + 1) * words,), -1, dtype=torch.int64, device="cuda")
            counts = torch.full((n + 1, 4), -1, dtype=torch.int32, device="cuda")
            assert g.extract_device(keys[:n * words] if words == 1 else keys[:n * 2].view(n, 2), counts[:n]) == n
            assert (keys[n * words:] == -1).all() and (counts[n] == -1).all()
            outs.append((keys.cpu().numpy()[:n * words], counts.cpu().numpy()[:n]))
        assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
        keys, counts = outs[0][0].view(np.uint64), outs[0][1].view(np.uint32)
        if words == 1:
            records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, k), (keys, counts), "%d segments" % segments)
        else:
            hi, lo, want = oracle.build_graph_wide(rs.reads, rs.offsets, k)
            order = np.lexsort((keys[1::2], keys[::2]))
            assert np.array_equal(keys[::2][order], hi) and np.array_equal(keys[1::2][order], lo)
            assert np.array_equal(counts[order], want)


@pytest.mark.parametrize("k", [21, 45])
@pytest.mark.parametrize("segments,vertices", [(2500, 1), (2500, 63), (2500, 9_000), (9000, 150_000), (9000, 156_000),
                                               (70_001, 40_000)])
def test_many_segments_of_few_vertices(segments, vertices, k):
    """Around the line (17 vertices a segment for 9000 of them) from which on a
    workgroup takes one segment, not 64; the last segments of a table, too."""
    print("[case] %d segments, %d vertices, k=%d" % (segments, vertices, k), flush=True)
    rng = np.random.default_rng(vertices)
    genome = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, vertices + k)].tobytes()
    rs = readsim.reads_from_strings([genome[:vertices + k - 2]] if vertices > 1 else [genome[:k]], k)
    with dbg.Graph(capacity=2048 * segments, flags=dbg.F_BINNED) as g:
        g.build(rs.reads, rs.offsets, k)
        n, words = g.vertex_count(), 1 if k < 32 else 2
        keys = torch.full(((n + 1) * words,), -1, dtype=torch.int64, device="cuda")
        counts = torch.full((n + 1, 4), -1, dtype=torch.int32, device="cuda")
        assert g.extract_device(keys[:n * words] if words == 1 else keys[:n * 2].view(n, 2), counts[:n]) == n
        assert (keys[n * words:] == -1).all() and (counts[n] == -1).all()
        keys, counts = keys.cpu().numpy()[:n * words].view(np.uint64), counts.cpu().numpy()[:n].view(np.uint32)
    if words == 1:
        records.assert_exact(oracle.build_graph(rs.reads, rs.offsets, k), (keys, counts), "few vertices")
    else:
        hi, lo, want = oracle.build_graph_wide(rs.reads, rs.offsets, k)
        order = np.lexsort((keys[1::2], keys[::2]))
        assert np.array_equal(keys[::2][order], hi) and np.array_equal(keys[1::2][order], lo)
        assert np.array_equal(counts[order], want)
