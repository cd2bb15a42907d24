"""Host input and results around the size from which they move through pinned
slots on several threads (16 MiB, in chunks of 2 MiB): the same bytes as through
device memory, also from several threads at once."""

import threading

import numpy as np
import pytest

import readsim
import paper_2401_02756_amd as dbg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K = 31
STAGED = 16 << 20


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def make(vertices, read_bytes, seed):
    """Reads of 1000 bases that cover a random genome of about that many vertices."""
    rng = np.random.default_rng(seed)
    genome = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, vertices + K)]
    reads = [genome.tobytes()]
    left = read_bytes - len(genome)
    while left > 0:
        n = min(1000, left)
        at = int(rng.integers(0, vertices - n))
        reads.append(genome[at:at + n].tobytes())
        left -= n
    return readsim.reads_from_strings(reads, K)


def in_order(keys, counts):
    order = np.argsort(keys, kind="stable")
    return keys[order], counts[order]


def check(rs):
    with dbg.Graph(expected_vertices=len(rs.reads), flags=dbg.F_BINNED) as h, \
            dbg.Graph(expected_vertices=len(rs.reads), flags=dbg.F_BINNED) as d:
        d.build_device(torch.from_numpy(rs.reads).cuda(), torch.from_numpy(rs.offsets.astype(np.int64)).cuda(), K)
        d.sync()
        n = d.vertex_count()
        keys = torch.empty(n, dtype=torch.int64, device="cuda")
        counts = torch.empty((n, 4), dtype=torch.int32, device="cuda")
        assert d.extract_device(keys, counts) == n
        want = in_order(keys.cpu().numpy().view(np.uint64), counts.cpu().numpy().view(np.uint32))
        for rep in range(2):
            h.reset()
            h.build(rs.reads, rs.offsets, K)
            got = in_order(*h.extract())
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("vertices,read_bytes", [
    (STAGED // 24 - 3000, STAGED - 200_000),   # results and input under
    (STAGED // 24 + 1, STAGED - 200_000),      # results just over
    (200_000, STAGED + 1),                     # input over
    (1_500_000, 2 * STAGED + 12_345),          # both, several chunks
])
def test_sizes(vertices, read_bytes):
    print("[case] %d vertices, %d bytes of reads" % (vertices, read_bytes), flush=True)
    check(make(vertices, read_bytes, vertices))


def test_threads():
    print("[case] three threads", flush=True)
    sets = [make(800_000 + 1000 * i, STAGED + 1_000_003 * i, i) for i in range(3)]
    errors = []

    def run(rs):
        try:
            check(rs)
        except BaseException as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=run, args=(rs,)) for rs in sets]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
