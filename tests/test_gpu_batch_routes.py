"""Batches whose graphs ask for different partitions.  The first graph that
runs decides the launch for all: tables of one level then go through the
shaped scatters, and tables laid out for two levels through the sorted tiles.
Both take the same record buffers."""

import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
import readsim
import records
import paper_2401_02756_amd as dbg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield


def reads_of(vertices, k, seed):
    rng = np.random.default_rng(seed)
    genome = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, vertices + k)].tobytes()
    return readsim.reads_from_strings([genome] + [genome[i:i + 100] for i in rng.integers(0, vertices, 300)], k)


@pytest.mark.parametrize("shapes", [(1, 1), (2, 2), (3, 3), (4, 3), (0, 2)])
@pytest.mark.parametrize("shaped_first", [True, False])
def test_shaped_and_automatic_graphs_in_one_batch(shaped_first, shapes):
    """Tables of 1 to 1024 segments in one level (automatic) and in two (set
    shapes), and one beyond, in both orders; built twice."""
    sizes = [1, 7, 100, 1000, 30, 1500]
    sets = [reads_of(700 * n if n < 1000 else 300_000, (21, 31)[i % 2], i) for i, n in enumerate(sizes)]
    ks = [(21, 31)[i % 2] for i in range(len(sizes))]
    gs = []
    for i, n in enumerate(sizes):
        set_shape = (i % 2 == 0) == shaped_first
        kw = dict(bin_shape1=shapes[0], bin_shape2=shapes[1]) if set_shape else {}
        gs.append(dbg.Graph(capacity=2048 * n, flags=dbg.F_BINNED, **kw))
    for rep in (1, 2):
        print("[case] shapes %s, shaped first %s, build %d" % (shapes, shaped_first, rep), flush=True)
        assert dbg.build_batch(gs, [(x.reads, x.offsets, k) for x, k in zip(sets, ks)]) == [0] * len(gs)
        for j, (g, x, k) in enumerate(zip(gs, sets, ks)):
            keys, counts = oracle.build_graph(x.reads, x.offsets, k)
            records.assert_exact((keys, counts * rep), g.extract(), "graph %d of %d segments, build %d" % (j, sizes[j], rep))
    for g in gs:
        g.close()


_MEMORY_CHILD = r"""
import sys
import numpy as np
import torch
sys.path.insert(0, sys.argv[1])
import paper_2401_02756_amd as dbg

torch.cuda.init()
n = 200_000_000
reads = torch.from_numpy(np.frombuffer(b"ACGT", np.uint8)[np.random.default_rng(1).integers(0, 4, 1000)]).cuda().repeat(n // 1000)
off = torch.arange(0, n + 1, 1000, device="cuda")
torch.cuda.synchronize()

def left(**kw):
    with dbg.Graph(capacity=1 << 23, flags=dbg.F_BINNED, **kw) as a, dbg.Graph(capacity=1 << 23, flags=dbg.F_BINNED, **kw) as b:
        assert dbg.build_batch_device([a, b], [0, 1000, n // 1000], [21, 21], reads, off) == [0, 0]
    return torch.cuda.mem_get_info()[0]

left()
print(left() - left(bin_shape1=3, bin_shape2=3))
"""


def test_both_routes_take_the_same_record_buffers():
    """A batch context that has taken one route does not hold a second pair of
    record buffers (16 bytes a base) for the other."""
    print("[case] 200 MB of reads, both routes", flush=True)
    out = subprocess.run([sys.executable, "-c", _MEMORY_CHILD, ROOT], capture_output=True, text=True, timeout=150, cwd=ROOT)
    assert out.returncode == 0, out.stderr[-2000:]
    more = int(out.stdout.strip().splitlines()[-1])
    assert more < 8 * 200_000_000, more
