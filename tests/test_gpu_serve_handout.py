"""The serving loop's hand-out of units at the edges of its 64-wide steps: request counts around
64 in one burst, empty files among them, chunks smaller and larger than the files (more units
than blocks, one unit a request), one block and many; and runs of changing size on one context,
whose buffers stay with it between runs."""
import os

import numpy as np
import pytest

from oracle import data as odata
from paper_2109_05366_amd import gfs, runner

pytestmark = pytest.mark.gpu

PAGE = 64 << 10
SIZES = [0, 8, 4096, PAGE, PAGE + 24, 3 * PAGE - 8, 10 * PAGE + 40]


@pytest.fixture(scope="module")
def cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gfs.lib()
    return torch


@pytest.fixture(scope="module")
def files(tmp_path_factory):
    d = tmp_path_factory.mktemp("handout")
    rng = np.random.RandomState(11)
    paths = []
    for i, n in enumerate(SIZES):
        p = os.path.join(d, "f%d.bin" % i)
        rng.randint(0, 256, n, dtype=np.uint8).tofile(p)
        paths.append(p)
    return paths, np.array([odata.file_checksum(p) for p in paths], dtype=np.uint64)


def _run(cache, ids, asked, want, chunk, grid):
    recs, summ = runner.serve(cache, [ids[f] for f in asked], [0] * len(asked), 16 << 20, chunk_bytes=chunk, grid=grid,
                              idle_timeout_s=20.0)
    np.testing.assert_array_equal(recs["result"], np.array(SIZES, dtype=np.int64)[asked])
    np.testing.assert_array_equal(recs["csum"], want[asked])
    assert sorted(recs["seq"]) == list(range(len(asked)))
    assert summ["delivered_bytes"] == int(np.array(SIZES)[asked].sum())


@pytest.mark.parametrize("chunk,grid", [(16 << 10, 0), (1 << 20, 0), (PAGE, 1), (4096 + 16, 3)])
def test_bursts_around_a_wave(files, cuda, chunk, grid):
    paths, want = files
    rng = np.random.RandomState(chunk + grid)
    cfg = runner.make_config(PAGE, 16 << 20, ra_cap_bytes=1 << 20, rpc_slots=16, timeout_s=20)
    with gfs.PageCache(cfg) as cache:
        ids = [cache.open(p) for p in paths]
        for n in (1, 63, 64, 65, 130, 2):
            print(f"[gpu] handout n={n} chunk={chunk} grid={grid}", flush=True)
            _run(cache, ids, rng.randint(0, len(SIZES), n), want, chunk, grid)
        _run(cache, ids, np.zeros(70, dtype=np.int64), want, chunk, grid)   # nothing but empty files
        assert cache.stats()["timeouts"] == 0


def test_two_runs_of_one_context_at_once(files, cuda):
    """Each run has buffers of its own, whichever of them the context keeps."""
    import threading
    torch = cuda
    paths, want = files
    cfg = runner.make_config(PAGE, 16 << 20, ra_cap_bytes=1 << 20, rpc_slots=16, timeout_s=20)
    asked = [np.random.RandomState(s).randint(0, len(SIZES), 40) for s in (1, 2)]
    got, failed = [None, None], []
    with gfs.PageCache(cfg) as cache:
        ids = [cache.open(p) for p in paths]

        def work(i):
            try:
                torch.cuda.set_device(0)
                with torch.cuda.stream(torch.cuda.Stream()):
                    for rep in range(4):
                        print(f"[gpu] run {i} of two, rep={rep}", flush=True)
                        got[i], _ = runner.serve(cache, [ids[f] for f in asked[i]], [0] * len(asked[i]), 16 << 20,
                                                 chunk_bytes=16 << 10, grid=8, idle_timeout_s=20.0)
                        np.testing.assert_array_equal(got[i]["csum"], want[asked[i]])
                        np.testing.assert_array_equal(got[i]["result"], np.array(SIZES, dtype=np.int64)[asked[i]])
            except Exception as e:   # noqa: BLE001 - reported below
                failed.append(repr(e))

        t = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
        for x in t:
            x.start()
        for x in t:
            x.join()
        assert not failed, failed
        assert cache.stats()["timeouts"] == 0
