"""Units of a batch launch are each one gread of a file: a unit reaching past the file's end, by
any size, delivers what the file has and ends there, and a unit whose read fails adds nothing to
its file's checksum and histogram, nor to the bytes delivered. A served chunk's first page is a
gread of its own, and the rest of the chunk another."""
import os

import numpy as np
import pytest

from paper_2109_05366_amd import gfs, runner

pytestmark = pytest.mark.gpu

PAGE = 64 << 10


@pytest.fixture(scope="module")
def cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gfs.lib()
    return torch


def _file(path, size, seed):
    data = np.random.RandomState(seed).randint(0, 256, size, dtype=np.uint8)
    data.tofile(path)
    return data


def _units(rows):
    units = np.zeros(len(rows), dtype=gfs.UNIT_DTYPE)
    for i, (f, out, offset, size) in enumerate(rows):
        units[i]["file"], units[i]["out"], units[i]["offset"], units[i]["size"] = f, out, offset, size
    return units


def _sum(data):
    return int(np.pad(data, (0, -len(data) % 4)).view("<u4").sum(dtype=np.uint64))


@pytest.mark.parametrize("beyond", [1, 300 << 10, 1 << 40, (1 << 64) - 1])
def test_units_past_the_end_of_the_file(beyond, tmp_path, cuda):
    size = (700 << 10) + 13
    data = _file(str(tmp_path / "f.bin"), size, 5)
    with gfs.PageCache(runner.make_config(PAGE, 64 * PAGE, ra_cap_bytes=4 * PAGE, timeout_s=20)) as cache:
        starts = [0, 16, 5, 512 << 10, size - 40, size - 1, size, size + 7, size + (1 << 30)]
        ids = [cache.open(str(tmp_path / "f.bin")) for _ in starts]   # an output row belongs to one file id
        rows = [(ids[i], i, o, min(max(size - o, 0) + beyond, (1 << 64) - 1)) for i, o in enumerate(starts)]
        r = runner.BatchReader(None, None, 1 << 20, 0, grid=4, units=_units(rows), nout=len(rows))
        for rep in range(2):
            print(f"[gpu] units past the end by {beyond}, rep={rep}", flush=True)
            r.launch(cache)
            res = r.result()
            assert [int(c) for c in res.csum] == [_sum(data[o:]) for o in starts]
            np.testing.assert_array_equal(res.hist, [np.bincount(data[o:], minlength=256) for o in starts])
            assert int(res.status.sum()) == sum(len(data[o:]) for o in starts)


@pytest.mark.parametrize("threads", [64, 256])
@pytest.mark.parametrize("cut", [100, (600 << 10) + 100])
def test_a_unit_that_fails_adds_nothing(cut, threads, tmp_path, cuda):
    """The second file is cut on disk once it is registered, inside its first or a later piece: the
    first file's unit is delivered, the second's fails whole."""
    size = (1 << 20) - 48
    good = _file(str(tmp_path / "good.bin"), size, 1)
    _file(str(tmp_path / "cut.bin"), size, 2)
    with gfs.PageCache(runner.make_config(PAGE, 64 * PAGE, ra_cap_bytes=2 * PAGE, timeout_s=20)) as cache:
        ids = [cache.open(str(tmp_path / n)) for n in ("good.bin", "cut.bin")]
        os.truncate(str(tmp_path / "cut.bin"), cut)
        r = runner.BatchReader(None, None, 1 << 20, 0, grid=1, threads=threads, nout=2,
                               units=_units([(ids[0], 0, 0, size), (ids[1], 1, 0, size)]))
        print(f"[gpu] a unit that fails, cut={cut} threads={threads}", flush=True)
        r.launch(cache)
        res = r.result()
        st = cache.stats()
    assert int(res.status[0]) == -5 and st["timeouts"] == 0
    assert [int(c) for c in res.csum] == [_sum(good), 0]
    np.testing.assert_array_equal(res.hist[0], np.bincount(good, minlength=256))
    assert not res.hist[1].any()
    assert st["delivered_bytes"] == size


def test_a_served_chunk_that_fails_counts_its_first_page_alone(tmp_path, cuda):
    size = (1 << 20) - 48
    _file(str(tmp_path / "cut.bin"), size, 2)
    with gfs.PageCache(runner.make_config(PAGE, 64 * PAGE, ra_cap_bytes=2 * PAGE, timeout_s=20)) as cache:
        fid = cache.open(str(tmp_path / "cut.bin"))
        os.truncate(str(tmp_path / "cut.bin"), (600 << 10) + 100)
        print("[gpu] a served chunk that fails", flush=True)
        recs, _ = runner.serve(cache, [fid], [0], 64 * PAGE, grid=2, idle_timeout_s=20.0)
        st = cache.stats()
    assert int(recs["result"][0]) == -5 and int(recs["csum"][0]) == 0 and int(recs["first_ns"][0]) > 0
    assert st["delivered_bytes"] == PAGE and st["timeouts"] == 0


@pytest.mark.parametrize("threads,blocks,cut", [(64, 300, 256 << 10), (256, 300, 256 << 10), (64, 600, 64 << 10)])
def test_units_read_in_pieces(threads, blocks, cut, tmp_path, cuda):
    """More blocks at work, on larger buffers, than are read whole (see test_cut_reads.py): units on,
    before and after the places a unit is cut at, units past the end of the file, one that fails in
    its last piece."""
    size, unit = (3 << 20) + 1003, 1 << 20
    data = _file(str(tmp_path / "f.bin"), size, 7)
    _file(str(tmp_path / "cut.bin"), size, 8)
    with gfs.PageCache(runner.make_config(PAGE, 256 * PAGE, ra_cap_bytes=4 * PAGE, timeout_s=20)) as cache:
        fid, bad = cache.open(str(tmp_path / "f.bin")), cache.open(str(tmp_path / "cut.bin"))
        os.truncate(str(tmp_path / "cut.bin"), (900 << 10) + 100)
        starts = [0, 16, cut - 16, cut, cut + 16, unit, 5, cut - 7, size - 40, size - unit - 3, size, size + 9]
        good = [(fid, 0, o, unit if i % 3 else (1 << 64) - 1 - i) for i, o in enumerate(starts) if i % 3 or size - o <= unit]
        good += [(fid, 0, 16 * i, 64 + i) for i in range(blocks - 1 - len(good))]
        got = [data[o:min(size, o + n)] for _, _, o, n in good]
        for rep, rows in enumerate((good, good, good + [(bad, 1, 0, unit)])):
            print(f"[gpu] pieces threads={threads} rep={rep}", flush=True)
            r = runner.BatchReader(None, None, unit, 0, grid=blocks, threads=threads, units=_units(rows), nout=2)
            r.launch(cache)
            res = r.result()
            assert [int(c) for c in res.csum] == [sum(_sum(g) for g in got), 0]
            np.testing.assert_array_equal(res.hist, [sum(np.bincount(g, minlength=256) for g in got), np.zeros(256, int)])
            assert sorted(res.status)[0] == (-5 if rep == 2 else 0)
            if rep < 2:
                assert int(res.status.sum()) == sum(len(g) for g in got)
        assert cache.stats()["delivered_bytes"] == 3 * sum(len(g) for g in got)


def test_served_chunks_read_in_pieces(tmp_path, cuda):
    """A burst of more than 256 chunks of 1 MiB in flight, cached and not, one of whose files fails."""
    size = (8 << 20) + 24
    datas = [_file(str(tmp_path / f"f{i}.bin"), size, i) for i in range(2)]
    _file(str(tmp_path / "cut.bin"), size, 9)
    with gfs.PageCache(runner.make_config(PAGE, 512 * PAGE, ra_cap_bytes=4 * PAGE, timeout_s=20)) as cache:
        ids = [cache.open(str(tmp_path / n)) for n in ("f0.bin", "f1.bin", "cut.bin")]
        os.truncate(str(tmp_path / "cut.bin"), (600 << 10) + 100)
        asked = np.array([i % 2 for i in range(40)] + [2])
        for rep in range(2):
            print(f"[gpu] served pieces rep={rep}", flush=True)
            recs, _ = runner.serve(cache, [ids[i] for i in asked], [0] * len(asked), 1 << 30, grid=512, idle_timeout_s=20.0)
            np.testing.assert_array_equal(recs["csum"], np.array([_sum(d) for d in datas] + [0], dtype=np.uint64)[asked])
            np.testing.assert_array_equal(recs["result"], np.array([size, size, -5])[asked])
        assert cache.stats()["timeouts"] == 0
