"""gread's copies at the edges of their 16-byte units, pages and groups of 64 pages: every
alignment of the file offset against the user buffer, reads shorter than a unit, up to a page's
edge, over it, and over more than 64 pages, by blocks of one to four waves, cold and cached; and
bytes beside the read's destination left alone."""
import ctypes

import numpy as np
import pytest

from paper_2109_05366_amd import build, gfs, runner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gfs.lib()
    return torch


def _file(tmp_path, size, seed):
    data = np.random.RandomState(seed).randint(0, 256, size, dtype=np.uint8)
    p = str(tmp_path / "f.bin")
    data.tofile(p)
    return p, data


@pytest.mark.parametrize("page,threads", [(4 << 10, 256), (4 << 10, 64), (16 << 10, 192), (64 << 10, 256), (64 << 10, 128)])
def test_reads_at_every_offset_alignment(page, threads, tmp_path, cuda):
    size = 70 * page + 4093                      # more than 64 pages, a ragged last one
    path, data = _file(tmp_path, size, page + threads)
    at = [a for a in range(16)]
    starts = ([a for a in at] + [page - 24 + a for a in at] + [63 * page + 5 * a for a in at] +
              [size - 40 - 16 * a for a in at] + [size - 1, size, size + 7])
    reads = {16: starts, 48: starts, page + 32: starts, 3 * page: starts[::3], 69 * page + 16: starts[::5]}
    cfg = runner.make_config(page, 128 * page, ra_cap_bytes=8 * page, timeout_s=20)
    for n, offs in reads.items():
        print(f"[gpu] reads page={page} threads={threads} size={n}", flush=True)
        with gfs.PageCache(cfg) as cache:
            fid = cache.open(path)
            offsets = np.array(offs, dtype=np.uint64)[:, None]
            for _ in range(2):                   # cold, then cached
                r = runner.ListReader(offsets, n, 2, threads)
                r.buf.fill_(0xA5)
                r.launch(cache, fid)
                res = r.result()
                want = np.full((len(offs), n), 0xA5, dtype=np.uint8)
                for i, o in enumerate(offs):
                    got = data[o:o + n]
                    want[i, :len(got)] = got
                np.testing.assert_array_equal(res.status, [len(data[o:o + n]) for o in offs])
                np.testing.assert_array_equal(res.out, want)
            st = cache.stats()
        assert st["timeouts"] == 0 and st["io_errors"] == 0 and st["hits"] > 0


def _probe():
    vp, u64, u32 = ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint32
    L = ctypes.CDLL(build.PROBE_LIB)
    L.gfs_test_api_probe.argtypes = [vp, vp, vp, ctypes.c_int, u64, u64, u64, u32, vp, vp, vp]
    L.gfs_test_api_probe.restype = ctypes.c_int
    return L


@pytest.mark.parametrize("page", [4 << 10, 64 << 10])
def test_reads_into_every_buffer_alignment(page, tmp_path, cuda):
    torch = cuda
    size = 5 * page + 77
    path, data = _file(tmp_path, size, page + 1)
    L = _probe()
    cfg = runner.make_config(page, 64 * page, ra_cap_bytes=4 * page, timeout_s=20)
    with gfs.PageCache(cfg) as cache:
        fid = cache.open(path)
        unused = cache.open(path)
        cache.close_file(unused)
        name = torch.tensor(list(path.encode()) + [0], dtype=torch.uint8, device="cuda")
        missing = torch.tensor(list(b"/none") + [0], dtype=torch.uint8, device="cuda")
        out = torch.zeros(10, dtype=torch.int64, device="cuda")
        for n in (1, 15, 16, 17, 31, 200, page + 3, 3 * page + 5):
            print(f"[gpu] buffer alignments page={page} size={n}", flush=True)
            for a in range(16):
                off = page - 9 + (5 * a) % 16
                buf = torch.full((n + 128,), 0xA5, dtype=torch.uint8, device="cuda")
                rc = L.gfs_test_api_probe(cache.handle, name.data_ptr(), missing.data_ptr(), unused, off, n, size, 256,
                                          buf.data_ptr() + 16 + a, out.data_ptr(),
                                          torch.cuda.current_stream().cuda_stream)
                assert rc == 0
                torch.cuda.synchronize()
                assert out[0].item() == fid and out[5].item() == n
                want = np.full(n + 128, 0xA5, dtype=np.uint8)
                want[16 + a:16 + a + n] = data[off:off + n]
                np.testing.assert_array_equal(buf.cpu().numpy(), want)


def test_two_files_that_share_a_row_of_lock_notes(tmp_path, cuda):
    """Files 0 and 64 keep the notes of their waiting misses in the same place: read together, by
    more blocks than a holder decides for at once, from offsets that make windows meet."""
    torch = cuda
    page, blocks = 4 << 10, 512
    cfg = runner.make_config(page, 2 * blocks * page, ra_cap_bytes=8 * page, max_files=66, timeout_s=20)
    with gfs.PageCache(cfg) as cache:
        ids, datas = [], []
        for i in range(65):
            size = 4 * blocks * page + 100 + i if i in (0, 64) else 10
            data = np.random.RandomState(i).randint(0, 256, size, dtype=np.uint8)
            p = str(tmp_path / f"f{i}.bin")
            data.tofile(p)
            ids.append(cache.open(p))
            datas.append(data)
        assert ids[64] - ids[0] == 64
        n = 2 * page + 48
        starts = (np.arange(blocks, dtype=np.uint64) * 4 * page)[:, None] + np.arange(2, dtype=np.uint64)[None, :] * 2 * page
        for rep in range(3):
            print(f"[gpu] shared notes rep={rep}", flush=True)
            pairs = [(runner.ListReader(starts, n, 2, 64), torch.cuda.Stream(), f) for f in (0, 64)]
            torch.cuda.synchronize()
            for r, s, f in pairs:
                r.launch(cache, ids[f], stream=s)
            for r, _, f in pairs:
                res = r.result()
                last = starts[:, -1].astype(int)
                want = np.stack([np.resize(np.pad(datas[f][o:o + n], (0, n)), n) for o in last])
                got_n = np.array([sum(len(datas[f][int(o):int(o) + n]) for o in row) for row in starts])
                np.testing.assert_array_equal(res.status, got_n)
                full = np.array([len(datas[f][o:o + n]) == n for o in last])
                np.testing.assert_array_equal(res.out[full], want[full])
            st = cache.stats()
            assert st["timeouts"] == 0 and st["io_errors"] == 0
            cache.reset()


@pytest.mark.parametrize("threads", [64, 256])
def test_batch_consumer_at_the_edges_of_its_rounds(threads, tmp_path, cuda):
    """A batch launch's checksum and histogram over files whose last unit ends inside a 16-byte
    piece, a word, and a round of eight pieces a thread."""
    page, unit, rnd = 4 << 10, 64 << 10, 8 * 16 * threads
    sizes = [1, 3, 15, 16, 17, rnd - 1, rnd, rnd + 16, rnd + 7, unit - 5, unit, unit + rnd + 2, 3 * unit + 19]
    cfg = runner.make_config(page, 1024 * page, ra_cap_bytes=16 * page, timeout_s=20)
    print(f"[gpu] batch consumer threads={threads}", flush=True)
    with gfs.PageCache(cfg) as cache:
        ids, datas = [], []
        for i, size in enumerate(sizes):
            data = np.random.RandomState(size).randint(0, 256, size, dtype=np.uint8)
            p = str(tmp_path / f"b{i}.bin")
            data.tofile(p)
            ids.append(cache.open(p))
            datas.append(data)
        r = runner.BatchReader(ids, sizes, unit, 2, grid=5, threads=threads)
        for _ in range(2):
            r.launch(cache)
            res = r.result()
            words = [np.pad(d, (0, -len(d) % 4)).view("<u4") for d in datas]
            # a file's units start on word boundaries, so their sums add up to the file's
            np.testing.assert_array_equal(res.csum, [w.sum(dtype=np.uint64) for w in words])
            np.testing.assert_array_equal(res.hist, [np.bincount(d, minlength=256) for d in datas])
            assert int(res.status.sum()) == sum(sizes)


@pytest.mark.parametrize("page,unit", [(4 << 10, (300 << 10) + 16), (512 << 10, (1 << 20) + 48), (64 << 10, 256 << 10)])
def test_batch_units_read_in_pieces(page, unit, tmp_path, cuda):
    """Units that start before, on and after the places a unit is cut at, and units that start off
    a 16-byte boundary, cold and cached: sums over each unit's own words, and the buffer's bytes."""
    size = 3 * unit + 100003
    path, data = _file(tmp_path, size, page + unit)
    cut = max(page, 256 << 10)
    starts = [0, 16, cut - 16, cut, cut + 16, unit, 5, cut - 7, cut + 1, size - 40, size - unit - 3]
    cfg = runner.make_config(page, max(64 * page, 16 << 20), ra_cap_bytes=max(page, 256 << 10), timeout_s=20)
    with gfs.PageCache(cfg) as cache:
        fid = cache.open(path)
        units = np.zeros(len(starts), dtype=gfs.UNIT_DTYPE)
        for i, o in enumerate(starts):
            units[i]["file"], units[i]["offset"] = fid, o
            units[i]["size"] = min(unit, size - o)
        r = runner.BatchReader(None, None, unit, 0, grid=3, units=units, nout=1)
        got = [data[o:o + int(u["size"])] for o, u in zip(starts, units)]
        for rep in range(2):
            print(f"[gpu] pieces page={page} unit={unit} rep={rep}", flush=True)
            r.launch(cache)
            res = r.result()
            assert int(res.csum[0]) == sum(int(np.pad(g, (0, -len(g) % 4)).view("<u4").sum(dtype=np.uint64)) for g in got)
            np.testing.assert_array_equal(res.hist[0], sum(np.bincount(g, minlength=256) for g in got))
            assert int(res.status.sum()) == sum(len(g) for g in got)
        one = runner.BatchReader(None, None, unit, 0, grid=1, units=units[3:4], nout=1)
        one.launch(cache)
        one.result()
        np.testing.assert_array_equal(one.buf.cpu().numpy()[:len(got[3])], got[3])
