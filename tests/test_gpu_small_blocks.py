"""Blocks of one and two waves: as many are resident at once as registers allow (two waves a SIMD,
so 8 and 4 blocks on each of the compute units), which the batch grid reports and the serialising
gate accepts, and their counts of bytes are right."""
import numpy as np
import pytest

from paper_2109_05366_amd import gfs, runner

pytestmark = pytest.mark.gpu

PAGE = 4 << 10


@pytest.fixture(scope="module")
def cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gfs.lib()
    return torch


def _cus(torch):
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("threads,per_cu", [(64, 8), (128, 4), (192, 2), (256, 2)])
def test_resident_blocks(threads, per_cu, cuda):
    assert gfs.gfs_batch_grid(threads) == per_cu * _cus(cuda)


@pytest.mark.parametrize("threads,per_cu", [(64, 8), (128, 4), (192, 2), (256, 2)])
@pytest.mark.parametrize("consumer", [0, 1, 2])
def test_serialised_reads_of_every_resident_block(threads, per_cu, consumer, tmp_path, cuda):
    blocks = per_cu * _cus(cuda)
    n = 1040
    data = np.random.RandomState(threads).randint(0, 256, 64 * PAGE + 123, dtype=np.uint8)
    data.tofile(str(tmp_path / "f.bin"))
    offs = np.random.RandomState(1).randint(0, len(data), (blocks, 1)).astype(np.uint64)
    parts = [data[int(o):int(o) + n] for o in offs[:, 0]]
    with gfs.PageCache(runner.make_config(PAGE, 128 * PAGE, ra_cap_bytes=8 * PAGE, timeout_s=20)) as cache:
        fid = cache.open(str(tmp_path / "f.bin"))
        print(f"[gpu] serialised threads={threads} blocks={blocks} consumer={consumer}", flush=True)
        r = runner.ListReader(offs, n, consumer, threads)
        r.buf.zero_()
        r.launch(cache, fid, serialize=True)
        res = r.result()
        assert cache.stats()["timeouts"] == 0
    np.testing.assert_array_equal(res.status, [len(p) for p in parts])
    if consumer == 0:
        np.testing.assert_array_equal(res.out, [np.pad(p, (0, -len(p) % 4)).view("<u4").sum(dtype=np.uint64) for p in parts])
    elif consumer == 1:
        np.testing.assert_array_equal(res.out, [np.bincount(p, minlength=256) for p in parts])
    else:
        np.testing.assert_array_equal(res.out, [np.pad(p, (0, n - len(p))) for p in parts])


@pytest.mark.parametrize("threads", [64, 128, 192, 256])
def test_counts_of_the_batch_and_buffer_readers(threads, tmp_path, cuda):
    torch = cuda
    size = (1 << 20) + 4099
    data = np.random.RandomState(threads).randint(0, 256, size, dtype=np.uint8)
    data[100000:300000] = 7                        # equal bytes meet in one counter
    data.tofile(str(tmp_path / "f.bin"))
    want = np.bincount(data, minlength=256)
    print(f"[gpu] counts threads={threads}", flush=True)
    with gfs.PageCache(runner.make_config(PAGE, 512 * PAGE, ra_cap_bytes=16 * PAGE, timeout_s=20)) as cache:
        fid = cache.open(str(tmp_path / "f.bin"))
        r = runner.BatchReader([fid], [size], 64 << 10, 4, grid=0, threads=threads)
        r.launch(cache)
        res = r.result()
        np.testing.assert_array_equal(res.hist[0], want)
        assert int(res.csum[0]) == int(np.pad(data, (0, -size % 4)).view("<u4").sum(dtype=np.uint64))
    dev = torch.from_numpy(data).cuda()
    step = 10007                                   # reads start at every alignment
    offs = torch.arange(0, size, step, dtype=torch.int64).reshape(-1, 1).cuda()
    out = torch.zeros(len(offs) * 256, dtype=torch.int32, device="cuda")
    status = torch.zeros(len(offs), dtype=torch.int64, device="cuda")
    gfs.gfs_launch_buffer_reader(dev.data_ptr(), size, offs.data_ptr(), len(offs), 1, step, threads, 1, out.data_ptr(),
                                 status.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy().reshape(-1, 256).sum(0), want)
    assert int(status.sum()) == size
