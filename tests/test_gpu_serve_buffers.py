"""The device memory that gfs_serve_run keeps with its context for the next run can be had back
without closing the context: gfs_reset_cache frees it, and a run after that allocates it again."""
import numpy as np
import pytest

from oracle import data as odata
from paper_2109_05366_amd import gfs, runner

pytestmark = pytest.mark.gpu

MiB = 1 << 20


def test_reset_gives_the_serving_buffers_back(tmp_path):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    path = str(tmp_path / "f.bin")
    np.random.RandomState(1).randint(0, 256, 3 * MiB + 8, dtype=np.uint8).tofile(path)
    want = odata.file_checksum(path)

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    with gfs.PageCache(runner.make_config(64 << 10, 16 * MiB, timeout_s=20)) as cache:
        fid = cache.open(path)
        for rep in range(3):   # the first run also makes the runtime allocate the kernel's scratch memory
            print(f"[gpu] serving buffers rep={rep}", flush=True)
            before = free()
            recs, _ = runner.serve(cache, [fid] * 3, [0] * 3, 64 * MiB, chunk_bytes=MiB, grid=256, idle_timeout_s=20.0)
            assert [int(c) for c in recs["csum"]] == [want] * 3
            kept = free()
            cache.reset()
            assert free() >= kept + 256 * MiB
            assert rep == 0 or (kept <= before - 256 * MiB and free() >= before - 16 * MiB)
