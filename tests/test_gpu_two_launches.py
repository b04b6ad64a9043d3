"""Two launches of different grids read one file at the same time: each miss gets a window within its
own launch's share of the cache, whichever launch's block decided it."""
import numpy as np
import pytest

from paper_2109_05366_amd import gfs, runner

pytestmark = pytest.mark.gpu

PAGE = 4 << 10


def test_windows_are_sized_by_the_launch_that_missed(tmp_path):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    frames, half, many, few, cap = 2048, 4096, 512, 8, 64
    data = np.random.RandomState(3).randint(0, 256, 2 * half * PAGE, dtype=np.uint8)
    data.tofile(str(tmp_path / "f.bin"))
    cfg = runner.make_config(PAGE, frames * PAGE, ra_cap_bytes=cap * PAGE, quota_blocks=512, trace_level=1,
                             trace_capacity=1 << 18, timeout_s=20)
    with gfs.PageCache(cfg) as cache:
        fid = cache.open(str(tmp_path / "f.bin"))
        pages = np.arange(half, dtype=np.uint64)
        launches = []
        for blocks, first in ((many, 0), (few, half)):
            offs = (pages.reshape(-1, blocks).T.copy() + np.uint64(first)) * np.uint64(PAGE)
            launches.append((runner.ListReader(offs, PAGE, 0, 64), torch.cuda.Stream(), offs))
        torch.cuda.synchronize()
        print("[gpu] two launches of different grids", flush=True)
        for r, s, _ in launches:
            r.launch(cache, fid, stream=s)
        words = data.view("<u4").reshape(-1, PAGE // 4).sum(axis=1, dtype=np.uint64)
        for r, _, offs in launches:
            res = r.result()
            np.testing.assert_array_equal(res.out, words[(offs // PAGE).astype(int)].sum(axis=1, dtype=np.uint64))
            assert (res.status == offs.shape[1] * PAGE).all()
        st = cache.stats()
        ev = cache.trace()
    assert st["timeouts"] == 0 and st["trace_events"] <= len(ev)
    miss = ev[ev["op"] == 3]
    mine = miss["page"] < half
    print(f"[gpu] windows up to {miss['a'][mine].max()} and {miss['a'][~mine].max()} pages", flush=True)
    assert miss["a"][mine].max() <= frames // many
    assert frames // many < miss["a"][~mine].max() <= cap
