"""A unit number that no request in the table holds stops the serving loop at once: the block that
finds it out sets the abort word that every block reads, instead of leaving alone and the others
to wait for the unit's completion until the idle limit."""
import ctypes
import os

import pytest

from paper_2109_05366_amd import build, gfs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [1, 64, 130])
def test_a_lost_unit_aborts_the_run(cap):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gfs.lib()
    ctypes.CDLL(build.LIB, mode=ctypes.RTLD_GLOBAL)
    if not os.path.exists(build.SERVE_PROBE_LIB):
        raise RuntimeError(f"{build.SERVE_PROBE_LIB} is not built; run __graft_entry__.build() first")
    L = ctypes.CDLL(build.SERVE_PROBE_LIB)
    L.gfs_test_serve_probe_bytes.restype = ctypes.c_uint64
    L.gfs_test_serve_lost_unit.argtypes = [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p]
    state = torch.zeros(L.gfs_test_serve_probe_bytes(cap), dtype=torch.uint8, device="cuda")
    out = torch.full((2,), -1, dtype=torch.int64, device="cuda")
    print(f"[gpu] lost unit cap={cap}", flush=True)
    assert L.gfs_test_serve_lost_unit(state.data_ptr(), cap, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert out.tolist() == [1, 1]   # leave, and the run is aborted
