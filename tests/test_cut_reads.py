"""When a batch unit or a served chunk is read and consumed in pieces: with more than a block a
compute unit at work, on more bytes than the last-level cache holds; otherwise it is read whole."""
import ctypes
import os

import pytest

from paper_2109_05366_amd import build, gfs

MiB = 1 << 20


@pytest.mark.parametrize("blocks,size,cut", [
    (1, MiB, False), (1, 1 << 32, False), (64, 4 * MiB, False), (128, 4 * MiB, False), (256, 4 * MiB, False),
    (256, MiB, False), (257, MiB, True), (320, MiB, True), (512, MiB, True), (512, 512 << 10, False),
    (512, (512 << 10) + 16, True), (1024, 256 << 10, False), (2048, 384 << 10, True), (2048, 16, False)])
def test_rule(blocks, size, cut):
    gfs.lib()
    ctypes.CDLL(build.LIB, mode=ctypes.RTLD_GLOBAL)
    if not os.path.exists(build.SERVE_PROBE_LIB):
        raise RuntimeError(f"{build.SERVE_PROBE_LIB} is not built; run __graft_entry__.build() first")
    L = ctypes.CDLL(build.SERVE_PROBE_LIB)
    L.gfs_test_cut_reads.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    assert bool(L.gfs_test_cut_reads(blocks, size)) == cut
