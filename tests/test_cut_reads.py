"""When a batch unit or a served chunk is read and consumed in pieces: with more than a block a
compute unit at work, on more bytes than the last-level cache holds; otherwise it is read whole.
The pieces of up to 512 blocks are 256 KiB, those of more 64 KiB."""
import ctypes
import os

import pytest

from paper_2109_05366_amd import build, gfs

MiB = 1 << 20


@pytest.mark.parametrize("blocks,size,cut", [
    (1, MiB, 0), (1, 1 << 32, 0), (64, 4 * MiB, 0), (128, 4 * MiB, 0), (256, 4 * MiB, 0),
    (256, MiB, 0), (257, MiB, 18), (320, MiB, 18), (512, MiB, 18), (512, 512 << 10, 0),
    (512, (512 << 10) + 16, 18), (513, MiB, 16), (1024, 192 << 10, 0), (1024, (192 << 10) + 16, 16), (2048, 384 << 10, 16), (2048, 16, 0)])
def test_rule(blocks, size, cut):
    gfs.lib()
    ctypes.CDLL(build.LIB, mode=ctypes.RTLD_GLOBAL)
    if not os.path.exists(build.SERVE_PROBE_LIB):
        raise RuntimeError(f"{build.SERVE_PROBE_LIB} is not built; run __graft_entry__.build() first")
    L = ctypes.CDLL(build.SERVE_PROBE_LIB)
    L.gfs_test_cut_reads.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    assert L.gfs_test_cut_reads(blocks, size) == cut
