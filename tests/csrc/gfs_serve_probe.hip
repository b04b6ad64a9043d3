// The serving loop's hand-out of units on a table of the test's own making: one wave takes a unit
// number that the control words count but no entry of the table holds.
// Built by the package's build step into tests/libgfs_serve_probe.so; the host functions that the
// serving loop calls are libgfs.so's, which is loaded first.
#include "../../paper_2109_05366_amd/csrc/gfs_serve.hip"

namespace {

// out[0] what pick_unit returned, out[1] the abort word after it
__global__ void lost_unit_kernel(SrvCtrl* ctl, SrvEntry* tab, uint32_t cap, int64_t* out) {
  uint64_t hint = 0, k = 0, size = 0, open = 0;
  uint32_t file = 0;
  if (gfsd::lane() == 0) gfsd::st_rlx(&ctl->units, 1);
  gfsd::drain_atomics();
  const int cmd = pick_unit(ctl, tab, cap, nullptr, nullptr, nullptr, 4096, 1, hint, &k, &file, &size, &open);
  gfsd::drain_atomics();
  if (gfsd::lane() == 0) {
    out[0] = cmd;
    out[1] = (int64_t)gfsd::ld_rlx(&ctl->abort);
  }
}

}  // namespace

extern "C" uint64_t gfs_test_serve_probe_bytes(uint32_t cap) { return sizeof(SrvCtrl) + cap * sizeof(SrvEntry); }
// state: gfs_test_serve_probe_bytes(cap) zero bytes, 256-byte aligned; out: two values
extern "C" int gfs_test_serve_lost_unit(void* state, uint32_t cap, int64_t* out, void* stream) {
  if (!state || !out || cap == 0) return -EINVAL;
  hipLaunchKernelGGL(lost_unit_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, (SrvCtrl*)state,
                     (SrvEntry*)((uint8_t*)state + sizeof(SrvCtrl)), cap, out);
  return hipGetLastError() == hipSuccess ? 0 : -EIO;
}
// log2 of the pieces in which `blocks` blocks that consume reads of `bytes` take them, 0: whole (host only)
extern "C" uint32_t gfs_test_cut_reads(uint64_t blocks, uint64_t bytes) {
  const uint32_t c = gfsd::cut_reads(blocks, bytes);
  return c == gfsd::kWhole ? 0 : c;
}
