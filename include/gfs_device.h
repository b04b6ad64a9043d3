/* gfs_device.h -- device side of the GPU file page cache: gopen / gread / gclose.
 *
 * Include from HIP code compiled for gfx950. The functions are block-collective
 * (Sec. 2.2: each threadblock issues a file call by invoking it from all of its
 * threads): every thread of the block must call them with the same arguments, and
 * every thread gets the same result. Blocks must have a multiple of 64 threads. Every
 * block must obtain its descriptor with gopen/gopen_id before calling gread, and
 * should gclose it at the end: the block's statistics are flushed there. A block has files
 * of one cache open at a time (its state in LDS is that cache's until gclose).
 *
 *   int     gopen (const gfs_dev* d, const char* path, int flags);
 *       Resolve a path registered with gfs_open (path: NUL-terminated, device-readable
 *       memory) to a descriptor. flags must be GFS_O_RDONLY (-EROFS otherwise); an
 *       unknown path gives -ENOENT.
 *   int     gopen_id(const gfs_dev* d, int file_id, int flags);
 *       Same, from the id gfs_open returned.
 *   int64_t gread (const gfs_dev* d, int fd, uint64_t offset, uint64_t size, void* dst);
 *       Copy file bytes [offset, min(offset+size, file size)) to dst (device memory of
 *       at least that many bytes, at any alignment). Returns the byte count (short only at EOF, 0 at or past it) or -EBADF,
 *       -EINVAL, -EIO (host read failed), -ENOSPC (the page's table buckets stayed full of
 *       other misses' reservations until the wait limit), -ETIMEDOUT (a wait exceeded the
 *       configured timeout; the cache must then be reset).
 *   int     gclose(const gfs_dev* d, int fd);
 *
 * How a read is served (Sec. 2.2 and Sec. 4.1): the request is divided into pages; each
 * page is looked up in the hashed page table and, on a hit, pinned and copied out. On a
 * miss the block takes the file's miss lock, asks the readahead detector for a window,
 * reserves the run of unmapped window pages around the miss in the page table, and
 * unlocks; it then gives the reserved pages frames with the clock hand (evicting in
 * place, Sec. 5.1), posts one request for the run to the host ring and waits for it
 * (synchronous prefetch, Sec. 4), pulls the fetched bytes from pinned staging into the
 * frames, publishes them, and copies its own page out. Blocks that find a page whose
 * frame is reserved or still being filled wait for it instead of fetching it again.
 *
 * Calling kernels: gread is inlined into its caller and its miss path needs about 250
 * VGPRs; give the kernel __launch_bounds__(GFS_MAX_BLOCK_THREADS) or less, or the compiler
 * caps registers lower and spills every call's state to scratch memory.
 */
#ifndef GFS_DEVICE_H
#define GFS_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gfs.h"
#include "gfs_layout.h"
#include "gfs_lock.h"

namespace gfsd {

constexpr int kENOENT = 2, kEIO = 5, kEBADF = 9, kEINVAL = 22, kENOSPC = 28, kEROFS = 30,
              kETIMEDOUT = 110;
constexpr uint32_t kMaxWindow = GFS_MAX_WINDOW_PAGES;
constexpr uint64_t kFrameMask = (1ull << GFS_ENTRY_FRAME_BITS) - 1;
/* page-table entry frame value of a page reserved by a miss that has no frame yet */
constexpr uint32_t kReserved = (uint32_t)kFrameMask;
/* group pass: no table entry; an entry whose frame is not ready to be copied from */
constexpr int32_t kAbsent = -1, kNotReady = -2;

/* Per-block state in LDS, shared by gopen/gread/gclose within one kernel. */
struct BlockState {
  int64_t status;           /* 0 or -errno for the current page */
  int64_t result;           /* host read result for the request this block pulls */
  uint64_t first_page;      /* first page of the request span */
  uint64_t gen;             /* ring generation of the request */
  int32_t frame;            /* pinned frame of the current page */
  int32_t pull;             /* 1: pull this block's own request; 2: help pull one frame;
                               3: fill the frame from the private buffer; 4: pull a private-policy
                               request (page into the frame, the rest into the private buffer) */
  uint32_t slot;            /* ring slot of the request */
  uint32_t list_n;          /* pages in list[] that got frames (a prefix) */
  uint32_t file;
  int32_t open_result;
  int32_t open_fd;          /* the descriptor gopen returned last (-1: none), and its file's */
  uint64_t open_size;       /* size, read once: a registered file cannot be closed while a
                               kernel holds it open, so gread need not read them again */
  uint64_t ctr[GFS_C_COUNT];    /* block-local statistics, added to the globals by gclose */
  uint32_t list[kMaxWindow];    /* run pages: the demanded page, then the rest ascending */
  uint32_t lframe[kMaxWindow];  /* frame given to list[k], or GFS_NO_FRAME */
  uint32_t lslot[kMaxWindow];   /* page-table slot reserved for list[k] (0xffffffff: none);
                                   after allocation, the indices of the frames this block pulls */
  uint32_t nclaim;              /* entries of lslot[] claimed for pulling */
  uint32_t help_page;           /* page of the frame a helping block pulls */
  int32_t pslot;                /* private policy: the block's slot (-1: none) */
  int32_t bframe[2][64];        /* group pass: frame pinned for page base + i, kAbsent (no table
                                   entry) or kNotReady; the two halves take turns (par) */
  uint64_t bbad[2];             /* group pass: pages whose frame turned out to hold another page */
  uint32_t par;                 /* the half the next group pass uses */
  uint32_t trig;                /* asynchronous readahead: this page access took a marker */
  uint32_t a_pending;           /* 1: this block has an asynchronous request outstanding, whose
                                   pages and frames are list[0..a_n) / lframe[0..a_n) */
  uint32_t a_slot, a_n, a_file;
  int32_t a_status;
  uint64_t a_gen, a_first;
  uint32_t naps;                /* back-off of the page access in progress (lane 0) */
  uint64_t read_last;           /* last page of the gread in progress: a readahead window
                                   opened by a miss covers the read up to it */
};

/* the lock queue's size assumes every block that calls gread holds this much LDS */
static_assert(sizeof(BlockState) >= GFS_BLOCK_LDS_MIN, "per-block state below the LDS bound the lock queue assumes");

__device__ __forceinline__ BlockState* block_state() {
  __shared__ BlockState gfs_block_state;
  return &gfs_block_state;
}

/* ------------------------------------------------------------------ thread / wave ids */
__device__ __forceinline__ uint32_t thread_id() {
  return threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
}
__device__ __forceinline__ uint32_t block_threads() { return blockDim.x * blockDim.y * blockDim.z; }
__device__ __forceinline__ uint32_t block_id() {
  return blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
}
__device__ __forceinline__ uint32_t lane() { return __lane_id(); }
__device__ __forceinline__ uint64_t lanemask_lt() {
  const uint32_t l = __lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}
/* lane i's value, i the same in every lane: a scalar read (a shuffle goes through LDS and costs
   about a hundred cycles) */
__device__ __forceinline__ uint64_t lane64(uint64_t v, int i) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)v, i) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), i) << 32);
}
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

/* ------------------------------------------------------------------ the device handle
 * Written by the host before any kernel and never changed while one runs, so its fields are
 * read as constants: through the scalar cache, and kept in scalar registers across waits and
 * barriers. As ordinary memory each field was a vector load after every one of them: about five
 * dependent round trips a page on the hit path. */
typedef const __attribute__((address_space(4))) gfs_dev hdev;
__device__ __forceinline__ hdev* H(const gfs_dev* d) { return (hdev*)d; }
/* A function that is not inlined gets the handle's address in vector registers; it is the same
   in every lane. */
__device__ __forceinline__ const gfs_dev* uniform(const gfs_dev* d) {
  const uint64_t a = (uint64_t)d;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return (const gfs_dev*)(((uint64_t)hi << 32) | lo);
}

/* ------------------------------------------------------------------ atomics (agent scope)
 * The library's atomics are all on global memory (metadata, pinned ring): said to the compiler,
 * which otherwise emits flat accesses that also wait for LDS. */
typedef __attribute__((address_space(1))) uint64_t gu64;
typedef __attribute__((address_space(1))) uint32_t gu32;
__device__ __forceinline__ gu64* G(uint64_t* p) { return (gu64*)p; }
__device__ __forceinline__ gu32* G(uint32_t* p) { return (gu32*)p; }
__device__ __forceinline__ uint64_t ld_rlx(uint64_t* p) {
  return __hip_atomic_load(G(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_acq(uint64_t* p) {
  return __hip_atomic_load(G(p), __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void acquire_system() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, ""); }
/* Ordering without cache maintenance. An agent-scope release writes the XCD's L2 back and an
 * acquire empties it, for the sake of plain (cached) accesses, and every block of the XCD pays:
 * a miss had about fifteen of them. gread's shared data need neither. The metadata are accessed
 * by atomics only, which are performed coherently across the XCDs; frame bytes are written with
 * device-scope stores (written through) and read with device-scope loads; the ring and the
 * staged bytes in host memory are accessed with system-scope loads and stores. So "B after A"
 * needs only that A has been performed before B is issued: the wait below for a wave's
 * outstanding memory operations (with a block barrier for those of other waves), and for a
 * reader that it issues a load only once it has seen the value the load depends on. The
 * workgroup fences keep the compiler from moving memory operations across the wait.
 * Without the releases and acquires: 256 MiB through 4 KiB pages 11.7 -> 7.0 ms (pull 95 -> 29 us,
 * allocation 36 -> 9, run 7.0 -> 3.5 a miss), random 64 KiB pages 13.9 -> 10.3. */
__device__ __forceinline__ void drain_atomics() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0x0F70);   /* vmcnt(0): every load, store and atomic done */
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
__device__ __forceinline__ uint32_t ld_rlx32(uint32_t* p) {
  return __hip_atomic_load(G(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rlx(uint64_t* p, uint64_t v) {
  __hip_atomic_store(G(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rel(uint64_t* p, uint64_t v) {
  __hip_atomic_store(G(p), v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rlx32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(G(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
/* the ring in pinned host memory */
__device__ __forceinline__ uint64_t ld_host(const void* p) {
  return __hip_atomic_load((gu64*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void st_host(void* p, uint64_t v) {
  __hip_atomic_store((gu64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ bool cas64(uint64_t* p, uint64_t& expected, uint64_t desired) {
  return __hip_atomic_compare_exchange_strong(G(p), &expected, desired, __ATOMIC_ACQ_REL,
                                              __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool cas64_rlx(uint64_t* p, uint64_t& expected, uint64_t desired) {
  return __hip_atomic_compare_exchange_strong(G(p), &expected, desired, __ATOMIC_RELAXED,
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool cas32(uint32_t* p, uint32_t& expected, uint32_t desired) {
  return __hip_atomic_compare_exchange_strong(G(p), &expected, desired, __ATOMIC_ACQ_REL,
                                              __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t fadd64(uint64_t* p, uint64_t v) {
  return __hip_atomic_fetch_add(G(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
/* block-local statistics: only thread 0 of the block (lane 0 of wave 0) adds */
__device__ __forceinline__ void bcount(BlockState* bs, int c, uint64_t v) {
  /* an LDS addition that returns nothing: not waited for, unlike a load and a store */
  __hip_atomic_fetch_add(&bs->ctr[c], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

/* ------------------------------------------------------------------ waiting */
__device__ __forceinline__ void nap(uint32_t& n) {
  if (n < 8) __builtin_amdgcn_s_sleep(2);
  else if (n < 64) __builtin_amdgcn_s_sleep(16);
  else __builtin_amdgcn_s_sleep(127);
  ++n;
}
/* shorter naps for the miss lock, whose holder keeps it for a few microseconds */
__device__ __forceinline__ void nap_short(uint32_t& n) {
  if (n < 16) __builtin_amdgcn_s_sleep(2);
  else __builtin_amdgcn_s_sleep(24);
  ++n;
}
__device__ __forceinline__ bool expired(const gfs_dev* d, uint64_t t0) {
  return wall_clock64() - t0 > H(d)->timeout_ticks;
}

/* ------------------------------------------------------------------ trace */
__device__ __attribute__((noinline)) void trace_store(const gfs_dev* d, uint32_t op, uint32_t block,
                                                      uint32_t file, uint32_t page, uint32_t frame, uint32_t a,
                                                      uint64_t b) {
  const uint64_t i = fadd64(&H(d)->g->trace_n, 1);
  if (i >= H(d)->trace_cap) return;
  gfs_event* e = ((gfs_event*)H(d)->trace) + i;
  e->op = op;
  e->block = block;
  e->file = file;
  e->page = page;
  e->frame = frame;
  e->a = a;
  e->b = b;
}
__device__ __forceinline__ void trace_ev(const gfs_dev* d, uint32_t level, uint32_t op, uint32_t block,
                                         uint32_t file, uint32_t page, uint32_t frame, uint32_t a, uint64_t b) {
  if (H(d)->trace_level >= level) trace_store(d, op, block, file, page, frame, a, b);
}

/* ------------------------------------------------------------------ hashed page table
 * Two candidate buckets of 16 entries (128 B) per key; an entry is key<<24 | frame and is
 * changed only by atomics. Lookups take no lock. A file's keys are inserted only under
 * that file's miss lock, first as reservations (frame field kReserved), so one key is never
 * inserted twice; the reserving block later stores the frame into its own entry, or
 * clears it. An evicting block clears the entry of the frame it claimed. */
__device__ __forceinline__ uint64_t page_key(uint32_t file, uint64_t page) {
  return ((uint64_t)(file + 1) << GFS_KEY_PAGE_BITS) | page;
}
__device__ __forceinline__ uint64_t key_hash(uint64_t k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ull;
  k ^= k >> 33;
  return k;
}
__device__ __forceinline__ void key_buckets_m(uint32_t mask, uint64_t key, uint32_t& b1, uint32_t& b2) {
  const uint64_t h = key_hash(key);
  b1 = (uint32_t)h & mask;
  b2 = (uint32_t)(h >> 32) & mask;
  if (b2 == b1) b2 = b1 ^ 1u;
}
__device__ __forceinline__ void key_buckets(const gfs_dev* d, uint64_t key, uint32_t& b1,
                                            uint32_t& b2) {
  key_buckets_m(H(d)->nbuckets_mask, key, b1, b2);
}
__device__ __forceinline__ uint64_t* slot_ptr(const gfs_dev* d, uint32_t b1, uint32_t b2, int i) {
  return H(d)->pt + (uint64_t)(i < GFS_BUCKET_SLOTS ? b1 : b2) * GFS_BUCKET_SLOTS + (i & 15);
}

/* wave-collective: lanes 0-15 read bucket 1, lanes 16-31 bucket 2; uniform result: the
 * frame, kReserved, or -1 when absent */
__device__ __forceinline__ int32_t pt_lookup_at(uint64_t* pt, uint32_t mask, uint64_t key) {
  uint32_t b1, b2;
  key_buckets_m(mask, key, b1, b2);
  const uint32_t l = lane();
  uint64_t e = 0;
  if (l < 32) e = ld_rlx(pt + (uint64_t)(l < GFS_BUCKET_SLOTS ? b1 : b2) * GFS_BUCKET_SLOTS + (l & 15));
  const uint64_t m = __ballot(l < 32 && (e >> GFS_ENTRY_FRAME_BITS) == key);
  if (m == 0) return -1;
  const uint64_t hit = __shfl(e, __ffsll((unsigned long long)m) - 1, 64);
  return (int32_t)(hit & kFrameMask);
}
__device__ int32_t pt_lookup_wave(const gfs_dev* d, uint64_t key) {
  return pt_lookup_at(H(d)->pt, H(d)->nbuckets_mask, key);
}

/* per lane: the 32 candidate entries of a key, loaded together (one round trip) */
__device__ __forceinline__ void pt_load_lane(const gfs_dev* d, uint32_t b1, uint32_t b2,
                                             uint64_t e[2 * GFS_BUCKET_SLOTS]) {
#pragma unroll
  for (int i = 0; i < 2 * GFS_BUCKET_SLOTS; ++i) e[i] = ld_rlx(slot_ptr(d, b1, b2, i));
}

/* per lane: true if key has an entry (a frame or a reservation) */
__device__ __attribute__((noinline)) bool pt_present_lane(const gfs_dev* d, uint64_t key) {
  d = uniform(d);
  uint32_t b1, b2;
  key_buckets(d, key, b1, b2);
  uint64_t e[2 * GFS_BUCKET_SLOTS];
  pt_load_lane(d, b1, b2, e);
  bool hit = false;
#pragma unroll
  for (int i = 0; i < 2 * GFS_BUCKET_SLOTS; ++i) hit |= (e[i] >> GFS_ENTRY_FRAME_BITS) == key;
  return hit;
}

/* per lane, under key's file lock: reserve key; returns the global slot index or -1 if
 * both buckets are full */
__device__ __attribute__((noinline)) int64_t pt_reserve_lane(const gfs_dev* d, uint64_t key) {
  d = uniform(d);
  const uint64_t ent = (key << GFS_ENTRY_FRAME_BITS) | kReserved;
  uint32_t b1, b2;
  key_buckets(d, key, b1, b2);
  for (int attempt = 0; attempt < 256; ++attempt) {
    uint64_t e[2 * GFS_BUCKET_SLOTS];
    pt_load_lane(d, b1, b2, e);
    int cnt1 = 0, cnt2 = 0, f1 = -1, f2 = -1;
#pragma unroll
    for (int i = 0; i < GFS_BUCKET_SLOTS; ++i) {
      if (e[i]) ++cnt1;
      else if (f1 < 0) f1 = i;
      if (e[GFS_BUCKET_SLOTS + i]) ++cnt2;
      else if (f2 < 0) f2 = GFS_BUCKET_SLOTS + i;
    }
    int pick = cnt2 < cnt1 ? f2 : f1;   /* less loaded bucket, ties to the first */
    if (pick < 0) pick = f1 >= 0 ? f1 : f2;
    if (pick < 0) return -1;
    uint64_t expect = 0;
    uint64_t* sp = slot_ptr(d, b1, b2, pick);
    if (cas64_rlx(sp, expect, ent)) return (int64_t)(sp - H(d)->pt);
  }
  return -1;
}

/* per lane: clear the entry key -> frame (the caller owns it) */
__device__ __attribute__((noinline)) bool pt_delete_lane(const gfs_dev* d, uint64_t key, uint32_t frame) {
  d = uniform(d);
  const uint64_t ent = (key << GFS_ENTRY_FRAME_BITS) | frame;
  uint32_t b1, b2;
  key_buckets(d, key, b1, b2);
  uint64_t e[2 * GFS_BUCKET_SLOTS];
  pt_load_lane(d, b1, b2, e);
  int at = -1;
#pragma unroll
  for (int i = 0; i < 2 * GFS_BUCKET_SLOTS; ++i)
    if (at < 0 && e[i] == ent) at = i;
  if (at < 0) return false;
  uint64_t expect = ent;
  return cas64_rlx(slot_ptr(d, b1, b2, at), expect, 0ull);
}

/* ------------------------------------------------------------------ frame words */
enum { PIN_RETRY = 0, PIN_VALID = 1, PIN_FILLING = 2, PIN_ERROR = 3 };

/* Pins are counted with fetch-and-add and fetch-and-subtract, so a pin costs one atomic
 * round trip and dropping one costs none (the wave does not wait for it). Every other change
 * of a frame word is a compare-and-swap against the word just read, or an addition (the
 * allocator's CLAIMED -> FILLING step), so a pin taken and dropped at any moment is never
 * lost: a block that pins a frame which turns out not to hold its page (or is not FILLING
 * or VALID) just drops the pin again. The clock hand claims only frames with no pins. */

/* Drop a pin. Relaxed: the caller's reads of the frame have completed (a block barrier
 * waits for them) before this is issued, and unpinning publishes nothing. */
/* ------------------------------------------------------------------ evicted-after-use bits
 * One bit per page of a file: set when the clock evicts the page after it was consumed (its
 * prefetch mark cleared by a pin, or it was the demanded page). A window leaves such pages
 * out of its run, unless the demanded page (the marker page, for an asynchronous window) is
 * one of them: a page a reader consumed and the cache dropped lies behind that reader, and a
 * demanded one means the file is being read again. */
__device__ __forceinline__ uint64_t* shadow_word(const gfs_dev* d, uint32_t file, uint64_t q) {
  return H(d)->shadow + (uint64_t)file * (GFS_SHADOW_PAGES / 64) + (q >> 6);
}
__device__ __forceinline__ bool shadow_lane(const gfs_dev* d, uint32_t file, uint64_t q) {
  if (q >= GFS_SHADOW_PAGES) return false;
  return ((ld_rlx(shadow_word(d, file, q)) >> (q & 63)) & 1ull) != 0;
}
__device__ __forceinline__ void shadow_set_lane(const gfs_dev* d, uint32_t file, uint64_t q) {
  if (q < GFS_SHADOW_PAGES)
    __hip_atomic_fetch_or(G(shadow_word(d, file, q)), 1ull << (q & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void frame_unpin(const gfs_dev* d, uint32_t f) {
  __hip_atomic_fetch_sub(G(&H(d)->fword[f]), GFS_FW_PIN_ONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* The bit updates of a demand pin: set the reference bit, clear the prefetched mark (the page
   has now been demanded). Idempotent; the wave does not wait for them. */
__device__ __forceinline__ void frame_pin_bits(const gfs_dev* d, uint32_t f, uint64_t w) {
  uint64_t* fw = &H(d)->fword[f];
  if (!(w & GFS_FW_REF))
    __hip_atomic_fetch_or(G(fw), GFS_FW_REF, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (w & GFS_FW_RA)
    __hip_atomic_fetch_and(G(fw), ~GFS_FW_RA, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* Pin frame f if it is filling or valid and still holds key; sets the reference bit and
 * clears the prefetched mark (the page has now been demanded). The tag is read after the pin
 * is in place (a frame cannot be claimed while pinned). */
__device__ int frame_pin(const gfs_dev* d, uint32_t f, uint64_t key, uint64_t* w_out = nullptr) {
  uint64_t* fw = &H(d)->fword[f];
  const uint64_t w = __hip_atomic_fetch_add(G(fw), GFS_FW_PIN_ONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (w_out) *w_out = w;
  const uint64_t st = w & GFS_FW_STATE;
  if ((st != GFS_FS_FILLING && st != GFS_FS_VALID) || ld_rlx(&H(d)->ftag[f]) != key) {
    frame_unpin(d, f);
    return PIN_RETRY;
  }
  if (st == GFS_FS_VALID && (w & GFS_FW_ERR)) {
    frame_unpin(d, f);   /* the host read of this page failed */
    return PIN_ERROR;
  }
  frame_pin_bits(d, f, w);
  return st == GFS_FS_VALID ? PIN_VALID : PIN_FILLING;
}

/* Lane: the pinned frame's word showed the marker bit; clear it. True for the one block whose
   clearing took it (that block advances the stream). */
__device__ __forceinline__ bool mark_take_lane(const gfs_dev* d, uint32_t f) {
  const uint64_t old = __hip_atomic_fetch_and(G(&H(d)->fword[f]), ~GFS_FW_MARK, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (old & GFS_FW_MARK) != 0;
}

/* One clock step at frame f (per lane). FREE or EVICT leave the frame CLAIMED by the
 * caller; EVICT reports the victim's key and prefetched mark. `seen` receives what the step
 * decided on, for the trace: the reference bit << 1 | pinned << 2 | lost race << 3 |
 * state << 4 (the word was read, then a compare-and-swap against it failed: SKIP). */
__device__ int hand_visit(const gfs_dev* d, uint32_t f, uint64_t& vkey, uint32_t& vra, uint32_t& seen) {
  uint64_t* fw = &H(d)->fword[f];
  uint64_t w = ld_rlx(fw);
  const uint64_t tag = ld_rlx(&H(d)->ftag[f]);   /* loaded with the word; used only on EVICT */
  const uint64_t st = w & GFS_FW_STATE;
  const uint64_t claimed = (((w >> GFS_FW_VER_SHIFT) + 1) << GFS_FW_VER_SHIFT) | GFS_FS_CLAIMED;
  seen = ((w & GFS_FW_REF) ? 2u : 0u) | ((w & GFS_FW_PINS) ? 4u : 0u) | ((uint32_t)st << 4);
  if (w & GFS_FW_PINS) return GFS_HAND_SKIP;
  if (st == GFS_FS_FREE) {
    if (cas64_rlx(fw, w, claimed)) return GFS_HAND_FREE;
    seen |= 8u;
    return GFS_HAND_SKIP;
  }
  if (st != GFS_FS_VALID) return GFS_HAND_SKIP;
  if (w & GFS_FW_REF) {
    if (cas64_rlx(fw, w, (w & ~GFS_FW_REF) + GFS_FW_VER_ONE)) return GFS_HAND_CLEAR;
    seen |= 8u;
    return GFS_HAND_SKIP;
  }
  const uint64_t old = w;
  if (!cas64_rlx(fw, w, claimed)) {
    seen |= 8u;
    return GFS_HAND_SKIP;
  }
  /* the tag read with the word is still the frame's: a tag is rewritten only by the block
     that claims the frame, and the CAS just succeeded against the word read with it */
  vkey = tag;
  vra = (old & GFS_FW_RA) ? 1u : 0u;
  return GFS_HAND_EVICT;
}

/* Wait (lane) until the pinned frame f is VALID. 0, -EIO or -ETIMEDOUT (pin dropped on error). */
__device__ int64_t wait_valid_lane(const gfs_dev* d, uint32_t f, uint64_t t0) {
  uint32_t n = 0;
  while (true) {
    const uint64_t w = ld_rlx(&H(d)->fword[f]);
    if ((w & GFS_FW_STATE) == GFS_FS_VALID) {
      if (w & GFS_FW_ERR) {
        frame_unpin(d, f);
        return -kEIO;
      }
      return 0;
    }
    if (expired(d, t0)) {
      frame_unpin(d, f);
      return -kETIMEDOUT;
    }
    nap(n);
  }
}

/* ------------------------------------------------------------------ per-file miss lock
 * A FIFO ticket lock whose waiters can leave the queue, and whose holder decides for the
 * waiters behind it. Blocks get the lock in ticket order, which keeps the readers of a file
 * together (an unfair lock lets a few blocks run far ahead and spreads the misses over the
 * whole file). Each ticket has a 64-bit queue slot (GFS_LOCK_SLOTS per file, more than the blocks
 * the device can hold at once) and a 64-bit note. A waiter writes what the
 * detector needs of its miss into the note and then announces the page in its slot
 * ("waiting n, page"); the holder passes the lock by writing "granted n" into the slot of
 * ticket n. A waiter whose page appears in the table while it waits (another block's window
 * covered it) writes "left n" instead, by compare-and-swap against the grant, and goes to the
 * pin path. A holder that has just claimed windows marks the waiters right behind it whose
 * pages lie in them "covered n" (their pages are about to be reserved, so the lock has nothing
 * to decide for them) and passes the lock to the first ticket that is neither left nor covered.
 * Ticket 0 of a cold file holds the lock at once. The low word of every slot value carries the
 * ticket, so stale values of earlier tickets never match.
 *
 * Deciding for others: what a decision costs under the lock is round trips to memory (state,
 * table probe, write-back, hand-off), not the decision, which is a few hundred nanoseconds in
 * registers. So the holder takes up to GFS_LOCK_BATCH - 1 waiters right behind it along: it
 * turns their slots from "waiting" to "taken" (a waiter can no longer leave then) while the
 * table probes for all their pages are in flight, decides for each in ticket order on the
 * state it holds and from what each noted of its miss and its launch, exactly as if each had held
 * the lock in turn, claims their windows, writes
 * state and claims back once, and leaves each its outcome in its slot ("decided n, window" or
 * "covered n"). 256 MiB through 4 KiB pages and 64 KiB windows, 4096 decisions: 22.2 ms when each
 * decision held the lock (4.8 us of it, 5.7 with the hand-off), 11.4 with seven decided for (2.2 us
 * of it), 6.4 by now (fifteen, and no cache maintenance: 1.4 us), where the ring slots are the
 * bound. */

enum { LOCK_OWN = 0, LOCK_LEFT = 1, LOCK_TIMEOUT = 2, LOCK_COVERED = 3, LOCK_DECIDED = 4 };

/* a ticket's slot; lq: the file's slots */
__device__ __forceinline__ uint64_t* lock_slot(uint64_t* lq, uint64_t n) { return lq + lock_slot_index(n); }
__device__ __forceinline__ uint64_t* lock_queue(const gfs_dev* d, uint32_t file) {
  return H(d)->lockq + (uint64_t)file * GFS_LOCK_SLOTS;
}
__device__ __forceinline__ uint64_t* lock_note_at(const gfs_dev* d, uint32_t file, uint64_t n) {
  return H(d)->lockn + lock_note_index(file, n);
}

/* Lane 0: leave the queue if ticket t has no grant or outcome yet; true if it left, false if its
   slot says something else by now, or soon will (taken): the caller goes on polling. */
__device__ bool lock_try_leave_lane(uint64_t* sl, uint64_t t) {
  uint64_t v = ld_rlx(sl);
  while (v != lock_granted(t) && v != lock_taken(t) && (uint32_t)v != (uint32_t)lock_covered(t)) {
    if (cas64_rlx(sl, v, lock_left(t))) return true;
  }
  return false;
}

/* Wave-collective. Waits for the file's miss lock for page `page` (key `key`), or for the
 * holder's decision for it; while waiting, looks up `key` in the table now and then and leaves
 * the queue if it appeared. Returns value << 3 | LOCK_OWN (value: the ticket), LOCK_DECIDED
 * (value: the window, see lock_decided), LOCK_LEFT, LOCK_COVERED (a holder's window covers the
 * page) or LOCK_TIMEOUT (left the queue after the wait timeout): in registers, as a result
 * through memory would be loaded back with the lock held. */
__device__ __attribute__((noinline)) uint64_t lock_file_wave(const gfs_dev* d, uint32_t file, uint64_t key,
                                                             uint64_t page, uint64_t note, uint64_t t0,
                                                             bool may_leave = true) {
  d = uniform(d);
  uint64_t* const lq = lock_queue(d, file);
  uint64_t t = 0;
  if (lane() == 0)
    t = __hip_atomic_fetch_add(G(&H(d)->locks[file].next), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  t = __shfl(t, 0, 64);
  uint64_t value = t;
  int res = LOCK_OWN;
  if (t != 0) {
    uint64_t* sl = lock_slot(lq, t);
    /* announce the miss, unless the grant is already there */
    int own = 0;
    if (lane() == 0) {
      uint64_t v = ld_rlx(sl);
      if (v != lock_granted(t)) {
        if (note == kNoNote) page = kNoPage;
        else st_rlx(lock_note_at(d, file, t), lock_note_tagged(note, file, t));
        drain_atomics();   /* the note is there before the slot says so */
        while (v != lock_granted(t)) {
          if (cas64_rlx(sl, v, lock_waiting(t, page))) break;
        }
      }
      own = v == lock_granted(t) ? 1 : 0;
    }
    own = __shfl(own, 0, 64);
    for (uint32_t n = 0; !own; ++n) {
      int st = -1;   /* -1: keep waiting */
      uint64_t v = 0;
      if (lane() == 0) {
        v = ld_rlx(sl);
        if (v == lock_granted(t)) st = LOCK_OWN;
        else if ((uint32_t)v == (uint32_t)lock_covered(t)) st = (v >> 62) ? LOCK_DECIDED : LOCK_COVERED;
      }
      st = __shfl(st, 0, 64);
      if (st < 0 && (n & 7) == 7) {
        /* the page may have been reserved by a window that covers it */
        const bool present = may_leave && pt_lookup_wave(d, key) >= 0;
        const bool late = expired(d, t0);
        if (present || late) {
          int out = 0;
          if (lane() == 0) out = lock_try_leave_lane(sl, t) ? 1 : 0;
          out = __shfl(out, 0, 64);
          if (out) st = present ? LOCK_LEFT : LOCK_TIMEOUT;
        }
      }
      if (st >= 0) {
        res = st;
        if (st == LOCK_DECIDED) value = __shfl(v, 0, 64) >> 32;
        break;
      }
      if (lane() == 0) {
        if (n < 64) __builtin_amdgcn_s_sleep(2);
        else __builtin_amdgcn_s_sleep(16);
      }
    }
  }
  drain_atomics();
  return (value << 3) | (uint64_t)res;
}

/* Wave-collective: pass the lock to the first ticket from n on that is still waiting for it and
 * whose page is in none of the windows the holder has claimed: lane i's [lo, hi) for the set bits
 * i of `claimed`. Without a window ticket n gets the grant by one exchange, and only if that
 * waiter had left does the wave read the following slots, 64 at a time, for the first ticket
 * still in the queue. With windows the wave looks at the slots first: tickets that left or were
 * marked covered are passed over, waiting tickets whose announced page lies in a window are
 * marked covered (a compare-and-swap that loses only to the waiter leaving), and the first other
 * ticket gets the grant; if that waiter left just before the exchange, the scan goes on after it.
 * A ticket that has not announced its page yet is granted the lock like any other. has_pre: lane
 * l's `pre` is the value of ticket n + l's slot, read earlier under the lock (0: not read), and
 * the first look uses it instead of reading the slots again. Everything the next holder reads
 * must have been performed before the call (drain_atomics). */
__device__ __attribute__((noinline)) void unlock_slots_wave(uint64_t* lq, uint64_t n, uint64_t claimed, uint64_t lo,
                                                            uint64_t hi, bool has_pre, uint64_t pre) {
  const uint32_t l = lane();
  bool look = claimed != 0;
  while (true) {
    if (look) {
      const uint64_t nl = n + l;
      uint64_t* sl = lock_slot(lq, nl);
      uint64_t v = has_pre ? pre : ld_rlx(sl);
      has_pre = false;
      const uint64_t pg = (v >> 32) & 0x7fffffffull;
      const bool gone = v == lock_left(nl) || v == lock_covered(nl);
      const bool waits = (v >> 63) && (uint32_t)v == ((uint32_t)nl << 2);
      bool in = false;
      for (uint64_t m = claimed; m; m &= m - 1) {
        const int i = __builtin_ctzll(m);
        const uint64_t wlo = lane64(lo, i), whi = lane64(hi, i);
        in |= pg >= wlo && pg < whi;
      }
      const bool cov = waits && in;
      const uint64_t skip = __ballot(gone || cov);
      const uint32_t first = ~skip ? (uint32_t)__builtin_ctzll(~skip) : 64u;
      if (cov && l < first) {
        /* loses only to the waiter leaving, which takes it out of the queue as well */
        (void)cas64_rlx(sl, v, lock_covered(nl));
      }
      if (first == 64) {
        n += 64;
        continue;
      }
      n += first;
    }
    uint64_t old = 0;
    if (l == 0)
      old = __hip_atomic_exchange(G(lock_slot(lq, n)), lock_granted(n), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __shfl(old, 0, 64);
    if (old != lock_left(n)) return;
    ++n;   /* that waiter had left: look for the next one still in the queue */
    look = true;
  }
}
/* the same for the holder of `ticket`, with one window or none (lo == hi), no slot read yet */
__device__ __forceinline__ void unlock_file_wave(const gfs_dev* d, uint32_t file, uint64_t ticket, uint64_t lo,
                                                 uint64_t hi) {
  drain_atomics();
  unlock_slots_wave(lock_queue(d, file), ticket + 1, hi > lo ? 1 : 0, lo, hi, false, 0);
}

/* ------------------------------------------------------------------ readahead detector
 * Wave-collective, under the file's miss lock. Streams live in the file record; lane i
 * looks at stream slot i. Sec. 2.3 (Linux readahead: per-descriptor sequential streams,
 * window doubled up to a maximum, several interleaved readers followed on one file) and
 * Sec. 4 (GPU-side window, RANDOM hint disables it). A miss inside a stream's zone
 * [next, next+size) doubles that stream's window. Otherwise a new stream replaces an empty
 * or the least recently used slot: if several of the file's recent misses are near p the
 * file is being read in aggregate by many blocks and the window is the cap-sized aligned
 * chunk around p; else the history of cached pages right behind p sizes it (context
 * readahead); with neither, it opens with the initial window at offset 0 or under
 * SEQUENTIAL advice, else with one page. The context rule needs more cached history than
 * the req pages from p to the end of the read that missed (a shorter one may be a random
 * read next to cached pages), and a context or new window covers at least those req pages
 * (Sec. 2.3: the prefetcher reads at least what the caller asked for), up to the cap. */
/* Per lane: the file's detector state, loaded together (lane i: recent miss i, stream
   slot i, lanes past them a copy that is not used); the decision below uses it after the
   caller waited for it. No load depends on the lane: loads under a lane condition were waited
   for one group after the other, a round trip more with the miss lock held. */
struct RaState {
  uint32_t advice, clk, rn;
  uint64_t r, s_next;
  uint32_t s_size, s_last, s_valid, s_marker;
};
__device__ __forceinline__ RaState ra_load_lane(gfs_file_dev* fe, uint32_t nrec, uint32_t nstreams) {
  const uint32_t l = lane();
  RaState st;
  st.advice = ld_rlx32(&fe->advice);
  st.clk = ld_rlx32(&fe->clock);
  st.rn = ld_rlx32(&fe->recent_n);
  st.r = ld_rlx(&fe->recent[l < nrec ? l : 0]);
  gfs_stream* sp = &fe->streams[l < nstreams ? l : 0];
  st.s_next = ld_rlx(&sp->next);
  st.s_size = ld_rlx32(&sp->size);
  st.s_last = ld_rlx32(&sp->last_use);
  st.s_valid = ld_rlx32(&sp->valid);
  st.s_marker = ld_rlx32(&sp->marker);
  return st;
}

/* The values of a round of loads are used only from here on, after the caller's wait: without
   this the compiler put work on the first of them between the loads, and so a wait for a round
   trip before the last ones were issued. */
__device__ __forceinline__ void ra_loaded(RaState& st, uint64_t& a, uint64_t& b) {
  asm volatile("" : "+v"(st.advice), "+v"(st.clk), "+v"(st.rn), "+v"(st.r), "+v"(st.s_next), "+v"(st.s_size),
               "+v"(st.s_last), "+v"(st.s_valid), "+v"(st.s_marker), "+v"(a), "+v"(b));
}

/* Which rule decided a window (GFS_RA_RULE_*, recorded in the trace with the detector's inputs). */
enum { RA_RULE_OFF = GFS_RA_RULE_OFF, RA_RULE_ZONE = GFS_RA_RULE_ZONE, RA_RULE_AGGREGATE = GFS_RA_RULE_AGGREGATE,
       RA_RULE_CONTEXT = GFS_RA_RULE_CONTEXT, RA_RULE_NEW = GFS_RA_RULE_NEW };

/* The largest window a decision may take: the configured cap, clipped to the share of the
   cache one resident block may hold (Sec. 5.1's quota: cache pages over the blocks reading at
   once, the smaller of the launch's grid and the configured resident count), so that the
   windows of all resident readers together do not exceed the cache. */
__device__ __forceinline__ uint32_t ra_cap_eff(const gfs_dev* d) {
  const uint64_t grid = (uint64_t)gridDim.x * gridDim.y * gridDim.z;
  const uint64_t r = grid < H(d)->ra_quota_blocks ? grid : H(d)->ra_quota_blocks;
  uint64_t q = H(d)->nframes / (r ? r : 1);
  if (q < 1) q = 1;
  return H(d)->ra_cap < q ? H(d)->ra_cap : (uint32_t)q;
}

/* The detector's constants, read before a block takes the miss lock, so that the holder's
   decision waits on no load of them. */
struct RaParams {
  uint32_t cap, nrec, nstreams, near_min, init;
  uint64_t radius;
};
__device__ __forceinline__ RaParams ra_params(const gfs_dev* d) {
  RaParams q;
  q.cap = ra_cap_eff(d);
  q.nrec = H(d)->ra_recent;
  q.nstreams = H(d)->streams;
  q.near_min = H(d)->ra_near_min;
  q.init = H(d)->ra_init;
  q.radius = H(d)->ra_near_pages;
  return q;
}

/* Wave-collective: how many consecutive pages right behind p are in the table (64 per round),
 * up to max(ceil(cap / 2), min(req, cap) + 1): enough to tell whether the history is longer
 * than the read that missed (req pages from p), and to size a context window min(2h, cap).
 * The miss path counts them before it takes the file's miss lock, while it would wait
 * anyway, so the lock's holder probes no table entries for this: the count is the table as
 * the block saw it when it missed (with accesses made one at a time, the same as under the
 * lock), and the decision uses it alone. */
__device__ __attribute__((noinline)) uint32_t ra_history_wave(const gfs_dev* d, uint32_t file, uint64_t p, uint32_t req) {
  d = uniform(d);
  const uint32_t l = lane();
  const uint32_t cap = ra_cap_eff(d);
  const uint32_t r = req < cap ? req : cap;
  const uint32_t hmax = (cap + 1) / 2 > r + 1 ? (cap + 1) / 2 : r + 1;
  uint32_t h = 0;
  while (h < hmax) {
    const uint64_t back = (uint64_t)h + 1 + l;
    bool mapped = false;
    if (back <= p && h + l < hmax) mapped = pt_present_lane(d, page_key(file, p - back));
    const uint64_t m = __ballot(mapped);
    const uint32_t run = (~m == 0ull) ? 64u : (uint32_t)__builtin_ctzll(~m);
    h += run;
    if (run < 64) break;
  }
  return h < hmax ? h : hmax;
}

/* The decision, on the state in st, which it advances (clock, recent misses, the stream it
   uses); `dirty` gets this lane's parts of the state that changed: 1 recent miss, 2 stream. */
__device__ __forceinline__ void ra_decide_wave(uint64_t p, uint32_t req, uint32_t hist, const RaParams& rp, RaState& st,
                                               uint32_t& dirty, uint64_t& ws, uint32_t& wn, uint32_t& near_out,
                                               uint32_t& h_out, uint32_t& rule_out, int& slot_out) {
  ws = p;
  wn = 1;
  near_out = 0;
  h_out = 0;
  rule_out = RA_RULE_OFF;
  slot_out = -1;
  if (rp.cap == 0 || __builtin_amdgcn_readfirstlane(st.advice) == GFS_ADV_RANDOM) return;
  const uint32_t l = lane();
  const uint32_t cap = rp.cap;
  /* how many of the file's last misses lie near p; then remember p */
  const uint64_t radius = rp.radius;
  const bool near_l = l < rp.nrec && l < st.rn && st.r + radius >= p && st.r <= p + radius;
  const uint32_t near = (uint32_t)__popcll(__ballot(near_l));
  near_out = near;
  st.clk += 1;
  if (l == st.rn % rp.nrec) {
    st.r = p;
    dirty |= 1u;
  }
  st.rn += 1;
  const uint64_t cm = __ballot(l < rp.nstreams && st.s_valid && st.s_next <= p && p < st.s_next + st.s_size);
  int j;
  if (cm) {
    /* p is inside a stream's zone: double that stream's window from its frontier */
    j = __builtin_ctzll(cm);
    ws = lane64(st.s_next, j);
    const uint32_t sz = __builtin_amdgcn_readlane(st.s_size, j);
    wn = 2 * sz < cap ? 2 * sz : cap;
    if (p >= ws + wn) ws = p;   /* a zone left by a launch with a larger cap: the window must hold p */
    rule_out = RA_RULE_ZONE;
  } else {
    const uint64_t inv = __ballot(l < rp.nstreams && !st.s_valid);
    if (inv) {
      j = __builtin_ctzll(inv);
    } else {
      /* the least recently used of lanes 0-7, the lowest of equals: minimum over the eight
         lanes by three lane permutations within the vector unit */
      static_assert(GFS_MAX_STREAMS == 8, "three steps");
      const uint32_t k = l < rp.nstreams ? st.s_last : ~0u;
      uint32_t m = k;
      const auto least = [&](uint32_t o) { m = o < m ? o : m; };
      least((uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xB1, 0xf, 0xf, true));    /* quad_perm 1,0,3,2 */
      least((uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4E, 0xf, 0xf, true));    /* quad_perm 2,3,0,1 */
      least((uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x141, 0xf, 0xf, true));   /* row_half_mirror */
      const uint32_t least8 = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
      j = __builtin_ctzll(__ballot(l < rp.nstreams && k == least8));
    }
    if (near >= rp.near_min) {
      /* many blocks missing close together: the file is read in aggregate (interleaved
         strides); take the cap-sized chunk aligned around p */
      wn = cap;
      ws = p - p % cap;
      rule_out = RA_RULE_AGGREGATE;
    } else {
      /* context: the consecutive cached pages right behind p (hist, counted by
         ra_history_wave); a stream that no slot tracks shows up as that history */
      const uint32_t h = hist;
      /* a history no longer than the read itself may be chance (a random read next to
         cached pages): only a longer one makes p a stream's continuation. Either way the
         window covers at least the rest of the read that missed (req pages from p), as a
         read larger than a page asks for them all */
      const uint32_t r = req < cap ? req : cap;
      uint32_t w0;
      if (h > r) {
        w0 = 2 * h;
        rule_out = RA_RULE_CONTEXT;
      } else {
        w0 = (p == 0 || st.advice == GFS_ADV_SEQUENTIAL) ? rp.init : 1u;
        rule_out = RA_RULE_NEW;
      }
      if (w0 < r) w0 = r;
      if (w0 > cap) w0 = cap;
      if (w0 < 1) w0 = 1;
      ws = p;
      wn = w0;
      h_out = h;
    }
  }
  if ((int)l == j) {
    st.s_next = ws + wn;
    st.s_size = wn;
    st.s_last = st.clk;
    st.s_valid = 1u;
    dirty |= 2u;
  }
  slot_out = j;
}
/* Write back what decisions changed. */
__device__ __forceinline__ void ra_store_lane(gfs_file_dev* fe, const RaState& st, uint32_t dirty, bool async_on) {
  const uint32_t l = lane();
  if (dirty & 1u) st_rlx(&fe->recent[l], st.r);
  if (dirty & 2u) {
    gfs_stream* sp = &fe->streams[l];
    st_rlx(&sp->next, st.s_next);
    st_rlx32(&sp->size, st.s_size);
    st_rlx32(&sp->last_use, st.s_last);
    st_rlx32(&sp->valid, st.s_valid);
    if (async_on) st_rlx32(&sp->marker, st.s_marker);
  }
  if (l == 0) {
    st_rlx32(&fe->clock, st.clk);
    st_rlx32(&fe->recent_n, st.rn);
  }
}

/* ------------------------------------------------------------------ clock allocation
 * Wave-collective, outside the miss lock. Gives frames to bs->list[0..n) in order: each
 * round takes as many consecutive hand tickets as pages remain, visits those frames in
 * parallel, and hands the k-th successful ticket to the next unserved page, which is the
 * order a one-at-a-time hand would produce. Each page that gets a frame is tagged, made
 * FILLING (pinned for the demanded page, marked prefetched otherwise) and its reserved
 * table entry is pointed at the frame. Returns how many pages got frames (a prefix of the
 * list); stops after 2 * nframes visits without enough frames. */
__device__ __attribute__((noinline)) uint32_t alloc_wave(const gfs_dev* d, uint32_t file, uint64_t demand, BlockState* bs,
                               uint32_t n, uint32_t bid, uint64_t mark = ~0ull) {
  d = uniform(d);
  const uint32_t l = lane();
  uint32_t assigned = 0;
  uint64_t visits = 0;
  uint32_t evicted = 0, wasted = 0;
  const uint64_t limit = 2ull * H(d)->nframes;
  while (assigned < n && visits < limit) {
    const uint32_t need = (n - assigned) < 64u ? (n - assigned) : 64u;
    uint64_t base = 0;
    if (l == 0) base = fadd64(&H(d)->g->hand, need);
    base = __shfl(base, 0, 64);
    int act = -1;
    uint32_t f = 0;
    uint64_t vkey = 0;
    uint32_t vra = 0, seen = 0;
    const uint64_t t = base + l;
    if (l < need) {
      f = (uint32_t)(t % H(d)->nframes);
      act = hand_visit(d, f, vkey, vra, seen);
      if (act == GFS_HAND_EVICT) {
        const uint32_t vf = (uint32_t)(vkey >> GFS_KEY_PAGE_BITS) - 1u;
        const uint32_t vp = (uint32_t)(vkey & ((1ull << GFS_KEY_PAGE_BITS) - 1));
        trace_ev(d, 1, GFS_EV_HAND, bid, vf, vp, f, GFS_HAND_EVICT | (vra << 8) | (seen << 8), t);
      } else {
        trace_ev(d, 1, GFS_EV_HAND, bid, 0xffffffffu, 0xffffffffu, f, (uint32_t)act | (seen << 8), t);
      }
    }
    const bool ok = (act == GFS_HAND_FREE || act == GFS_HAND_EVICT);
    const uint64_t sm = __ballot(ok);
    evicted += (uint32_t)__popcll(__ballot(act == GFS_HAND_EVICT));
    wasted += (uint32_t)__popcll(__ballot(act == GFS_HAND_EVICT && vra));
    if (ok) {
      const uint32_t k = assigned + (uint32_t)__popcll(sm & lanemask_lt());
      const uint64_t q = bs->list[k];
      if (act == GFS_HAND_EVICT) {
        pt_delete_lane(d, vkey, f);
        if (!vra)
          shadow_set_lane(d, (uint32_t)(vkey >> GFS_KEY_PAGE_BITS) - 1u, vkey & ((1ull << GFS_KEY_PAGE_BITS) - 1));
      }
      const uint64_t key = page_key(file, q);
      st_rlx(&H(d)->ftag[f], key);
      st_rlx(&H(d)->ffill[f], 0ull);   /* the request that fills it is not known yet */
      /* CLAIMED (no flags, no pins of ours) -> FILLING, version + 1, pinned for the demanded
         page, prefetched mark otherwise; an addition keeps pins other blocks hold briefly */
      const uint64_t delta = (GFS_FS_FILLING - GFS_FS_CLAIMED) + GFS_FW_VER_ONE +
                             (q == demand ? GFS_FW_PIN_ONE : GFS_FW_RA) + (q == mark ? GFS_FW_MARK : 0ull);
      drain_atomics();   /* tag and fill word before FILLING, FILLING before the table entry */
      __hip_atomic_fetch_add(G(&H(d)->fword[f]), delta, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      drain_atomics();
      st_rlx(H(d)->pt + bs->lslot[k], (key << GFS_ENTRY_FRAME_BITS) | f);
      bs->lframe[k] = f;
      trace_ev(d, 1, GFS_EV_ALLOC, bid, file, (uint32_t)q, f, q == demand ? 0u : 1u, t);
    }
    if (l == 0) bcount(bs, GFS_C_HAND, need);
    assigned += (uint32_t)__popcll(sm);
    visits += need;
  }
  if (l == 0) {
    bcount(bs, GFS_C_EVICTIONS, evicted);
    bcount(bs, GFS_C_WASTED, wasted);
  }
  wave_sync_lds();
  return assigned;
}

/* ------------------------------------------------------------------ vector copy */
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(1))) v4u gv4u;

/* Eight 16-byte units from staging (host memory: system-scope loads, which take nothing an earlier
 * use of the slot left in a cache) to a frame (device-scope stores, written through to memory for
 * readers of other XCDs). All eight loads are issued before the first is waited for, in the
 * statement itself; units not in `ok` are loaded from a readable address and not stored. */
__device__ __forceinline__ void copy_in8(uint8_t* const (&to)[8], const uint8_t* const (&from)[8], uint32_t ok) {
  v4u a[8];
  asm volatile("global_load_dwordx4 %0, %8, off sc0 sc1\n\t"
               "global_load_dwordx4 %1, %9, off sc0 sc1\n\t"
               "global_load_dwordx4 %2, %10, off sc0 sc1\n\t"
               "global_load_dwordx4 %3, %11, off sc0 sc1\n\t"
               "global_load_dwordx4 %4, %12, off sc0 sc1\n\t"
               "global_load_dwordx4 %5, %13, off sc0 sc1\n\t"
               "global_load_dwordx4 %6, %14, off sc0 sc1\n\t"
               "global_load_dwordx4 %7, %15, off sc0 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(a[4]), "=&v"(a[5]), "=&v"(a[6]), "=&v"(a[7])
               : "v"(from[0]), "v"(from[1]), "v"(from[2]), "v"(from[3]), "v"(from[4]), "v"(from[5]), "v"(from[6]), "v"(from[7])
               : "memory");
#pragma unroll
  for (uint32_t j = 0; j < 8; ++j)
    if ((ok >> j) & 1)   /* the pause keeps the data registers until the store has read them */
      asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(to[j]), "v"(a[j]) : "memory");
}

/* Block-cooperative copy_in8 of n bytes, rounded up to 16 (both sides hold whole pages); both
 * pointers 16-byte aligned. */
__device__ __attribute__((noinline)) void copy_in(uint8_t* dst, const uint8_t* src, uint64_t n, uint32_t tid,
                                                  uint32_t nt) {
  const uint64_t n16 = (n + 15) >> 4;
  for (uint64_t i = tid; i < n16; i += 8ull * nt) {
    uint8_t* to[8];
    const uint8_t* from[8];
    uint32_t ok = 0;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const uint64_t u = i + (uint64_t)j * nt;
      if (u < n16) ok |= 1u << j;
      from[j] = src + ((u < n16 ? u : i) << 4);
      to[j] = dst + (u << 4);
    }
    copy_in8(to, from, ok);
  }
}

/* ------------------------------------------------------------------ reading frames
 * A frame is written by blocks of any XCD and reused for page after page, and the XCDs' L2s do
 * not follow each other's writes. Its bytes are read with device-scope loads (sc1), which do
 * not take a line another XCD has replaced, so a pin needs no acquire. With one per
 * hit, emptying the XCD's L2 each time, 256 MiB of cached 4 KiB pages in 128 KiB reads took
 * 253 us instead of 165, 4080-byte records 332 instead of 273. The loads go out after the pin's
 * result was seen (and a block barrier for the other waves), and the bytes reached memory before
 * the frame was published. They are nontemporal as well: page bytes pass once.
 * N loads of 16 bytes at any alignment, issued together and waited for in the same statement;
 * every address must be readable. */
template <int N>
__device__ __forceinline__ void ld_frame(v4u (&a)[N], const uint8_t* const (&p)[N]) {
  static_assert(N == 1 || N == 2 || N == 4 || N == 8, "loads issued together");
  if constexpr (N == 1) {
    asm volatile("global_load_dwordx4 %0, %1, off sc1 nt\n\ts_waitcnt vmcnt(0)" : "=&v"(a[0]) : "v"(p[0]) : "memory");
  } else if constexpr (N == 2) {
    asm volatile("global_load_dwordx4 %0, %2, off sc1 nt\n\t"
                 "global_load_dwordx4 %1, %3, off sc1 nt\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(a[0]), "=&v"(a[1]) : "v"(p[0]), "v"(p[1]) : "memory");
  } else if constexpr (N == 4) {
    asm volatile("global_load_dwordx4 %0, %4, off sc1 nt\n\t"
                 "global_load_dwordx4 %1, %5, off sc1 nt\n\t"
                 "global_load_dwordx4 %2, %6, off sc1 nt\n\t"
                 "global_load_dwordx4 %3, %7, off sc1 nt\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
                 : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]) : "memory");
  } else {
    asm volatile("global_load_dwordx4 %0, %8, off sc1 nt\n\t"
                 "global_load_dwordx4 %1, %9, off sc1 nt\n\t"
                 "global_load_dwordx4 %2, %10, off sc1 nt\n\t"
                 "global_load_dwordx4 %3, %11, off sc1 nt\n\t"
                 "global_load_dwordx4 %4, %12, off sc1 nt\n\t"
                 "global_load_dwordx4 %5, %13, off sc1 nt\n\t"
                 "global_load_dwordx4 %6, %14, off sc1 nt\n\t"
                 "global_load_dwordx4 %7, %15, off sc1 nt\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(a[4]), "=&v"(a[5]), "=&v"(a[6]), "=&v"(a[7])
                 : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7]) : "memory");
  }
}
typedef __attribute__((address_space(1))) uint8_t gu8;
__device__ __forceinline__ uint8_t ld_frame_byte(const uint8_t* p) {
  return __hip_atomic_load((const gu8*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* One round of a copy of n16 16-byte units: units i, i + nt, ... (N of them) of this thread.
   Loads past the last unit read it again and are not stored. */
template <int N>
__device__ __forceinline__ void copy_round(gv4u* o, const uint8_t* src, uint32_t i, uint32_t n16, uint32_t nt) {
  v4u a[N];
  const uint8_t* p[N];
#pragma unroll
  for (uint32_t k = 0; k < N; ++k) {
    const uint32_t u = i + k * nt;
    p[k] = src + ((uint64_t)(u < n16 ? u : n16 - 1) << 4);
  }
  ld_frame(a, p);
#pragma unroll
  for (uint32_t k = 0; k < N; ++k)
    if (i + k * nt < n16) o[i + k * nt] = a[k];
}

/* The copy-out of n bytes of one frame to a user buffer, both at any alignment: 16-byte stores
 * aligned in dst, loads from wherever the bytes lie in the frame (the memory unit splits one
 * that crosses lines), the fewer than 16 bytes before and after them one byte a thread. Eight
 * loads a thread are in flight, in the last round as many as it needs. */
__device__ __forceinline__ void copy_out(uint8_t* dst, const uint8_t* src, uint32_t n, uint32_t tid, uint32_t nt) {
  uint32_t head = (0u - (uint32_t)(uintptr_t)dst) & 15u;
  if (head > n) head = n;
  const uint32_t tail = (n - head) & 15u;
  if (head | tail) {
    const uint32_t e = tid < 16 ? tid : n - tail + (tid - 16);
    if (tid < head || (tid >= 16 && tid - 16 < tail)) ((gu8*)dst)[e] = ld_frame_byte(src + e);
  }
  const uint32_t n16 = (n - head) >> 4;
  src += head;
  gv4u* o = (gv4u*)(dst + head);
  uint32_t i0 = 0;   /* the same in every thread */
  for (; i0 + 4 * nt < n16; i0 += 8 * nt) copy_round<8>(o, src, i0 + tid, n16, nt);
  if (i0 + 2 * nt < n16) copy_round<4>(o, src, i0 + tid, n16, nt);
  else if (i0 + nt < n16) copy_round<2>(o, src, i0 + tid, n16, nt);
  else if (i0 < n16) copy_round<1>(o, src, i0 + tid, n16, nt);
}

/* Lane: this block holds a pin on frame f (page p), which another block's request is
 * filling. Wait for it to become VALID; meanwhile, once the request's host read is done,
 * try to take over copying this frame's bytes from staging (the PULL bit), so that blocks
 * waiting on a large window pull its pages in parallel. Leaves in bs: status, frame, and
 * pull = 2 with slot/gen/first_page/result when this block must pull frame f. */
__device__ __attribute__((noinline)) void join_or_help_lane(const gfs_dev* d, uint32_t f, uint64_t p, uint64_t t0,
                                  BlockState* bs) {
  d = uniform(d);
  uint64_t* fw = &H(d)->fword[f];
  uint32_t n = 0;
  bs->frame = (int32_t)f;
  bs->pull = 0;
  while (true) {
    uint64_t w = ld_rlx(fw);
    if ((w & GFS_FW_STATE) == GFS_FS_VALID) {
      if (w & GFS_FW_ERR) {
        frame_unpin(d, f);
        bs->status = -kEIO;
      } else {
        bs->status = 0;
      }
      return;
    }
    if (!(w & GFS_FW_PULL)) {
      const uint64_t ff = ld_rlx(&H(d)->ffill[f]);
      if (ff >> 63) {
        /* an asynchronous request: nobody publishes it, so look at the host's completion in
           the ring slot itself (the slot cannot be reused while this frame is filling) */
        const uint32_t s = (uint32_t)((ff >> 40) & 0x7fffff) - 1;
        const uint64_t gen = ff & ((1ull << 40) - 1);
        gfs_rpc_slot* rs = &H(d)->ring[s];
        if (ld_host(&rs->done_seq) == gen) {   /* the staged bytes and the result were written before it */
          if (cas64_rlx(fw, w, (w | GFS_FW_PULL) + GFS_FW_VER_ONE)) {
            bs->status = 0;
            bs->pull = 2;
            bs->slot = s;
            bs->gen = gen;
            bs->first_page = ld_host(&rs->offset) >> H(d)->page_shift;
            bs->result = (int64_t)ld_host(&rs->result);
            bs->help_page = (uint32_t)p;
            return;
          }
          continue;
        }
      } else if (ff) {
        const uint32_t s = (uint32_t)(ff >> 40) - 1;
        gfs_req_dev* rq = &H(d)->reqd[s];
        const uint64_t ready = ld_rlx(&rq->ready);
        if (ready != 0 && (ready & ((1ull << 40) - 1)) == (ff & ((1ull << 40) - 1))) {
          /* the request record was written before ready */
          if (cas64_rlx(fw, w, (w | GFS_FW_PULL) + GFS_FW_VER_ONE)) {
            bs->status = 0;
            bs->pull = 2;
            bs->slot = s;
            bs->gen = ready;
            bs->first_page = ld_rlx(&rq->first_page);
            bs->result = (int64_t)ld_rlx((uint64_t*)&rq->result);
            bs->help_page = (uint32_t)p;
            return;
          }
          continue;
        }
      }
    }
    if (expired(d, t0)) {
      frame_unpin(d, f);
      bcount(bs, GFS_C_TIMEOUTS, 1);
      bs->status = -kETIMEDOUT;
      return;
    }
    nap(n);
  }
}

/* Wave-collective, under the file's miss lock, for a window of at most 64 pages with p
 * absent: find the run of absent pages around p inside [ws, ws + wn) and reserve them.
 * Lane i loads both buckets of page ws + i once; the run is read off the ballot of
 * present pages; each run lane takes a free entry of its less loaded bucket from the
 * loaded copy with one compare-and-swap (and reloads only if that swap loses a race).
 * Fills bs->list/lslot/lframe in allocation order (p first, then the rest ascending);
 * returns the run length and sets failed if some page found both buckets full. */
__device__ uint32_t reserve_run_small_wave(const gfs_dev* d, uint32_t file, uint64_t p, uint64_t ws,
                                           uint32_t wn, BlockState* bs, uint32_t& failed) {
  const uint32_t l = lane();
  const uint64_t q = ws + l;
  const uint64_t key = page_key(file, q);
  const uint64_t ent = (key << GFS_ENTRY_FRAME_BITS) | kReserved;
  uint32_t b1 = 0, b2 = 0;
  uint64_t e[2 * GFS_BUCKET_SLOTS];
  bool present = false, gone = false;
  if (l < wn) {
    key_buckets(d, key, b1, b2);
    pt_load_lane(d, b1, b2, e);
    gone = shadow_lane(d, file, q);
#pragma unroll
    for (int i = 0; i < 2 * GFS_BUCKET_SLOTS; ++i) present |= (e[i] >> GFS_ENTRY_FRAME_BITS) == key;
  }
  const uint32_t pi = (uint32_t)(p - ws);
  uint64_t pm = __ballot(l < wn && present);
  const uint64_t gm = __ballot(gone);
  if (((gm >> pi) & 1ull) == 0) pm |= gm;     /* pages evicted after use stop it, unless p is one */
  if (wn < 64) pm |= ~0ull << wn;             /* pages outside the window stop the run */
  pm &= ~(1ull << pi);                         /* p itself is absent (probed under the lock) */
  const uint64_t below = pm & ((1ull << pi) - 1);
  const uint64_t above = pi == 63 ? 0ull : (pm >> (pi + 1)) << (pi + 1);
  const uint32_t a = below ? 64u - (uint32_t)__builtin_clzll(below) : 0u;
  const uint32_t b = above ? (uint32_t)__builtin_ctzll(above) - 1u : 63u;
  const uint32_t n = b - a + 1;
  uint32_t bad = 0;
  if (l >= a && l <= b) {
    const uint32_t i = l == pi ? 0u : (l < pi ? l - a + 1 : l - a);
    int64_t slot = -1;
    int cnt1 = 0, cnt2 = 0, f1 = -1, f2 = -1;
#pragma unroll
    for (int k = 0; k < GFS_BUCKET_SLOTS; ++k) {
      if (e[k]) ++cnt1;
      else if (f1 < 0) f1 = k;
      if (e[GFS_BUCKET_SLOTS + k]) ++cnt2;
      else if (f2 < 0) f2 = GFS_BUCKET_SLOTS + k;
    }
    int pick = cnt2 < cnt1 ? f2 : f1;
    if (pick < 0) pick = f1 >= 0 ? f1 : f2;
    if (pick >= 0) {
      uint64_t expect = 0;
      uint64_t* sp = slot_ptr(d, b1, b2, pick);
      if (cas64_rlx(sp, expect, ent)) slot = (int64_t)(sp - H(d)->pt);
      else slot = pt_reserve_lane(d, key);    /* the entry was taken meanwhile: reload */
    }
    bs->list[i] = (uint32_t)q;
    bs->lslot[i] = slot < 0 ? 0xffffffffu : (uint32_t)slot;
    bs->lframe[i] = GFS_NO_FRAME;
    bad = slot < 0 ? 1u : 0u;
  }
  failed = bad;
  return n;
}

/* ------------------------------------------------------------------ ring slots
 * Ticketed requests use the first S = sync_slots slots. Shared ring (default): one ticket
 * counter, ticket t uses slot t mod S in generation t / S + 1. Partitioned (GPUfs's queue):
 * block b always posts into slot b mod S, whose own counter gives the generation; the ticket
 * is then (generation - 1) * S + slot, so the same two helpers recover slot and generation.
 * The remaining slots belong to asynchronous windows: a window takes a free one without
 * waiting (or is not issued), because its pages are pulled only when readers reach them, and a
 * ticketed request queued behind such a slot could wait for readers that wait for it. */
__device__ __forceinline__ void ring_ticket_lane(const gfs_dev* d, uint32_t bid, uint64_t& tk) {
  const uint32_t S = H(d)->sync_slots;
  if (H(d)->partitioned) {
    const uint32_t s = bid % S;
    tk = fadd64(&H(d)->slot_tail[s], 1) * S + s;
  } else {
    tk = fadd64(&H(d)->g->ring_tail, 1);
  }
}
__device__ __forceinline__ uint32_t ring_slot(const gfs_dev* d, uint32_t, uint64_t tk) {
  return (uint32_t)(tk % H(d)->sync_slots);
}
__device__ __forceinline__ uint64_t ring_gen(const gfs_dev* d, uint64_t tk) { return tk / H(d)->sync_slots + 1; }

/* Wave: write a request into ring slot rs and post it as generation gen. Four lanes' words go
 * over the host link as one write: every write takes the slot's line away from the host threads
 * that poll it, and a look over the whole ring stalls on each line that went. Random 64 KiB
 * pages 10.0 -> 9.5 ms against five writes a request, 4 KiB pages through 64 KiB windows
 * 7.15 -> 6.85. */
__device__ __forceinline__ void post_request_wave(gfs_rpc_slot* rs, uint32_t file, uint32_t npages, uint64_t off0,
                                                  uint64_t len, uint64_t tk, uint64_t gen) {
  constexpr size_t at = offsetof(gfs_rpc_slot, file_id);
  static_assert(offsetof(gfs_rpc_slot, npages) == at + 4 && offsetof(gfs_rpc_slot, offset) == at + 8 &&
                offsetof(gfs_rpc_slot, length) == at + 16 && offsetof(gfs_rpc_slot, ticket) == at + 24 && at % 8 == 0,
                "four words");
  const uint32_t l = lane();
  const uint64_t v = l == 0 ? (uint64_t)file | ((uint64_t)npages << 32) : l == 1 ? off0 : l == 2 ? len : tk;
  if (l < 4) st_host((uint64_t*)&rs->file_id + l, v);
  drain_atomics();
  if (l == 0) st_host(&rs->req_seq, gen);
}

/* Lane: take a free slot of the asynchronous windows (busy 0 -> 1), starting at the block's
   own; -1 if every one is held. The slot's next generation is one past its last completed. */
__device__ int32_t async_slot_take_lane(const gfs_dev* d, uint32_t bid) {
  const uint32_t A = H(d)->rpc_slots - H(d)->sync_slots;
  for (uint32_t i = 0; i < A; ++i) {
    const uint32_t s = H(d)->sync_slots + (bid + i) % A;
    uint64_t* b = &H(d)->reqd[s].busy;
    uint64_t z = 0;
    if (ld_rlx(b) == 0 && cas64_rlx(b, z, 1ull)) return (int32_t)s;
  }
  return -1;
}

/* ------------------------------------------------------------------ private policy
 * The paper's design (Sec. 4.1 and Sec. 5.1). A miss reserves the one page in the table
 * without the file's lock (reserve_unique_wave); the frame comes from the block's own share
 * of the frames,
 * least recently allocated first (a frame another block has pinned is passed over); the
 * bytes come from the block's private buffer if it holds the page, else from a host read of
 * the page plus the static prefetch size, whose tail becomes the new private buffer. */

__device__ int64_t reserve_unique_wave(const gfs_dev* d, uint64_t key);

/* Lane: claim frame f of the block's share: FREE, or VALID with no pins (its page is
   evicted; the reference bit plays no part). CLAIMED on success. */
__device__ int lra_visit(const gfs_dev* d, uint32_t f, uint64_t& vkey, uint32_t& vra) {
  uint64_t* fw = &H(d)->fword[f];
  uint64_t w = ld_rlx(fw);
  const uint64_t tag = ld_rlx(&H(d)->ftag[f]);
  const uint64_t st = w & GFS_FW_STATE;
  const uint64_t claimed = (((w >> GFS_FW_VER_SHIFT) + 1) << GFS_FW_VER_SHIFT) | GFS_FS_CLAIMED;
  if (w & GFS_FW_PINS) return GFS_HAND_SKIP;
  if (st == GFS_FS_FREE) return cas64_rlx(fw, w, claimed) ? GFS_HAND_FREE : GFS_HAND_SKIP;
  if (st != GFS_FS_VALID) return GFS_HAND_SKIP;
  const uint64_t old = w;
  if (!cas64_rlx(fw, w, claimed)) return GFS_HAND_SKIP;
  vkey = tag;
  vra = (old & GFS_FW_RA) ? 1u : 0u;
  return GFS_HAND_EVICT;
}

/* Wave 0: the miss path of the private policy. 0: done (bs filled in), 1: look again,
   2: timed out. */
__device__ __attribute__((noinline)) int miss_private_wave(const gfs_dev* d, uint32_t file, uint64_t p, uint64_t key, uint64_t fsize,
                                 BlockState* bs, uint32_t bid, uint64_t t0) {
  d = uniform(d);
  const uint32_t l = lane();
  /* the page's table entry, made unique without the file's lock (the policy decides nothing
     under it: the window is the static prefetch after p, into the block's own buffer) */
  const uint64_t tr0 = wall_clock64();
  const int64_t slot = reserve_unique_wave(d, key);
  if (l == 0) bcount(bs, GFS_T_RUN, wall_clock64() - tr0);
  if (slot == -1) return 1;   /* another block's entry: go to the pin path */
  if (slot < 0) {
    /* both buckets of the key are full: reservations of misses in flight come and go, so
       back off and look again; only a table still full at the wait limit is an error */
    if (!expired(d, t0)) {
      if (l == 0) {
        bcount(bs, GFS_C_RETRIES, 1);
        nap(bs->naps);
      }
      return 1;
    }
    if (l == 0) {
      bs->status = -kENOSPC;
      bs->pull = 0;
      bs->frame = -1;
    }
    return 0;
  }
  int status = 0, asked = 0;
  uint64_t tk = 0;
  const uint64_t npages = H(d)->files[file].npages;
  const uint32_t cap = H(d)->ra_cap;
  const uint32_t span = (uint32_t)((npages - p) < (uint64_t)(1 + cap) ? (npages - p) : (uint64_t)(1 + cap));
  if (l == 0) {
    gfs_pslot* ps = &H(d)->pslots[bs->pslot];
    const bool in_pb = ps->n && ps->file == file && ps->first <= p && p < ps->first + ps->n;
    trace_ev(d, 1, GFS_EV_MISS, bid, file, (uint32_t)p, 0, in_pb ? 1u : span, p);
    /* a frame of the block's share, least recently allocated first */
    const uint64_t ta0 = wall_clock64();
    const uint32_t q = H(d)->quota;
    const uint32_t base = (uint32_t)bs->pslot * q;
    int32_t fr = -1;
    for (uint32_t i = 0; i < 2 * q && fr < 0; ++i) {
      const uint32_t idx = ps->lra_next;
      ps->lra_next = idx + 1 == q ? 0 : idx + 1;
      const uint32_t f = base + idx;
      uint64_t vkey = 0;
      uint32_t vra = 0;
      const int act = lra_visit(d, f, vkey, vra);
      if (act == GFS_HAND_EVICT) {
        pt_delete_lane(d, vkey, f);
        bcount(bs, GFS_C_EVICTIONS, 1);
        const uint32_t vf = (uint32_t)(vkey >> GFS_KEY_PAGE_BITS) - 1u;
        const uint32_t vp = (uint32_t)(vkey & ((1ull << GFS_KEY_PAGE_BITS) - 1));
        trace_ev(d, 1, GFS_EV_HAND, bid, vf, vp, f, GFS_HAND_EVICT, idx);
      } else if (act == GFS_HAND_SKIP) {
        trace_ev(d, 1, GFS_EV_HAND, bid, 0xffffffffu, 0xffffffffu, f, GFS_HAND_SKIP, idx);
      }
      if (act == GFS_HAND_FREE || act == GFS_HAND_EVICT) fr = (int32_t)f;
    }
    bcount(bs, GFS_C_HAND, 1);
    if (fr < 0) {
      /* every frame of the share is pinned by other blocks: give the page back, retry */
      st_rlx(H(d)->pt + slot, 0ull);
      bcount(bs, GFS_C_NOFRAME, 1);
      status = 1;
    } else {
      st_rlx(&H(d)->ftag[fr], key);
      st_rlx(&H(d)->ffill[fr], 0ull);
      drain_atomics();   /* tag and fill word before FILLING, FILLING before the table entry */
      __hip_atomic_fetch_add(G(&H(d)->fword[fr]), (GFS_FS_FILLING - GFS_FS_CLAIMED) + GFS_FW_VER_ONE + GFS_FW_PIN_ONE,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      drain_atomics();
      st_rlx(H(d)->pt + slot, (key << GFS_ENTRY_FRAME_BITS) | (uint64_t)fr);
      trace_ev(d, 1, GFS_EV_ALLOC, bid, file, (uint32_t)p, (uint32_t)fr, 0, (uint64_t)ps->lra_next);
      bcount(bs, GFS_T_ALLOC, wall_clock64() - ta0);
      bcount(bs, GFS_C_MISSES, 1);
      bs->frame = fr;
      bs->file = file;
      bs->status = 0;
      if (in_pb) {
        trace_ev(d, 1, GFS_EV_PBHIT, bid, file, (uint32_t)p, (uint32_t)fr, 0, 0);
        bcount(bs, GFS_C_PB_HITS, 1);
        bs->pull = 3;
        bs->help_page = (uint32_t)p;
      } else {
        /* one request: the page and the prefetch that follows it, posted below */
        ring_ticket_lane(d, bid, tk);
        const uint32_t s = ring_slot(d, bid, tk);
        const uint64_t gen = ring_gen(d, tk);
        uint32_t nn = 0;
        const uint64_t ts0 = wall_clock64();
        while (ld_rlx(&H(d)->slot_free[s]) != gen - 1) {
          if (expired(d, t0)) {
            status = 2;
            break;
          }
          nap(nn);
        }
        bcount(bs, GFS_T_SLOT, wall_clock64() - ts0);
        asked = 1;
      }
    }
  }
  status = __shfl(status, 0, 64);
  if (__shfl(asked, 0, 64)) {
    tk = __shfl(tk, 0, 64);
    const uint32_t s = ring_slot(d, bid, tk);
    const uint64_t gen = ring_gen(d, tk);
    gfs_rpc_slot* rs = &H(d)->ring[s];
    const uint64_t off0 = p << H(d)->page_shift;
    uint64_t len = (uint64_t)span << H(d)->page_shift;
    if (off0 + len > fsize) len = fsize - off0;
    if (status == 0) post_request_wave(rs, file, span, off0, len, tk, gen);
    if (l == 0) {
      if (status == 0) {
        trace_ev(d, 1, GFS_EV_REQ, bid, file, (uint32_t)p, GFS_NO_FRAME, span, tk);
        bcount(bs, GFS_C_REQUESTS, 1);
        bcount(bs, GFS_C_REQ_BYTES, len);
        bcount(bs, GFS_C_FETCHED, 1);
        uint32_t nn = 0;
        const uint64_t th0 = wall_clock64();
        while (ld_host(&rs->done_seq) != gen) {
          if (expired(d, t0)) {
            status = 2;
            break;
          }
          nap(nn);
        }
        bcount(bs, GFS_T_HOST, wall_clock64() - th0);
        if (status == 0) bs->result = (int64_t)ld_host(&rs->result);
      }
      if (status == 0) {
        bs->pull = 4;
        bs->slot = s;
        bs->gen = gen;
        bs->first_page = p;
        bs->list_n = span;
      } else {
        /* the frame stays FILLING with the pin; the cache must be reset after a timeout */
        bs->status = -kETIMEDOUT;
        bs->pull = 0;
        bcount(bs, GFS_C_TIMEOUTS, 1);
      }
    }
    status = __shfl(status, 0, 64);
  }
  if (status == 1) {
    if (expired(d, t0)) return 2;
    if (l == 0) nap(bs->naps);
    return 1;
  }
  return 0;
}

/* Wave 0, after the run's pages got frames (bs->list/lframe[0..got), the demanded page first):
 * post one request for the span of those pages, tell blocks waiting on its frames which request
 * fills them, wait for the host, and publish the finished read for the helpers. Leaves in bs:
 * status, the demanded page's frame, pull = 1 (this block pulls the request). Returns 0. */
__device__ __attribute__((noinline)) int post_wait_wave(const gfs_dev* d, uint32_t file, uint64_t fsize, BlockState* bs, uint32_t bid,
                              uint64_t t0, uint32_t got) {
  d = uniform(d);
  const uint32_t l = lane();
  /* span of the pages that got frames: p and a contiguous piece of the run */
  uint64_t lo = ~0ull, hi = 0;
  for (uint32_t k = l; k < got; k += 64) {
    const uint64_t q = bs->list[k];
    lo = q < lo ? q : lo;
    hi = q > hi ? q : hi;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t olo = __shfl_xor(lo, off, 64), ohi = __shfl_xor(hi, off, 64);
    lo = olo < lo ? olo : lo;
    hi = ohi > hi ? ohi : hi;
  }
  /* post the request for the span [lo, hi] and wait for the host */
  const uint32_t span = (uint32_t)(hi - lo + 1);
  const uint64_t off0 = lo << H(d)->page_shift;
  uint64_t len = (uint64_t)span << H(d)->page_shift;
  if (off0 + len > fsize) len = fsize - off0;
  int64_t status = 0;
  uint64_t tk = 0;
  if (l == 0) {
    ring_ticket_lane(d, bid, tk);
    const uint32_t s = ring_slot(d, bid, tk);
    const uint64_t gen = ring_gen(d, tk);
    uint32_t nn = 0;
    const uint64_t ts0 = wall_clock64();
    while (ld_rlx(&H(d)->slot_free[s]) != gen - 1) {
      if (expired(d, t0)) {
        status = -kETIMEDOUT;
        break;
      }
      nap(nn);
    }
    bcount(bs, GFS_T_SLOT, wall_clock64() - ts0);
  }
  status = __shfl(status, 0, 64);
  tk = __shfl(tk, 0, 64);
  const uint32_t s = ring_slot(d, bid, tk);
  const uint64_t gen = ring_gen(d, tk);
  if (status == 0) {
    post_request_wave(&H(d)->ring[s], file, span, off0, len, tk, gen);
    if (l == 0) {
      trace_ev(d, 1, GFS_EV_REQ, bid, file, (uint32_t)lo, GFS_NO_FRAME, span, tk);
      bcount(bs, GFS_C_MISSES, 1);
      bcount(bs, GFS_C_REQUESTS, 1);
      bcount(bs, GFS_C_REQ_BYTES, len);
      bcount(bs, GFS_C_FETCHED, got);
      bcount(bs, GFS_C_RA_PAGES, got - 1);
    }
    /* tell waiting blocks which request fills each frame: (slot + 1) << 40 | gen */
    const uint64_t fill = ((uint64_t)(s + 1) << 40) | (gen & ((1ull << 40) - 1));
    for (uint32_t k = l; k < got; k += 64) st_rlx(&H(d)->ffill[bs->lframe[k]], fill);
  }
  if (l == 0) {
    if (status == 0) {
      gfs_rpc_slot* rs = &H(d)->ring[s];
      uint32_t nn = 0;
      const uint64_t th0 = wall_clock64();
      while (ld_host(&rs->done_seq) != gen) {
        if (expired(d, t0)) {
          status = -kETIMEDOUT;
          break;
        }
        nap(nn);
      }
      bcount(bs, GFS_T_HOST, wall_clock64() - th0);
      if (status == 0) {
        /* the staged bytes and the result were written by the host before done_seq */
        const uint64_t result = ld_host(&rs->result);
        bs->result = (int64_t)result;
        /* let blocks waiting on frames of this request pull their own pages */
        gfs_req_dev* rq = &H(d)->reqd[s];
        st_rlx((uint64_t*)&rq->result, result);
        st_rlx(&rq->first_page, lo);
        st_rlx32(&rq->file, file);
        st_rlx32(&rq->remaining, got);
        drain_atomics();
        st_rlx(&rq->ready, gen);
      }
    }
    if (status) bcount(bs, GFS_C_TIMEOUTS, 1);
    bs->status = status;
    bs->frame = (int32_t)bs->lframe[0];
    bs->pull = status == 0 ? 1 : 0;
    bs->slot = s;
    bs->gen = gen;
    bs->first_page = lo;
    bs->list_n = got;
    bs->file = file;
  }
  return 0;
}

/* Wave-collective, without the miss lock: reserve the table entry of key if no entry for it
 * exists, so that one block alone fetches the page. Lanes 0-31 load the key's two buckets; lane
 * 0 takes a free entry of the less loaded bucket by compare-and-swap; once that swap has been
 * performed the lanes look again, and if another block's entry for the same key is there the
 * reservation is withdrawn. Of two blocks that reserve one key at once, the later swap sees the
 * earlier one, so at most one reservation stays (both may withdraw; both then look again).
 * Returns the entry's index, -1 when the key has (or just got) another entry, -2 when both
 * buckets stayed full. */
__device__ int64_t reserve_unique_wave(const gfs_dev* d, uint64_t key) {
  uint32_t b1, b2;
  key_buckets(d, key, b1, b2);
  const uint32_t l = lane();
  const uint64_t ent = (key << GFS_ENTRY_FRAME_BITS) | kReserved;
  for (int attempt = 0; attempt < 64; ++attempt) {
    uint64_t e = 0;
    if (l < 32) e = ld_rlx(slot_ptr(d, b1, b2, (int)l));
    if (__ballot(l < 32 && (e >> GFS_ENTRY_FRAME_BITS) == key)) return -1;
    const uint64_t free1 = __ballot(l < 16 && e == 0), free2 = __ballot(l >= 16 && l < 32 && e == 0);
    const uint32_t used1 = 16u - (uint32_t)__popcll(free1), used2 = 16u - (uint32_t)__popcll(free2);
    uint64_t fm = used2 < used1 ? free2 : free1;   /* less loaded bucket, ties to the first */
    if (fm == 0) fm = free1 ? free1 : free2;
    if (fm == 0) return -2;
    const int pick = __builtin_ctzll(fm);
    uint64_t* sp = slot_ptr(d, b1, b2, pick);
    int won = 0;
    if (l == 0) {
      uint64_t z = 0;
      won = cas64_rlx(sp, z, ent) ? 1 : 0;
    }
    won = __shfl(won, 0, 64);
    if (!won) continue;   /* the entry was taken meanwhile: look again */
    drain_atomics();      /* the swap is performed before the second look goes out */
    uint64_t e2 = 0;
    if (l < 32 && (int)l != pick) e2 = ld_rlx(slot_ptr(d, b1, b2, (int)l));
    if (__ballot(l < 32 && (int)l != pick && (e2 >> GFS_ENTRY_FRAME_BITS) == key)) {
      if (l == 0) {
        uint64_t x = ent;
        (void)cas64_rlx(sp, x, 0ull);
      }
      return -1;
    }
    return (int64_t)(sp - H(d)->pt);
  }
  return -2;
}

/* Wave 0: the miss path of a file whose windows are one page (readahead off, or RANDOM advice):
 * no detector decision to make, so no miss lock; the page's reservation is made unique by
 * reserve_unique_wave. Same results and trace events as the locked path for such a file.
 * Returns as miss_shared_wave. */
__device__ __attribute__((noinline)) int miss_one_page_wave(const gfs_dev* d, uint32_t file, uint64_t p, uint64_t key, uint64_t fsize,
                                  BlockState* bs, uint32_t bid, uint64_t t0) {
  d = uniform(d);
  const uint32_t l = lane();
  const uint64_t tr0 = wall_clock64();
  const int64_t slot = reserve_unique_wave(d, key);
  if (slot == -1) return 1;   /* another block's entry: go to the pin path */
  if (slot < 0) {
    /* both buckets full of other misses' reservations: back off; -ENOSPC at the wait limit */
    if (!expired(d, t0)) {
      if (l == 0) {
        bcount(bs, GFS_C_RETRIES, 1);
        nap(bs->naps);
      }
      return 1;
    }
    if (l == 0) {
      bs->status = -kENOSPC;
      bs->pull = 0;
      bs->frame = -1;
    }
    return 0;
  }
  if (l == 0) {
    trace_ev(d, 1, GFS_EV_MISS, bid, file, (uint32_t)p, (uint32_t)RA_RULE_OFF << 24, 1, p);
    bs->list[0] = (uint32_t)p;
    bs->lslot[0] = (uint32_t)slot;
    bs->lframe[0] = GFS_NO_FRAME;
  }
  wave_sync_lds();
  const uint64_t tl3 = wall_clock64();
  if (l == 0) bcount(bs, GFS_T_RUN, tl3 - tr0);
  const uint32_t got = alloc_wave(d, file, p, bs, 1, bid);
  if (l == 0) bcount(bs, GFS_T_ALLOC, wall_clock64() - tl3);
  if (got == 0) {
    /* every frame pinned or filling: give the page back and retry the access */
    if (l == 0) {
      st_rlx(H(d)->pt + slot, 0ull);
      bcount(bs, GFS_C_NOFRAME, 1);
    }
    if (expired(d, t0)) return 2;
    if (l == 0) nap(bs->naps);
    return 1;
  }
  return post_wait_wave(d, file, fsize, bs, bid, t0, 1);
}

/* Wave 0: the shared policy's miss path for page p of `file` (key), found absent from the
 * table: take the file's miss lock, decide and claim the window, reserve and allocate its
 * run, post the request and wait for the host. Out of line: it runs once per host request
 * and holds most of the library's registers, which the hit path then does not have to share.
 * Returns 0 when bs is filled in (status, frame, pull), 1 to look the page up again, 2 when
 * the wait timed out. */
__device__ __attribute__((noinline)) int miss_shared_wave(const gfs_dev* d, uint32_t file, uint64_t p,
                                                          uint64_t key, uint64_t fsize, BlockState* bs,
                                                          uint32_t bid, uint64_t t0) {
  d = uniform(d);
  if (H(d)->ra_cap == 0 || ld_rlx32(&H(d)->files[file].advice) == GFS_ADV_RANDOM)
    return miss_one_page_wave(d, file, p, key, fsize, bs, bid, t0);
  const uint32_t l = lane();
  /* the pages of the read that missed, from p on */
  const uint64_t rl = bs->read_last;
  const uint32_t req = rl >= p ? (rl - p + 1 < 0xffffffffull ? (uint32_t)(rl - p + 1) : 0xffffffffu) : 1u;
  /* the cached history behind p, counted before the lock (see ra_history_wave) */
  const uint32_t hist_pre = ra_history_wave(d, file, p, req);
  const RaParams rp = ra_params(d);
  /* what the critical section needs from the device and file records, read now: after the
     grant, each would be a load on the path every waiter waits on */
  gfs_file_dev* const fe = &H(d)->files[file];
  uint64_t* const clp = H(d)->claims[file].e;
  uint64_t* const lq = lock_queue(d, file);
  const uint64_t npages = fe->npages;
  uint64_t* const pt = H(d)->pt;
  const uint32_t ptmask = H(d)->nbuckets_mask;
  const bool tracing = H(d)->trace_level >= 1;
  const bool async_on = H(d)->ra_async != 0;
  const uint64_t tl0 = wall_clock64();
  const uint64_t lr = lock_file_wave(d, file, key, p, lock_note(req, hist_pre, rp.cap, bid), t0);
  const int lk = (int)(lr & 7);
  const uint64_t tl1 = wall_clock64();
  if (lk != LOCK_OWN && l == 0) {
    bcount(bs, GFS_T_LOCK, tl1 - tl0);
    bcount(bs, lk == LOCK_DECIDED ? GFS_C_LOCKS : GFS_C_LOCK_LEFT, lk == LOCK_TIMEOUT ? 0 : 1);
  }
  if (lk == LOCK_TIMEOUT) return 2;
  if (lk == LOCK_LEFT) return 1;   /* the page was reserved while this block waited: go to the pin path */
  if (lk == LOCK_COVERED) {
    /* a holder's window covers the page: wait until its reservation shows in the
       table or no running claim covers the page any more, then look again */
    uint32_t nw = 0;
    while (pt_lookup_wave(d, key) < 0 && !expired(d, t0)) {
      uint64_t cl = 0;
      if (l < GFS_CLAIMS) cl = ld_rlx(&H(d)->claims[file].e[l]);
      const uint64_t c_lo = cl >> 32, c_hi = (cl >> 32) + ((cl & 0xffffffffull) >> 1);
      if (__ballot(l < GFS_CLAIMS && (cl & 1ull) && c_lo <= p && p < c_hi) == 0) break;
      if (l == 0) nap_short(nw);
    }
    return 1;
  }
  uint64_t cws, cwe, mark = ~0ull;
  uint64_t* claim;
  uint64_t tl2 = tl1;
  if (lk == LOCK_DECIDED) {
    const uint32_t w = (uint32_t)(lr >> 3);
    cws = p - (w & 0x3ffu);
    cwe = p + ((w >> 10) & 0x7ffu);
    claim = &clp[(w >> 21) & 31u];
    if ((w >> 26) & 1u) mark = p + 1;
  } else {
    const uint64_t ticket = lr >> 3;
    /* every block waiting on this file's lock waits for this wave: let it issue first, and
       keep the statistics until the lock is passed on */
    __builtin_amdgcn_s_setprio(3);
    /* one round: the detector state, the file's window claims, and the queue slots
       behind this ticket (a waiter that arrives or leaves after this read is handled by the
       compare-and-swaps and the grant's exchange) */
    RaState ras = ra_load_lane(fe, rp.nrec, rp.nstreams);
    uint64_t cl = ld_rlx(&clp[l & (GFS_CLAIMS - 1)]);
    const uint64_t nl = ticket + 1 + l;
    uint64_t qv = ld_rlx(lock_slot(lq, nl));
    drain_atomics();   /* the table probes below go out after the claims were read */
    ra_loaded(ras, cl, qv);
    bool cl_on = l < GFS_CLAIMS && (cl & 1ull);
    uint64_t cl_lo = cl >> 32, cl_hi = (cl >> 32) + ((cl & 0xffffffffull) >> 1);
    uint64_t free_cl = __ballot(l < GFS_CLAIMS && !cl_on);
    /* the waiters right behind that can be decided for: announced, with a page, and as many as
       there are free claims left beside this block's own */
    const bool gone = qv == lock_left(nl) || (uint32_t)qv == (uint32_t)lock_covered(nl);
    const bool waits = (qv >> 63) && (uint32_t)qv == ((uint32_t)nl << 2) && (uint32_t)(qv >> 32) != (0x80000000u | kNoPage);
    const uint64_t stop = __ballot(!gone && !waits);
    uint32_t end = stop ? (uint32_t)__builtin_ctzll(stop) : 64u;   /* slots looked at: [0, end) */
    const uint32_t nfree = (uint32_t)__popcll(free_cl);
    const uint32_t room = nfree ? (nfree - 1 < GFS_LOCK_BATCH - 1 ? nfree - 1 : GFS_LOCK_BATCH - 1) : 0u;
    uint64_t cand = __ballot(waits) & (end == 64 ? ~0ull : (1ull << end) - 1);
    {
      uint64_t m = cand;
      for (uint32_t k = 0; k < room && m; ++k) m &= m - 1;
      if (m) {   /* more than there is room for: the first of the rest gets the lock */
        end = (uint32_t)__builtin_ctzll(m);
        cand &= (1ull << end) - 1;
      }
    }
    /* take them, read their notes, and probe the table for all the pages, in one round: items 0 (this
       block) and 1.. (the candidates in order), two a half wave each. A waiter writes its note before
       it announces, so a note read after the announcement was seen is that one, or one that another
       file's waiter has written over it since */
    const uint64_t qn = ld_rlx(lock_note_at(d, file, nl));
    uint64_t held = 0;
    bool took = false;
    if ((cand >> l) & 1) {
      uint64_t v = qv;
      took = cas64_rlx(lock_slot(lq, nl), v, lock_taken(nl));
    }
    uint32_t nitems = 1 + (uint32_t)__popcll(cand);
    {
      uint64_t e[GFS_LOCK_BATCH / 2], k[GFS_LOCK_BATCH / 2];
      uint64_t m = cand;
#pragma unroll
      for (uint32_t u = 0; u < GFS_LOCK_BATCH / 2; ++u) {
        e[u] = 0;
        k[u] = ~0ull;
        if (2 * u >= nitems) continue;
        uint64_t pa = p, pb = p;
        if (u) {
          pa = (uint32_t)__builtin_amdgcn_readlane((int)(qv >> 32), __builtin_ctzll(m)) & 0x7fffffffu;
          m &= m - 1;
        }
        const bool second = 2 * u + 1 < nitems;
        if (second) {
          pb = (uint32_t)__builtin_amdgcn_readlane((int)(qv >> 32), __builtin_ctzll(m)) & 0x7fffffffu;
          m &= m - 1;
        }
        k[u] = page_key(file, l < 32 ? pa : pb);
        uint32_t b1, b2;
        key_buckets_m(ptmask, k[u], b1, b2);
        e[u] = ld_rlx(pt + (uint64_t)((l & GFS_BUCKET_SLOTS) ? b2 : b1) * GFS_BUCKET_SLOTS + (l & 15));
      }
#pragma unroll
      for (uint32_t u = 0; u < GFS_LOCK_BATCH / 2; ++u) {
        const uint64_t m2 = __ballot((e[u] >> GFS_ENTRY_FRAME_BITS) == k[u]);
        held |= ((uint32_t)m2 ? 1ull : 0ull) << (2 * u) | ((m2 >> 32) ? 2ull : 0ull) << (2 * u);
      }
    }
    const uint64_t lost = __ballot(took && !lock_note_is(qn, file, nl));
    if (lost) {
      /* the first whose note is gone gets the lock instead: it and the taken ones behind it wait
         again, before the lock is passed on */
      end = (uint32_t)__builtin_ctzll(lost);
      if (took && l >= end) st_rlx(lock_slot(lq, nl), qv);
      drain_atomics();
      took = took && l < end;
      cand &= (1ull << end) - 1;
      nitems = 1 + (uint32_t)__popcll(cand);
    }
    const uint64_t taken = __ballot(took);
    /* decide in ticket order */
    const uint64_t td0 = wall_clock64();
    uint32_t dirty = 0, ndec = 0;
    uint64_t claimed = 0, outv = 0;
    uint32_t own = 0;   /* 0: look again at once, 1: a running claim holds the page, 2: decided */
    uint64_t own_a = 0, own_b = 0;
    uint32_t own_cj = 0;
    uint64_t m = cand;
    for (uint32_t it = 0; it < nitems; ++it) {
      uint32_t at = 0;
      uint64_t ip = p;
      uint32_t ireq = req, ihist = hist_pre, ibid = bid;
      RaParams irp = rp;
      if (it) {
        at = (uint32_t)__builtin_ctzll(m);
        m &= m - 1;
        if (((taken >> at) & 1) == 0) continue;   /* it left */
        ip = (uint32_t)__builtin_amdgcn_readlane((int)(qv >> 32), (int)at) & 0x7fffffffu;
        const LockNote nt = lock_note_read(lane64(qn, (int)at));
        ireq = nt.req;
        ihist = nt.hist;
        ibid = nt.bid;
        irp.cap = nt.cap;   /* of the waiter's launch, which may not be this block's */
      }
      const bool covered = __ballot(cl_on && cl_lo <= ip && ip < cl_hi) != 0;
      const bool present = ((held >> it) & 1) != 0;
      uint64_t o = lock_covered(ticket + 1 + at);
      if (!present && !covered && free_cl) {
        /* a miss: decide the window, clip it to the file and out of running claims, claim it */
        uint64_t ws;
        uint32_t wn, near, hist, rule;
        int rslot;
        ra_decide_wave(ip, ireq, ihist, irp, ras, dirty, ws, wn, near, hist, rule, rslot);
        if (ws + wn > npages) wn = (uint32_t)(npages - ws);
        /* asynchronous readahead: the page after the demanded one is the stream's marker */
        const bool marked = async_on && rslot >= 0 && ip + 1 < ws + wn;
        if (async_on && (int)l == rslot) ras.s_marker = marked ? (uint32_t)(ip + 1) : GFS_NO_MARKER;
        if (tracing && l == 0)
          trace_ev(d, 1, GFS_EV_MISS, ibid, file, (uint32_t)ip, (near & 0xffu) | (hist << 8) | (rule << 24), wn,
                   ws | ((uint64_t)ireq << 32));
        uint64_t a = ws, b = ws + wn;
        for (uint64_t c = __ballot(cl_on && cl_lo < b && cl_hi > a); c; c &= c - 1) {
          const int i = __builtin_ctzll(c);
          const uint64_t clo = lane64(cl_lo, i), chi = lane64(cl_hi, i);
          if (chi <= ip) a = a > chi ? a : chi;
          else b = b < clo ? b : clo;   /* no running claim holds ip, so this one lies above it */
        }
        const uint32_t cj = (uint32_t)__builtin_ctzll(free_cl);
        free_cl &= free_cl - 1;
        claimed |= 1ull << cj;
        if (l == cj) {
          cl_on = true;
          cl_lo = a;
          cl_hi = b;
        }
        ++ndec;
        if (it == 0) {
          own = 2;
          own_a = a;
          own_b = b;
          own_cj = cj;
          if (marked) mark = p + 1;
        } else {
          o = lock_decided(ticket + 1 + at, (uint32_t)(ip - a), (uint32_t)(b - ip), cj, marked);
        }
      } else if (it == 0) {
        own = present ? 0u : 1u;
      }
      if (it && l == at) outv = o;
    }
    const uint64_t td1 = wall_clock64();
    /* write back; the outcomes go out, and the lock is passed on, once that has been performed */
    if (ndec) ra_store_lane(fe, ras, dirty, async_on);
    if ((claimed >> l) & 1) st_rlx(&clp[l], (cl_lo << 32) | ((cl_hi - cl_lo) << 1) | 1ull);
    const uint64_t tu0 = wall_clock64();
    drain_atomics();
    if (took) st_rlx(lock_slot(lq, nl), outv);
    /* slots beyond the 64 read count as not announced */
    const uint64_t shifted = __shfl(qv, (int)((l + end) & 63u), 64);
    const uint64_t pre = l + end < 64 ? shifted : 0ull;
    unlock_slots_wave(lq, ticket + 1 + end, claimed, cl_lo, cl_hi, true, pre);
    __builtin_amdgcn_s_setprio(0);
    tl2 = wall_clock64();
    if (l == 0) {
      bcount(bs, GFS_T_LOCK, tl1 - tl0);
      bcount(bs, GFS_C_LOCKS, 1);
      bcount(bs, GFS_T_DECIDE, td1 - td0);
      bcount(bs, GFS_T_CRIT, tl2 - tl1);
      bcount(bs, GFS_T_UNLOCK, tl2 - tu0);
    }
    if (own != 2) {
      /* filled, reserved, or about to be reserved by a window being claimed: go to the pin
         path (after a nap if the claim is still running) */
      if (own == 1) {
        if (expired(d, t0)) return 2;
        if (l == 0) nap(bs->naps);
      }
      return 1;
    }
    cws = own_a;
    cwe = own_b;
    claim = &clp[own_cj];
  }
  /* reserve the run of unmapped pages around p inside the claimed window */
  const uint32_t cwn = (uint32_t)(cwe - cws);
  uint32_t n = 0, failed = 0;
  if (cwn <= 64) {
    /* one round: lane i loads the buckets of window page cws + i, the run around p is
       read off the ballot of present pages, and each run lane reserves its page from
       the buckets it already holds */
    n = reserve_run_small_wave(d, file, p, cws, cwn, bs, failed);
  } else {
    /* pages evicted after use end the run too, unless p is one */
    const bool clip = !shadow_lane(d, file, p);
    uint64_t a = p;
    for (uint64_t base = p; base > cws;) {
      const bool valid = (uint64_t)l < base - cws;
      bool stop = !valid;
      if (valid)
        stop = (int)pt_present_lane(d, page_key(file, base - 1 - l)) | (int)(clip && shadow_lane(d, file, base - 1 - l));
      const uint64_t sm = __ballot(stop);
      const uint32_t k = sm ? (uint32_t)__builtin_ctzll(sm) : 64u;
      a = base - k;
      if (k < 64) break;
      base -= 64;
    }
    uint64_t b = p;
    for (uint64_t base = p + 1; base < cwe;) {
      const bool valid = (uint64_t)l < cwe - base;
      bool stop = !valid;
      if (valid) stop = (int)pt_present_lane(d, page_key(file, base + l)) | (int)(clip && shadow_lane(d, file, base + l));
      const uint64_t sm = __ballot(stop);
      const uint32_t k = sm ? (uint32_t)__builtin_ctzll(sm) : 64u;
      b = base + k - 1;
      if (k < 64) break;
      base += 64;
    }
    n = (uint32_t)(b - a + 1);
    /* allocation order: the demanded page first, then the rest of the run ascending */
    for (uint32_t i = l; i < n; i += 64) {
      uint64_t q;
      if (i == 0) q = p;
      else if (i <= p - a) q = a + i - 1;
      else q = a + i;
      const int64_t slot = pt_reserve_lane(d, page_key(file, q));
      bs->list[i] = (uint32_t)q;
      bs->lslot[i] = slot < 0 ? 0xffffffffu : (uint32_t)slot;
      bs->lframe[i] = GFS_NO_FRAME;
      failed |= slot < 0 ? 1u : 0u;
    }
  }
  failed = (uint32_t)(__ballot(failed != 0) != 0);
  /* the reservations are in the table: release the claim */
  drain_atomics();
  if (l == 0) st_rlx(claim, 0ull);
  wave_sync_lds();
  const uint64_t tl3 = wall_clock64();
  if (l == 0) bcount(bs, GFS_T_RUN, tl3 - tl2);
  /* a reservation can fail only if both buckets are full: keep the prefix before the
     first failure (the demanded page comes first) and drop the rest */
  uint32_t keep = n;
  if (failed) {
    uint32_t firstbad = n;
    for (uint32_t i = l; i < n; i += 64)
      if (bs->lslot[i] == 0xffffffffu) firstbad = i < firstbad ? i : firstbad;
    for (int off = 32; off > 0; off >>= 1) {
      const uint32_t o = __shfl_xor(firstbad, off, 64);
      firstbad = o < firstbad ? o : firstbad;
    }
    keep = firstbad;
  }
  const uint32_t got = keep ? alloc_wave(d, file, p, bs, keep, bid, mark) : 0;
  if (l == 0) bcount(bs, GFS_T_ALLOC, wall_clock64() - tl3);
  /* release reservations that got no frame (the table was full or no frame was free) */
  for (uint32_t i = got + l; i < n; i += 64) {
    if (bs->lslot[i] != 0xffffffffu)
      st_rlx(H(d)->pt + bs->lslot[i], 0ull);
  }
  if (got == 0) {
    if (l == 0) bcount(bs, keep ? GFS_C_NOFRAME : GFS_C_RETRIES, 1);
    if (keep == 0 && expired(d, t0)) {
      /* the demanded page's buckets stayed full until the wait limit */
      if (l == 0) {
        bs->status = -kENOSPC;
        bs->pull = 0;
        bs->frame = -1;
      }
      return 0;
    }
    if (expired(d, t0)) return 2;
    if (l == 0) nap(bs->naps);
    return 1;   /* buckets full of reservations in flight, or every frame pinned or
                   filling: back off and retry the access */
  }
  if (got < n && l == 0)
    trace_ev(d, 1, GFS_EV_NOFRAME, bid, file, bs->list[got], GFS_NO_FRAME, 0, 0);
  return post_wait_wave(d, file, fsize, bs, bid, t0, got);
}

/* ------------------------------------------------------------------ one page, wave 0
 * Leaves in bs: status; on success the pinned frame, and pull = 1 when this block posted
 * the request and must pull it. absent: the caller's group pass has just found no table
 * entry for the page, so the first look is taken as made (the miss path looks again). */
__device__ __forceinline__ void acquire_page_wave(const gfs_dev* d, uint32_t file, uint64_t p, uint64_t fsize,
                                  BlockState* bs, uint32_t bid, bool absent) {
  d = uniform(d);
  const uint64_t key = page_key(file, p);
  const uint32_t l = lane();
  const uint64_t t0 = wall_clock64();   /* the wait deadline's start */
  if (l == 0) {
    bs->trig = 0;
    bs->naps = 0;
  }
  while (true) {
    const int32_t f = absent ? -1 : pt_lookup_wave(d, key);
    absent = false;
    if (f >= 0 && (uint32_t)f != kReserved) {
      int r = PIN_RETRY;
      uint64_t w = 0;
      if (l == 0) r = frame_pin(d, (uint32_t)f, key, &w);
      r = __shfl(r, 0, 64);
      if (r == PIN_VALID) {
        if (l == 0) {
          bcount(bs, GFS_C_HITS, 1);
          trace_ev(d, 2, GFS_EV_HIT, bid, file, (uint32_t)p, (uint32_t)f, 0, 0);
          bs->frame = f;
          bs->status = 0;
          bs->pull = 0;
          if (H(d)->ra_async && (w & GFS_FW_MARK)) bs->trig = mark_take_lane(d, (uint32_t)f) ? 1u : 0u;
        }
        return;
      }
      if (r == PIN_FILLING) {
        if (l == 0) {
          bcount(bs, GFS_C_JOINS, 1);
          trace_ev(d, 2, GFS_EV_JOIN, bid, file, (uint32_t)p, (uint32_t)f, 0, 0);
          if (H(d)->ra_async && (w & GFS_FW_MARK)) bs->trig = mark_take_lane(d, (uint32_t)f) ? 1u : 0u;
          const uint64_t tj0 = wall_clock64();
          join_or_help_lane(d, (uint32_t)f, p, t0, bs);
          bcount(bs, GFS_T_JOIN, wall_clock64() - tj0);
        }
        return;
      }
      if (r == PIN_ERROR) {
        if (l == 0) {
          bs->status = -kEIO;
          bs->frame = -1;
          bs->pull = 0;
        }
        return;
      }
      if (l == 0) bcount(bs, GFS_C_RETRIES, 1);
    }
    if (f >= 0 && (uint32_t)f != kReserved) {
      /* the pin lost a race (the frame changed under it): wait a little and look again */
    } else if (f < 0 && H(d)->policy == GFS_POLICY_PRIVATE) {
      const int r = miss_private_wave(d, file, p, key, fsize, bs, bid, t0);
      if (r == 0) return;
      if (r == 2) break;
      continue;
    } else if (f < 0 && bs->a_pending) {
      /* a block posts a request only with no asynchronous request of its own outstanding (so
         that no block waits for a ring slot that only it would free): the block finishes that
         request first and then looks again */
      if (l == 0) {
        bs->status = 0;
        bs->pull = 5;
        bs->frame = -1;
      }
      return;
    } else if (f < 0) {
      const int r = miss_shared_wave(d, file, p, key, fsize, bs, bid, t0);
      if (r == 0) return;
      if (r == 2) break;
      continue;
    }
    /* reserved by another block's miss, or a lost race: wait a little and look again */
    if (expired(d, t0)) break;
    if (l == 0) nap(bs->naps);
  }
  if (l == 0) {
    bcount(bs, GFS_C_TIMEOUTS, 1);
    bs->status = -kETIMEDOUT;
    bs->pull = 0;
    bs->frame = -1;
  }
}

/* Bytes of page q held in the staging of a request whose span starts at first (clamped to
 * what the host returned and to the file). */
__device__ __forceinline__ uint64_t staged_bytes(const gfs_dev* d, uint64_t q, uint64_t first,
                                                 int64_t result, uint64_t fsize) {
  const uint64_t P = H(d)->page_size;
  const uint64_t rel = (q - first) * P;
  int64_t avail = result - (int64_t)rel;
  if (avail < 0) avail = 0;
  uint64_t pb = fsize - (q << H(d)->page_shift);
  if (pb > P) pb = P;
  return (uint64_t)avail < pb ? (uint64_t)avail : pb;
}
__device__ __forceinline__ bool staged_short(const gfs_dev* d, uint64_t q, uint64_t first,
                                             int64_t result, uint64_t fsize) {
  const uint64_t P = H(d)->page_size;
  uint64_t pb = fsize - (q << H(d)->page_shift);
  if (pb > P) pb = P;
  return result < 0 || (uint64_t)result < (q - first) * P + pb;
}

/* Wave 0: claim the request's frames that no helping block has taken (PULL bit); their
 * indices go to bs->lslot[0..nclaim). A frame counts as the request's only while its fill word
 * names the request (fill): once helpers have published it, the clock may have given it to
 * another request, which the caller must not touch. The word is read first and, once it is
 * there, the fill word after it, and the claim is a compare-and-swap against that word, so a frame that
 * changed hands in between is not claimed. */
__device__ __attribute__((noinline)) void claim_pulls_wave(const gfs_dev* d, BlockState* bs, uint64_t fill) {
  d = uniform(d);
  const uint32_t l = lane();
  uint32_t nclaim = 0;
  for (uint32_t base = 0; base < bs->list_n; base += 64) {
    const uint32_t k = base + l;
    bool won = false;
    if (k < bs->list_n) {
      const uint32_t f = bs->lframe[k];
      uint64_t* fw = &H(d)->fword[f];
      uint64_t w = ld_rlx(fw);
      while ((w & GFS_FW_STATE) == GFS_FS_FILLING && !(w & GFS_FW_PULL) && ld_rlx(&H(d)->ffill[f]) == fill) {
        if (cas64_rlx(fw, w, (w | GFS_FW_PULL) + GFS_FW_VER_ONE)) {
          won = true;
          break;
        }
      }
    }
    const uint64_t m = __ballot(won);
    if (won) bs->lslot[nclaim + __popcll(m & lanemask_lt())] = k;
    nclaim += (uint32_t)__popcll(m);
  }
  if (l == 0) bs->nclaim = nclaim;
  wave_sync_lds();
}

/* Block-collective: copy claimed pages from the ring slot's staging into their frames, as far as
 * the host returned bytes (rounded up to 16). pull == 1: the frames listed in lslot[0..nclaim);
 * pull == 2: the one helped frame. All units of all pages are one sequence, so that a thread has
 * eight loads over the host link in flight whatever the page size: a 4 KiB page is one load a
 * thread. */
__device__ __attribute__((noinline)) void block_pull(const gfs_dev* d, const BlockState* bs) {
  d = uniform(d);
  const uint32_t tid = thread_id(), nt = block_threads();
  const uint32_t sh = H(d)->page_shift, ush = sh - 4;
  const uint8_t* const stg = H(d)->staging + (uint64_t)bs->slot * H(d)->max_req_bytes;
  uint8_t* const frames = H(d)->frames;
  const bool help = bs->pull == 2;
  const uint64_t first = bs->first_page;
  const uint64_t have = bs->result > 0 ? (uint64_t)bs->result : 0;
  const uint32_t total = (help ? 1u : bs->nclaim) << ush;   /* at most 1024 pages of 2^17 units */
  for (uint32_t u0 = tid; u0 < total; u0 += 8 * nt) {
    uint8_t* to[8];
    const uint8_t* from[8];
    uint32_t ok = 0;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const uint32_t u = u0 + j * nt;
      from[j] = stg;
      to[j] = frames;
      if (u >= total) continue;
      const uint32_t k = help ? 0u : bs->lslot[u >> ush];
      const uint64_t q = help ? bs->help_page : bs->list[k];
      const uint32_t f = help ? (uint32_t)bs->frame : bs->lframe[k];
      const uint32_t at = (u & ((1u << ush) - 1)) << 4;
      const uint64_t so = ((q - first) << sh) + at;
      if (so < have) {
        ok |= 1u << j;
        from[j] = stg + so;
        to[j] = frames + ((uint64_t)f << sh) + at;
      }
    }
    copy_in8(to, from, ok);
  }
}

/* Lane: publish a pulled frame VALID (reference bit set, ERR if the host read came short). */
__device__ __forceinline__ void publish_frame(const gfs_dev* d, uint32_t f, bool short_read) {
  uint64_t* fw = &H(d)->fword[f];
  uint64_t w = ld_rlx(fw);
  while (true) {
    uint64_t nw = ((w & ~(GFS_FW_STATE | GFS_FW_PULL)) | GFS_FS_VALID | GFS_FW_REF) + GFS_FW_VER_ONE;
    if (short_read) nw |= GFS_FW_ERR;
    if (cas64_rlx(fw, w, nw)) break;
  }
}

/* Lane 0 (after the frames are published): count them off the request; the block that
 * publishes the last one frees the ring slot. */
__device__ __forceinline__ void request_done_lane(const gfs_dev* d, uint32_t s, uint64_t gen,
                                                  uint32_t cnt) {
  if (cnt == 0) return;
  const uint32_t before = __hip_atomic_fetch_sub(G(&H(d)->reqd[s].remaining), cnt, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
  if (before == cnt) {
    st_rlx(&H(d)->slot_free[s], gen);
    if (s >= H(d)->sync_slots) {   /* an asynchronous window's slot: its generation first */
      drain_atomics();
      st_rlx(&H(d)->reqd[s].busy, 0ull);
    }
  }
}

/* Wave 0, after the block's pull, a wait by every wave and a barrier: publish the frames
 * this block pulled and count them off. Returns the status of this block's page: for its
 * own request the demanded page (list[0]), which a helper may be pulling, so it may wait.
 * On an error the block's pin on its page has been dropped. */
__device__ __attribute__((noinline)) int64_t publish_pull_wave(const gfs_dev* d, BlockState* bs, uint64_t fsize,
                                     uint64_t t0) {
  d = uniform(d);
  const uint32_t l = lane();
  uint32_t bad = 0;
  int64_t st = 0;
  if (bs->pull == 2) {
    if (l == 0) {
      const bool sh = staged_short(d, bs->help_page, bs->first_page, bs->result, fsize);
      publish_frame(d, (uint32_t)bs->frame, sh);
      request_done_lane(d, bs->slot, bs->gen, 1);
      bad = sh ? 1u : 0u;
      st = sh ? -kEIO : 0;
      if (sh) frame_unpin(d, (uint32_t)bs->frame);
    }
  } else {
    for (uint32_t c = l; c < bs->nclaim; c += 64) {
      const uint32_t k = bs->lslot[c];
      const bool sh = staged_short(d, bs->list[k], bs->first_page, bs->result, fsize);
      publish_frame(d, bs->lframe[k], sh);
      bad += sh ? 1u : 0u;
    }
    drain_atomics();   /* every lane's frames are published */
    if (l == 0) {
      request_done_lane(d, bs->slot, bs->gen, bs->nclaim);
      /* the demanded page: pulled here, or by a helper that may still be copying it (an
         asynchronous request has none: frame -1) */
      if (bs->frame >= 0) {
        st = wait_valid_lane(d, (uint32_t)bs->frame, t0);
        if (st == -kETIMEDOUT) bcount(bs, GFS_C_TIMEOUTS, 1);
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off, 64);
  if (l == 0) bcount(bs, GFS_C_IOERR, bad);
  return __shfl(st, 0, 64);
}

/* Block-collective: the private policy's fills. pull 3: the page from the block's private
 * buffer into its frame; pull 4: the staged request's first page into the frame and the
 * rest of the span into the private buffer. */
__device__ void private_pull(const gfs_dev* d, const BlockState* bs, uint64_t fsize) {
  const uint32_t tid = thread_id(), nt = block_threads();
  const uint64_t P = H(d)->page_size;
  const uint32_t f = (uint32_t)bs->frame;
  const gfs_pslot* ps = &H(d)->pslots[bs->pslot];
  uint8_t* pb = H(d)->pbuf + (uint64_t)bs->pslot * H(d)->ra_cap * P;
  if (bs->pull == 3) {
    const uint64_t q = bs->help_page;
    uint64_t n = fsize - (q << H(d)->page_shift);
    if (n > P) n = P;
    copy_in(H(d)->frames + (uint64_t)f * P, pb + (q - ps->first) * P, n, tid, nt);
    return;
  }
  const uint8_t* stg = H(d)->staging + (uint64_t)bs->slot * H(d)->max_req_bytes;
  copy_in(H(d)->frames + (uint64_t)f * P, stg,
                     staged_bytes(d, bs->first_page, bs->first_page, bs->result, fsize), tid, nt);
  const int64_t rest = bs->result - (int64_t)P;
  if (rest > 0) copy_in(pb, stg + P, (uint64_t)rest, tid, nt);
}

/* Thread 0, after private_pull and a block barrier: publish the frame; for a host request,
 * free its ring slot and make the rest of the span the private buffer (only whole pages
 * unless the read stopped at the end of the file). 0 or -EIO (the pin is then dropped). */
__device__ int64_t private_publish_lane(const gfs_dev* d, BlockState* bs, uint64_t fsize) {
  gfs_pslot* ps = &H(d)->pslots[bs->pslot];
  const uint32_t f = (uint32_t)bs->frame;
  if (bs->pull == 3) {
    publish_frame(d, f, false);
    ps->used += 1;
    return 0;
  }
  const uint64_t P = H(d)->page_size;
  const bool short_page = staged_short(d, bs->first_page, bs->first_page, bs->result, fsize);
  publish_frame(d, f, short_page);
  if (short_page) bcount(bs, GFS_C_IOERR, 1);
  st_rlx(&H(d)->slot_free[bs->slot], bs->gen);   /* the block's barrier came after its last read of the staging */
  const uint64_t off0 = bs->first_page << H(d)->page_shift;
  uint64_t expect = (uint64_t)bs->list_n * P;
  if (expect > fsize - off0) expect = fsize - off0;
  const int64_t rest = bs->result - (int64_t)P;
  uint32_t n = 0;
  if (rest > 0) n = (uint32_t)((bs->result == (int64_t)expect) ? ((uint64_t)rest + P - 1) / P : (uint64_t)rest / P);
  bcount(bs, GFS_C_PB_WASTED, ps->n - ps->used);
  bcount(bs, GFS_C_RA_PAGES, n);
  ps->file = bs->file;
  ps->first = bs->first_page + 1;
  ps->n = n;
  ps->used = 0;
  if (short_page) {
    frame_unpin(d, f);
    return -kEIO;
  }
  return 0;
}

/* ------------------------------------------------------------------ asynchronous readahead
 * Sec. 2.3: Linux reads the next window while the reader still consumes the current one. A
 * stream's marker page (the page after the demanded one in a demand window, the first page
 * of an asynchronous window) carries GFS_FW_MARK from its allocation; the first block whose
 * access finds it clears it and, after copying its own page, advances the stream: window
 * [next, next + min(2 size, cap)), the run of unmapped pages from its start, posted to the
 * host with nobody waiting. Blocks that need one of its pages join the frame and pull it from
 * staging once the host is done (the ring slot says so); the block that posted the request
 * pulls the rest when it next needs to post, reaches the next marker, or closes the file. */

/* Wave-collective, outside the lock: reserve the run of unmapped pages that starts at ws,
   within [ws, ws + n), ascending into bs->list/lslot/lframe; returns its length and sets
   failed if a page found both buckets full. */
__device__ uint32_t reserve_from_wave(const gfs_dev* d, uint32_t file, uint64_t ws, uint32_t n, bool clip,
                                      BlockState* bs, uint32_t& failed) {
  const uint32_t l = lane();
  uint32_t count = 0, bad = 0;
  for (uint32_t base = 0; base < n; base += 64) {
    const bool valid = base + l < n;
    const uint64_t q = ws + base + l;
    const uint64_t key = page_key(file, q);
    uint32_t b1 = 0, b2 = 0;
    uint64_t e[2 * GFS_BUCKET_SLOTS];
    bool present = false, gone = false;
    if (valid) {
      key_buckets(d, key, b1, b2);
      pt_load_lane(d, b1, b2, e);
      gone = clip && shadow_lane(d, file, q);
#pragma unroll
      for (int i = 0; i < 2 * GFS_BUCKET_SLOTS; ++i) present |= (e[i] >> GFS_ENTRY_FRAME_BITS) == key;
    }
    const uint64_t stop = __ballot(!valid || present || gone);
    const uint32_t k = stop ? (uint32_t)__builtin_ctzll(stop) : 64u;
    if (l < k) {
      int cnt1 = 0, cnt2 = 0, f1 = -1, f2 = -1;
#pragma unroll
      for (int i = 0; i < GFS_BUCKET_SLOTS; ++i) {
        if (e[i]) ++cnt1;
        else if (f1 < 0) f1 = i;
        if (e[GFS_BUCKET_SLOTS + i]) ++cnt2;
        else if (f2 < 0) f2 = GFS_BUCKET_SLOTS + i;
      }
      int pick = cnt2 < cnt1 ? f2 : f1;
      if (pick < 0) pick = f1 >= 0 ? f1 : f2;
      int64_t slot = -1;
      if (pick >= 0) {
        uint64_t expect = 0;
        uint64_t* sp = slot_ptr(d, b1, b2, pick);
        if (cas64_rlx(sp, expect, (key << GFS_ENTRY_FRAME_BITS) | kReserved)) slot = (int64_t)(sp - H(d)->pt);
        else slot = pt_reserve_lane(d, key);
      }
      bs->list[base + l] = (uint32_t)q;
      bs->lslot[base + l] = slot < 0 ? 0xffffffffu : (uint32_t)slot;
      bs->lframe[base + l] = GFS_NO_FRAME;
      bad |= slot < 0 ? 1u : 0u;
    }
    count = base + k;
    if (k < 64) break;
  }
  failed = (uint32_t)(__ballot(bad != 0) != 0);
  return count;
}

/* Wave 0, with no asynchronous request of the block outstanding: the block's access found
   marker page m of file `file`. Advance the stream whose marker m still is (lowest slot),
   reserve and allocate the window's unmapped run, and post it to the host without waiting;
   the request becomes the block's outstanding one. Gives up quietly when no stream names m,
   the window is empty, a running claim holds its first page, or no frame is free. */
__device__ __attribute__((noinline)) void async_issue_wave(const gfs_dev* d, uint32_t file, uint64_t m, uint64_t fsize, BlockState* bs,
                                 uint32_t bid, uint64_t t0) {
  d = uniform(d);
  const uint32_t l = lane();
  /* a slot of its own first: with none free the window is not issued (readers then miss at
     its first page and the stream goes on synchronously) */
  int32_t aslot = -1;
  if (l == 0) aslot = async_slot_take_lane(d, bid);
  aslot = __shfl(aslot, 0, 64);
  if (aslot < 0) return;
  const uint32_t s = (uint32_t)aslot;
  /* the waiter announces no page, so no holder marks it covered or decides for it */
  const uint64_t lk = lock_file_wave(d, file, 0, kNoPage, kNoNote, t0, false);
  const uint64_t ticket = lk >> 3;
  if ((lk & 7) != LOCK_OWN) {
    if (l == 0) st_rlx(&H(d)->reqd[s].busy, 0ull);
    return;
  }
  __builtin_amdgcn_s_setprio(3);
  const RaState ras = ra_load_lane(&H(d)->files[file], H(d)->ra_recent, H(d)->streams);
  uint64_t cl = 0;
  if (l < GFS_CLAIMS) cl = ld_rlx(&H(d)->claims[file].e[l]);
  const uint64_t npages = H(d)->files[file].npages;
  /* the window leaves out pages evicted after use, unless the marker page is one */
  const bool clip = !shadow_lane(d, file, m);
  drain_atomics();
  const uint64_t sm = __ballot(l < H(d)->streams && ras.s_valid && ras.s_marker == (uint32_t)m);
  if (sm == 0) {
    unlock_file_wave(d, file, ticket, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    if (l == 0) st_rlx(&H(d)->reqd[s].busy, 0ull);
    return;
  }
  const int j = __ffsll((unsigned long long)sm) - 1;
  const uint32_t clk = __shfl(ras.clk, 0, 64) + 1;
  const uint64_t ws = __shfl(ras.s_next, j, 64);
  const uint32_t sz = __shfl(ras.s_size, j, 64);
  const uint32_t cap = ra_cap_eff(d);
  const uint32_t wn = 2 * sz < cap ? 2 * sz : cap;
  gfs_file_dev* fe = &H(d)->files[file];
  if (l == 0) {
    gfs_stream* st = &fe->streams[j];
    st_rlx(&st->next, ws + wn);
    st_rlx32(&st->size, wn);
    st_rlx32(&st->last_use, clk);
    st_rlx32(&st->marker, (uint32_t)ws);
    st_rlx32(&fe->clock, clk);
  }
  const uint32_t wnc = ws < npages ? (uint32_t)((npages - ws) < wn ? (npages - ws) : wn) : 0u;
  if (l == 0) {
    trace_ev(d, 1, GFS_EV_ADV, bid, file, (uint32_t)m, 0, wnc, ws);
    bcount(bs, GFS_C_ADVANCES, 1);
  }
  /* a running claim on the first page: that block is fetching it; else stop at the next claim */
  const bool cl_on = l < GFS_CLAIMS && (cl & 1ull);
  const uint64_t cl_lo = cl >> 32, cl_hi = (cl >> 32) + ((cl & 0xffffffffull) >> 1);
  const bool held = __ballot(cl_on && cl_lo <= ws && ws < cl_hi) != 0;
  const uint64_t free_cl = __ballot(l < GFS_CLAIMS && !cl_on);
  uint64_t hi_b = cl_on && cl_lo > ws ? cl_lo : ~0ull;
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t b = __shfl_xor(hi_b, off, 64);
    hi_b = b < hi_b ? b : hi_b;
  }
  const uint64_t cwe = ws + wnc < hi_b ? ws + wnc : hi_b;
  if (wnc == 0 || held || free_cl == 0 || cwe <= ws) {
    unlock_file_wave(d, file, ticket, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    if (l == 0) st_rlx(&H(d)->reqd[s].busy, 0ull);
    return;
  }
  const uint32_t cj = (uint32_t)__builtin_ctzll(free_cl);
  uint64_t* claim = &H(d)->claims[file].e[cj];
  if (l == 0) st_rlx(claim, (ws << 32) | ((cwe - ws) << 1) | 1ull);
  unlock_file_wave(d, file, ticket, ws, cwe);
  __builtin_amdgcn_s_setprio(0);
  uint32_t failed = 0;
  const uint32_t n = reserve_from_wave(d, file, ws, (uint32_t)(cwe - ws), clip, bs, failed);
  drain_atomics();
  if (l == 0) st_rlx(claim, 0ull);
  wave_sync_lds();
  uint32_t keep = n;
  if (failed) {
    uint32_t firstbad = n;
    for (uint32_t i = l; i < n; i += 64)
      if (bs->lslot[i] == 0xffffffffu) firstbad = i < firstbad ? i : firstbad;
    for (int off = 32; off > 0; off >>= 1) {
      const uint32_t o = __shfl_xor(firstbad, off, 64);
      firstbad = o < firstbad ? o : firstbad;
    }
    keep = firstbad;
  }
  /* no demanded page: every page is prefetched; the window's first page is the new marker */
  const uint32_t got = keep ? alloc_wave(d, file, ~0ull, bs, keep, bid, ws) : 0;
  for (uint32_t i = got + l; i < n; i += 64)
    if (bs->lslot[i] != 0xffffffffu) st_rlx(H(d)->pt + bs->lslot[i], 0ull);
  if (got == 0) {
    if (l == 0) st_rlx(&H(d)->reqd[s].busy, 0ull);
    return;
  }
  if (got < n && l == 0) trace_ev(d, 1, GFS_EV_NOFRAME, bid, file, bs->list[got], GFS_NO_FRAME, 0, 0);
  /* the pages that got frames are [ws, ws + got) */
  const uint64_t off0 = ws << H(d)->page_shift;
  uint64_t len = (uint64_t)got << H(d)->page_shift;
  if (off0 + len > fsize) len = fsize - off0;
  /* the slot is this window's alone: its staging is free once its last request was counted
     off (that cleared busy), and its next generation is one past the last completed */
  const uint64_t gen = ld_rlx(&H(d)->slot_free[s]) + 1;
  const uint64_t tk = (gen - 1) * H(d)->rpc_slots + s;   /* for the trace only */
  if (l == 0)   /* frames count themselves off the request as they are published */
    __hip_atomic_store(G(&H(d)->reqd[s].remaining), got, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t fill = (1ull << 63) | ((uint64_t)(s + 1) << 40) | (gen & ((1ull << 40) - 1));
  for (uint32_t k = l; k < got; k += 64) st_rlx(&H(d)->ffill[bs->lframe[k]], fill);
  post_request_wave(&H(d)->ring[s], file, got, off0, len, tk, gen);   /* after the count and the fill words */
  if (l == 0) {
    trace_ev(d, 1, GFS_EV_REQ, bid, file, (uint32_t)ws, GFS_NO_FRAME, got, tk);
    bcount(bs, GFS_C_REQUESTS, 1);
    bcount(bs, GFS_C_REQ_BYTES, len);
    bcount(bs, GFS_C_FETCHED, got);
    bcount(bs, GFS_C_RA_PAGES, got);
    bs->a_pending = 1;
    bs->a_slot = s;
    bs->a_gen = gen;
    bs->a_first = ws;
    bs->a_n = got;
    bs->a_file = file;
  }
}

/* Block-collective: finish the block's outstanding asynchronous request, if any: wait for the
   host, pull every frame no other block has claimed, publish them. 0 or -ETIMEDOUT. */
__device__ __attribute__((noinline)) int64_t async_finish_block(const gfs_dev* d, BlockState* bs) {
  d = uniform(d);
  const uint32_t tid = thread_id();
  __syncthreads();
  if (!bs->a_pending) return 0;
  const uint64_t t0 = wall_clock64();
  if (tid == 0) {
    gfs_rpc_slot* rs = &H(d)->ring[bs->a_slot];
    uint32_t nn = 0;
    int st = 0;
    const uint64_t th0 = wall_clock64();
    /* the slot's generations only grow: one past a_gen means the host finished this request,
       blocks that joined its frames pulled and published every one of them, and the slot went
       to a later request (nothing is left to claim: no frame's fill word names this one) */
    uint64_t ds;
    while ((int64_t)((ds = ld_host(&rs->done_seq)) - bs->a_gen) < 0) {
      if (expired(d, t0)) {
        st = -kETIMEDOUT;
        break;
      }
      nap(nn);
    }
    bcount(bs, GFS_T_HOST, wall_clock64() - th0);
    if (st) bcount(bs, GFS_C_TIMEOUTS, 1);
    if (st == 0 && ds != bs->a_gen) st = 1;   /* done, and nothing left to pull */
    bs->a_status = st;
    bs->result = (int64_t)ld_host(&rs->result);
    bs->slot = bs->a_slot;
    bs->gen = bs->a_gen;
    bs->first_page = bs->a_first;
    bs->list_n = bs->a_n;
    bs->frame = -1;
    bs->pull = 1;
  }
  __syncthreads();
  int64_t st = bs->a_status;
  if (st == 0) {
    const uint64_t fsize = H(d)->files[bs->a_file].size;
    if (tid < 64)
      claim_pulls_wave(d, bs, (1ull << 63) | ((uint64_t)(bs->a_slot + 1) << 40) | (bs->a_gen & ((1ull << 40) - 1)));
    __syncthreads();
    block_pull(d, bs);
    drain_atomics();   /* every wave's frame bytes are in memory before the frames are published */
    __syncthreads();
    if (tid < 64) (void)publish_pull_wave(d, bs, fsize, t0);
  }
  __syncthreads();
  if (tid == 0) {
    bs->a_pending = 0;
    bs->pull = 0;
  }
  __syncthreads();
  return st < 0 ? st : 0;
}

/* ------------------------------------------------------------------ the group pass
 * A read's pages are taken 64 at a time. Those the cache holds are looked up and pinned
 * together, copied by the whole block and unpinned together: two dependent round trips
 * (table, pin) a group instead of two a page. The others go through gread_page, in order.
 * Not used while the policy trace is recorded: a traced run makes its accesses one at a time
 * in page order.
 *
 * Every wave of the block looks up its share. Half a wave takes a page: its 32 lanes load the
 * page's two buckets, two 128-byte lines, where one lane a page would load 32 scattered
 * entries (32 pages of 4 KiB: 2048 separate fetches). Lane j of wave w then owns page
 * group_page(j, w, W): it pins the frame, keeps the frame's tag in flight beside the copy and
 * compares it before the unpin. */
__device__ __forceinline__ uint32_t group_page(uint32_t j, uint32_t w, uint32_t W) {
  return (((j >> 1) * W + w) << 1) + (j & 1u);
}

/* One wave: look up its pages of the group (base + i for the set bits i of todo below n), lane
 * j returning page group_page(j)'s frame, kAbsent or kNotReady. Four pairs of pages are loaded
 * before the first is waited for. */
__device__ __forceinline__ int32_t group_lookup(const gfs_dev* d, uint32_t file, uint64_t base, uint32_t n,
                                                uint64_t todo, uint32_t w, uint32_t W) {
  const uint32_t l = lane();
  uint64_t* const pt = H(d)->pt;
  const uint32_t mask = H(d)->nbuckets_mask;
  const uint32_t un = __builtin_amdgcn_readfirstlane(n);   /* whole pairs are skipped by a branch */
  int32_t f = kAbsent;
  for (uint32_t r0 = 0; group_page(2 * r0, w, W) < un; r0 += 4) {
    uint64_t e[4], key[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      e[u] = 0;
      key[u] = ~0ull;
      if (group_page(2 * (r0 + u), w, W) >= un) continue;
      const uint32_t i = group_page(2 * (r0 + u) + (l >> 5), w, W);
      key[u] = page_key(file, base + i);
      if (i < n && ((todo >> i) & 1)) {
        uint32_t b1, b2;
        key_buckets_m(mask, key[u], b1, b2);
        e[u] = ld_rlx(pt + (uint64_t)((l & GFS_BUCKET_SLOTS) ? b2 : b1) * GFS_BUCKET_SLOTS + (l & 15));
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      if (group_page(2 * (r0 + u), w, W) >= un) continue;
      const uint64_t m = __ballot((e[u] >> GFS_ENTRY_FRAME_BITS) == key[u]);   /* keys are never 0 */
      const uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
      const int fe = (int)((uint32_t)e[u] & (uint32_t)kFrameMask);
      if (lo) {
        const int g = __builtin_amdgcn_readlane(fe, (int)__builtin_ctz(lo));
        if (l == 2 * (r0 + u)) f = g;
      }
      if (hi) {
        const int g = __builtin_amdgcn_readlane(fe, 32 + (int)__builtin_ctz(hi));
        if (l == 2 * (r0 + u) + 1) f = g;
      }
    }
  }
  return f == (int32_t)kReserved ? kNotReady : f;
}

/* The block copies the pinned pages of a group smaller than a round of the whole block each:
 * all their 16-byte units in one sequence, eight loads a thread in flight. Units are aligned
 * in dst; page bytes before its first and after its last unit go one byte a thread. */
__device__ __forceinline__ void copy_group(const gfs_dev* d, const int32_t* frame, uint64_t base, uint32_t n,
                                           uint64_t offset, uint64_t end, uint8_t* dst, uint32_t tid, uint32_t nt) {
  const uint32_t sh = H(d)->page_shift, ush = sh - 4, P = 1u << sh;
  const uint8_t* const frames = H(d)->frames;
  /* dst address of the first page's start (maybe before dst), and the first dst-aligned
     position in every page */
  uint8_t* const d0 = dst + (int64_t)((base << sh) - offset);
  const uint32_t h = (0u - (uint32_t)(uintptr_t)d0) & 15u;
  const uint64_t pb = base << sh;
  /* bytes wanted, relative to the group's first page */
  const uint32_t lo = offset > pb ? (uint32_t)(offset - pb) : 0u;
  const uint32_t hi = end - pb < ((uint64_t)n << sh) ? (uint32_t)(end - pb) : n << sh;
  const uint32_t total = n << ush;
  for (uint32_t u0 = tid; u0 < total; u0 += 8 * nt) {
    v4u a[8];
    const uint8_t* p[8];
    uint32_t ok = 0;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const uint32_t u = u0 + j * nt;
      const uint32_t i = u >> ush, at = ((u & ((1u << ush) - 1)) << 4) + h, pos = (i << sh) + at;
      const int32_t f = u < total ? frame[i] : kAbsent;
      const bool take = f >= 0 && at + 16 <= P && pos >= lo && pos + 16 <= hi;
      if (take) ok |= 1u << j;
      p[j] = frames + (take ? ((uint64_t)(uint32_t)f << sh) + at : 0);   /* not taken: any readable bytes */
    }
    ld_frame(a, p);
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const uint32_t u = u0 + j * nt;
      if ((ok >> j) & 1) *(gv4u*)(d0 + (((u >> ush) << sh) + ((u & ((1u << ush) - 1)) << 4) + h)) = a[j];
    }
  }
  if ((h | lo | hi) & 15u) {
    /* 32 threads a page: 16 for the bytes before its first unit, 16 for those after its last */
    for (uint32_t i = tid >> 5; i < n; i += nt >> 5) {
      const int32_t f = frame[i];
      if (f < 0) continue;
      const uint32_t p0 = i << sh;
      const uint32_t plo = lo > p0 ? lo - p0 : 0u, phi = hi - p0 < P ? hi - p0 : P;
      uint32_t a = plo <= h ? h : h + ((plo - h + 15u) & ~15u);
      if (a > phi) a = phi;
      const uint32_t b = a + ((phi - a) & ~15u);
      const uint32_t k = tid & 15u;
      const uint32_t at = (tid & 16u) ? b + k : plo + k;
      if (at < ((tid & 16u) ? phi : a))
        ((gu8*)d0)[p0 + at] = ld_frame_byte(frames + ((uint64_t)(uint32_t)f << sh) + at);
    }
  }
}

/* Block-collective: deliver the cached, valid pages among base + i, i a set bit of todo (below
 * n <= 64). Returns the pages delivered; first_absent is set if the first page left over has
 * no table entry. Every thread's copies are complete and the pins dropped on return. */
__device__ __forceinline__ uint64_t group_pass(const gfs_dev* d, BlockState* bs, uint32_t file, uint64_t base,
                                               uint32_t n, uint64_t todo, uint64_t offset, uint64_t end,
                                               uint8_t* dst, bool& first_absent) {
  const uint32_t tid = thread_id(), nt = block_threads(), l = lane();
  const uint32_t w = __builtin_amdgcn_readfirstlane(tid >> 6), W = nt >> 6;
  const bool timed = H(d)->page_timers != 0;
  const uint64_t t0 = timed ? wall_clock64() : 0;
  const uint32_t par = bs->par;
  const uint32_t mine = group_page(l, w, W);
  int32_t f = group_lookup(d, file, base, n, todo, w, W);
  uint64_t pw = 0, tag = 0;
  if (f >= 0) {
    pw = __hip_atomic_fetch_add(G(&H(d)->fword[f]), GFS_FW_PIN_ONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    /* a frame being filled is joined, a failed one reported and a marker page's mark taken by
       gread_page */
    if ((pw & GFS_FW_STATE) != GFS_FS_VALID || (pw & GFS_FW_ERR) || (H(d)->ra_async && (pw & GFS_FW_MARK))) {
      frame_unpin(d, (uint32_t)f);
      f = kNotReady;
    } else {
      /* read after the pin, so it names the page the bytes belong to: a pinned frame cannot
         be claimed. Waited for after the copy */
      tag = ld_rlx(&H(d)->ftag[f]);
    }
  }
  if (mine < n) bs->bframe[par][mine] = f;
  __syncthreads();
  const int32_t fl = l < n ? bs->bframe[par][l] : kAbsent;
  uint64_t hits = __ballot(fl >= 0);
  if (tid == 0) {
    bs->par = par ^ 1u;   /* every thread has read par, and has left the other half */
    bs->bbad[par ^ 1u] = 0;
  }
  const uint64_t t1 = timed ? wall_clock64() : 0;
  const uint32_t sh = H(d)->page_shift;
  if (hits) {
    if (n > 1 && (1u << sh) < 128u * nt) {
      copy_group(d, bs->bframe[par], base, n, offset, end, dst, tid, nt);
    } else {
      for (uint64_t m = hits; m; m &= m - 1) {
        const uint32_t i = (uint32_t)__builtin_ctzll(m);
        const uint64_t pb = (base + i) << sh;
        const uint64_t lo = offset > pb ? offset : pb;
        const uint64_t hi = end < pb + (1ull << sh) ? end : pb + (1ull << sh);
        copy_out(dst + (lo - offset), H(d)->frames + ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(fl, (int)i) << sh) + (lo - pb),
                 (uint32_t)(hi - lo), tid, nt);
      }
    }
    /* bytes copied from a frame that holds another page (it was reused between the lookup and
       the pin) are overwritten by the next look: gread has not returned, nobody reads dst yet */
    if (f >= 0 && tag != page_key(file, base + mine))
      __hip_atomic_fetch_or(&bs->bbad[par], 1ull << mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  const uint64_t bad = bs->bbad[par];
  const uint64_t t2 = timed ? wall_clock64() : 0;
  if (f >= 0) {
    if (!((bad >> mine) & 1)) frame_pin_bits(d, (uint32_t)f, pw);
    frame_unpin(d, (uint32_t)f);
  }
  hits &= ~bad;
  if (tid == 0) {
    bcount(bs, GFS_C_HITS, (uint64_t)__popcll(hits));
    if (bad) bcount(bs, GFS_C_RETRIES, (uint64_t)__popcll(bad));
    if (timed) {
      bcount(bs, GFS_T_ACQUIRE, t1 - t0);
      bcount(bs, GFS_T_COPY, t2 - t1);
      bcount(bs, GFS_T_UNPIN, wall_clock64() - t2);
    }
  }
  const uint64_t left = todo & ~hits;
  first_absent = left && __builtin_amdgcn_readlane(fl, (int)__builtin_ctzll(left)) == kAbsent;
  return hits;
}

/* Block-collective: deliver page p of the read [offset, end) through the one-page path: a hit,
 * a join, or a miss that fetches it. Out of line, so that the registers of the miss path are
 * not the caller's. absent: the page was just looked up and has no table entry. 0 or -errno. */
__device__ __attribute__((noinline)) int64_t gread_page(const gfs_dev* d, BlockState* bs, uint32_t file, uint64_t p,
                                                        uint64_t fsize, uint64_t offset, uint64_t end, uint8_t* dst,
                                                        bool absent) {
  d = uniform(d);
  const uint32_t tid = thread_id(), nt = block_threads();
  const uint32_t bid = block_id();
  const uint64_t P = H(d)->page_size;
  const bool ptm = H(d)->page_timers != 0;
  while (true) {
    const uint64_t ta0 = ptm ? wall_clock64() : 0;
    if (tid < 64) acquire_page_wave(d, file, p, fsize, bs, bid, absent);
    absent = false;
    __syncthreads();
    if (bs->pull == 5) {
      /* a miss while this block's asynchronous request is outstanding: finish it, look again */
      const int64_t e = async_finish_block(d, bs);
      if (e < 0) return e;
      continue;
    }
    if (bs->pull >= 3) {
      const uint64_t tp0 = wall_clock64();
      private_pull(d, bs, fsize);
      drain_atomics();   /* every wave's frame bytes are in memory before the frames are published */
      __syncthreads();
      if (tid == 0) {
        const int64_t st = private_publish_lane(d, bs, fsize);
        if (st < 0) bs->status = st;
        bs->pull = 0;
        bcount(bs, GFS_T_PULL, wall_clock64() - tp0);
      }
      __syncthreads();
    } else if (bs->pull) {
      const uint64_t tp0 = wall_clock64();
      if (bs->pull == 1) {
        if (tid < 64)
          claim_pulls_wave(d, bs, ((uint64_t)(bs->slot + 1) << 40) | (bs->gen & ((1ull << 40) - 1)));
        __syncthreads();
      }
      block_pull(d, bs);
      drain_atomics();   /* every wave's frame bytes are in memory before the frames are published */
      __syncthreads();
      if (tid < 64) {
        const int64_t st = publish_pull_wave(d, bs, fsize, wall_clock64());
        if (tid == 0) {
          if (st < 0) bs->status = st;
          bs->pull = 0;
          bcount(bs, GFS_T_PULL, wall_clock64() - tp0);
        }
      }
      __syncthreads();
    }
    const int64_t st = bs->status;
    const int32_t f = bs->frame;
    const bool trig = bs->trig != 0;
    if (st < 0) {
      __syncthreads();
      return st;
    }
    const uint64_t ta1 = ptm ? wall_clock64() : 0;
    const uint64_t pbase = p << H(d)->page_shift;
    const uint64_t lo = offset > pbase ? offset : pbase;
    const uint64_t hi = end < pbase + P ? end : pbase + P;
    copy_out(dst + (lo - offset), H(d)->frames + (uint64_t)f * P + (lo - pbase), (uint32_t)(hi - lo), tid, nt);
    __syncthreads();
    if (tid == 0) {
      const uint64_t ta2 = ptm ? wall_clock64() : 0;
      frame_unpin(d, (uint32_t)f);
      if (ptm) {
        bcount(bs, GFS_T_ACQUIRE, ta1 - ta0);
        bcount(bs, GFS_T_COPY, ta2 - ta1);
        bcount(bs, GFS_T_UNPIN, wall_clock64() - ta2);
      }
    }
    if (trig) {
      /* this access took its stream's marker: finish the block's previous asynchronous
         request, then issue the stream's next window without waiting for it */
      const int64_t e = async_finish_block(d, bs);
      if (e < 0) return e;
      if (tid < 64) async_issue_wave(d, file, p, fsize, bs, bid, wall_clock64());
      __syncthreads();
    }
    return 0;
  }
}

}  // namespace gfsd

/* ====================================================================== public API */

__device__ int gopen_id(const gfs_dev* d, int file_id, int flags) {
  gfsd::BlockState* bs = gfsd::block_state();
  __syncthreads();   /* every thread is past the block's earlier calls */
  for (uint32_t c = gfsd::thread_id(); c < GFS_C_COUNT; c += gfsd::block_threads()) bs->ctr[c] = 0;
  if (gfsd::thread_id() == 0) {
    /* one round trip for both fields */
    const bool id_ok = file_id >= 0 && (uint32_t)file_id < gfsd::H(d)->max_files;
    gfs_file_dev* fe = &gfsd::H(d)->files[id_ok ? file_id : 0];
    const uint32_t is_open = gfsd::ld_rlx32(&fe->open);
    const uint64_t size = gfsd::ld_rlx(&fe->size);
    int v;
    if (flags != GFS_O_RDONLY) {
      v = -gfsd::kEROFS;
    } else if (!id_ok || is_open == 0) {
      v = -gfsd::kENOENT;
    } else {
      __hip_atomic_fetch_add(gfsd::G(&gfsd::H(d)->files[file_id].handles), 1u, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      v = file_id;
    }
    bs->pslot = -1;
    if (v >= 0 && gfsd::H(d)->policy == GFS_POLICY_PRIVATE) {
      /* the block's private slot: its own frames and private buffer until gclose. A slot
         given back by a block that just ended may not show yet: look again, with naps,
         until the wait timeout */
      const uint64_t t0 = wall_clock64();
      uint32_t naps = 0;
      while (bs->pslot < 0) {
        for (uint32_t i = 0; i < gfsd::H(d)->npslots && bs->pslot < 0; ++i) {
          const uint32_t s = (gfsd::block_id() + i) % gfsd::H(d)->npslots;
          uint32_t z = 0;
          if (gfsd::ld_rlx32(&gfsd::H(d)->pslots[s].owner) == 0 && gfsd::cas32(&gfsd::H(d)->pslots[s].owner, z, 1u))
            bs->pslot = (int32_t)s;
        }
        if (bs->pslot >= 0 || gfsd::expired(d, t0)) break;
        gfsd::nap(naps);
      }
      if (bs->pslot < 0) {
        __hip_atomic_fetch_sub(gfsd::G(&gfsd::H(d)->files[file_id].handles), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v = -gfsd::kENOSPC;
      } else {
        gfs_pslot* ps = &gfsd::H(d)->pslots[bs->pslot];
        ps->n = 0;   /* a new owner starts with an empty private buffer */
        ps->used = 0;
      }
    }
    bs->pull = 0;
    bs->trig = 0;
    bs->par = 0;
    bs->bbad[0] = 0;
    bs->a_pending = 0;   /* an asynchronous request is finished by gclose, before the next gopen */
    bs->open_result = v;
    bs->open_fd = v;
    bs->open_size = v >= 0 ? size : 0;
  }
  __syncthreads();
  const int v = bs->open_result;
  __syncthreads();
  return v;
}

__device__ int gopen(const gfs_dev* d, const char* path, int flags) {
  gfsd::BlockState* bs = gfsd::block_state();
  if (gfsd::thread_id() == 0) {
    int id = -1;
    for (uint32_t i = 0; i < gfsd::H(d)->max_files && id < 0; ++i) {
      if (gfsd::ld_rlx32(&gfsd::H(d)->files[i].open) == 0) continue;
      const char* nm = gfsd::H(d)->names + (uint64_t)i * GFS_NAME_MAX;
      uint32_t j = 0;
      while (j < GFS_NAME_MAX && nm[j] == path[j] && nm[j] != 0) ++j;
      if (j < GFS_NAME_MAX && nm[j] == 0 && path[j] == 0) id = (int)i;
    }
    bs->open_result = id;
  }
  __syncthreads();
  const int id = bs->open_result;
  __syncthreads();
  if (flags != GFS_O_RDONLY) return -gfsd::kEROFS;
  if (id < 0) return -gfsd::kENOENT;
  return gopen_id(d, id, flags);
}

__device__ int gclose(const gfs_dev* d, int fd) {
  if (fd < 0 || (uint32_t)fd >= gfsd::H(d)->max_files) return -gfsd::kEBADF;
  gfsd::BlockState* bs = gfsd::block_state();
  /* an asynchronous request still outstanding is pulled in before the block lets go */
  __syncthreads();
  if (bs->a_pending) (void)gfsd::async_finish_block(d, bs);
  if (gfsd::H(d)->policy == GFS_POLICY_PRIVATE) {
    if (gfsd::thread_id() == 0 && bs->pslot >= 0) {
      gfs_pslot* ps = &gfsd::H(d)->pslots[bs->pslot];
      gfsd::bcount(bs, GFS_C_PB_WASTED, ps->n - ps->used);   /* the private buffer is dropped */
      ps->n = 0;
      ps->used = 0;
      __hip_atomic_store(gfsd::G(&ps->owner), 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      bs->pslot = -1;
    }
    __syncthreads();
  }
  /* a counter a thread */
  for (uint32_t c = gfsd::thread_id(); c < GFS_C_COUNT; c += gfsd::block_threads()) {
    const uint64_t v = bs->ctr[c];
    if (v) gfsd::fadd64(&gfsd::H(d)->g->ctr[c], v);
    bs->ctr[c] = 0;
  }
  if (gfsd::thread_id() == 0) {
    __hip_atomic_fetch_sub(gfsd::G(&gfsd::H(d)->files[fd].handles), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bs->open_fd = -1;
  }
  __syncthreads();
  return 0;
}

namespace gfsd {
/* gread of `size` bytes by a block that is reading `ahead` (at least size) from offset on, in pieces:
   the detector sees the whole read. */
__device__ __attribute__((always_inline)) int64_t gread_piece(const gfs_dev* d, int fd, uint64_t offset, uint64_t size,
                                                              uint64_t ahead, void* dst) {
  BlockState* bs = block_state();
  if (fd < 0 || (uint32_t)fd >= H(d)->max_files) return -kEBADF;
  uint64_t fsize;
  if (fd == bs->open_fd) {
    fsize = bs->open_size;   /* checked by gopen */
  } else {
    gfs_file_dev* fe = &H(d)->files[fd];
    if (ld_rlx32(&fe->open) == 0) return -kEBADF;
    fsize = fe->size;
  }
  if (block_threads() & 63u) return -kEINVAL;
  if (size == 0 || offset >= fsize) return 0;
  const uint64_t end = (size > fsize - offset) ? fsize : offset + size;
  const uint32_t tid = thread_id();
  const uint32_t sh = H(d)->page_shift;
  const uint64_t plast = (end - 1) >> sh;
  const bool grouped = H(d)->trace_level == 0;
  /* read by wave 0's miss path, after this store */
  if (tid == 0) bs->read_last = ((ahead > fsize - offset ? fsize : offset + ahead) - 1) >> sh;
  for (uint64_t base = offset >> sh; base <= plast; base += 64) {
    const uint32_t n = plast - base < 64 ? (uint32_t)(plast - base) + 1 : 64u;
    uint64_t todo = n == 64 ? ~0ull : (1ull << n) - 1;
    while (true) {
      bool absent = false;
      if (grouped) todo &= ~group_pass(d, bs, (uint32_t)fd, base, n, todo, offset, end, (uint8_t*)dst, absent);
      if (todo == 0) break;
      /* the first page not delivered; the window its miss fetches may hold the next ones, so
         the group is looked at again */
      const int64_t e = gread_page(d, bs, (uint32_t)fd, base + (uint64_t)__builtin_ctzll(todo), fsize, offset, end,
                                   (uint8_t*)dst, absent);
      if (e < 0) return e;
      todo &= todo - 1;
      if (todo == 0) break;
    }
  }
  if (tid == 0) bcount(bs, GFS_C_DELIVERED, end - offset);
  return (int64_t)(end - offset);
}
/* The pieces (log2 of their bytes; kWhole: none) in which blocks that each consume a read of `bytes`
 * after it are better off reading and consuming it. With more than 256 of them (one a compute unit)
 * at work on more than the last-level cache holds (256 MiB), a consumer finds a piece there but not a
 * whole read. With fewer blocks a piece's look-up is time nothing else fills, and with fewer bytes
 * there is little to gain. 512 pieces of 256 KiB take half of that cache; more blocks, which are
 * small ones, take pieces of 64 KiB, whose look-ups hide behind the other blocks of the unit, and
 * from 192 MiB on.
 * Batch units over 1.5 GiB of cached 64 KiB pages, us whole, cut at 256 KiB and at 64 KiB; 256
 * threads: 512 blocks x 1 MiB 868, 750, -, 384 x 1 MiB 810, 797, -, 256 x 1 MiB 844, 845, -,
 * 128 x 1 MiB 1378, 1485, -, 64 x 4 MiB 2487, 2789, -, 512 x 512 KiB 700, 700, -; 128 threads:
 * 1024 x 1 MiB 1007, 892, 835, 768 x 1 MiB 955, 804, 764, 512 x 1 MiB 939, 839, 912, 1024 x 256 KiB
 * 744, -, 708, 1024 x 128 KiB 714, -, 694; 64 threads: 2048 x 1 MiB 1212, 982, 865, 1024 x 256 KiB
 * 847, -, 817, 768 x 256 KiB 929, -, 951, 512 x 1 MiB 1238, 1211, 1332. Serving, cached, 512 blocks,
 * chunks of 1 MiB: 20 requests of 16 MiB 316, 306, -, one 168, 182, -. */
constexpr uint32_t kWhole = 63;
__host__ __device__ __forceinline__ constexpr uint32_t cut_reads(uint64_t blocks, uint64_t bytes) {
  return blocks <= 256 || blocks * bytes <= ((blocks <= 512 ? 256ull : 192ull) << 20) ? kWhole : blocks <= 512 ? 18u : 16u;
}
/* Bytes of the next piece, at offset, of a read with `left` bytes to go, for a block that consumes
 * each piece before it reads the next (cut: cut_reads' answer). Cuts lie at multiples of the piece, or
 * of a larger page, so that no page is looked up twice and a piece's look-up is a few per cent of its
 * copy. A read that starts off a 16-byte boundary is read whole, as its pieces would not start on
 * one in the buffer. */
__device__ __forceinline__ uint64_t piece_bytes(const gfs_dev* d, uint64_t offset, uint64_t left, uint32_t cut) {
  const uint32_t sh = H(d)->page_shift;
  const uint64_t b = 1ull << (sh > cut ? sh : cut);
  const uint64_t n = b - (offset & (b - 1));
  return (offset & 15u) || n > left ? left : n;
}
}  // namespace gfsd

__device__ __attribute__((always_inline)) int64_t gread(const gfs_dev* d, int fd, uint64_t offset,
                                                        uint64_t size, void* dst) {
  return gfsd::gread_piece(d, fd, offset, size, size, dst);
}

#endif /* GFS_DEVICE_H */
