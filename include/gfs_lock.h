/* gfs_lock.h -- what the queue slots and notes of the per-file miss lock hold.
 *
 * Internal to the library: plain functions on integers, shared by the device code
 * (gfs_device.h says how the lock works) and by host code that models it.
 */
#ifndef GFS_LOCK_H
#define GFS_LOCK_H

#include <stdint.h>

#include "gfs.h"
#include "gfs_layout.h"

namespace gfsd {

/* ---- a ticket's slot: the low word carries the ticket, so stale values of earlier ones never match */
constexpr uint32_t kNoPage = 0x7fffffffu;   /* announced by a waiter that must hold the lock itself */
constexpr uint64_t lock_granted(uint64_t n) { return (uint64_t)(((uint32_t)n << 2) | 1u); }
constexpr uint64_t lock_left(uint64_t n) { return (uint64_t)(((uint32_t)n << 2) | 2u); }
constexpr uint64_t lock_covered(uint64_t n) { return (uint64_t)(((uint32_t)n << 2) | 3u); }
constexpr uint64_t lock_waiting(uint64_t n, uint64_t page) {
  return (1ull << 63) | (page << 32) | (uint64_t)((uint32_t)n << 2);
}
constexpr uint64_t lock_taken(uint64_t n) { return (1ull << 62) | (uint64_t)((uint32_t)n << 2); }
/* decided: the claimed window [page - below, page + above) in claim slot `claim`; marked: the page
   after the demanded one is its stream's marker */
constexpr uint64_t lock_decided(uint64_t n, uint32_t below, uint32_t above, uint32_t claim, bool marked) {
  return (1ull << 62) | ((uint64_t)(below | (above << 10) | (claim << 21) | (marked ? 1u << 26 : 0u)) << 32) |
         lock_covered(n);
}
static_assert(GFS_MAX_WINDOW_PAGES <= 1024 && GFS_CLAIMS <= 32, "a window's extent and claim slot fit lock_decided");

/* ---- a miss as its waiter notes it: pages of the read from the missed one on, cached history behind
 * it, the largest window its launch allows, the block (for the trace); kNoNote if they do not fit,
 * which no holder decides on. A read longer than any window is noted as 2047 pages: the decision
 * does not tell them apart. */
struct LockNote {
  uint32_t req, hist, cap, bid;
};
constexpr uint64_t kNoNote = ~0ull;
constexpr uint32_t kNoteReq = 2047;
constexpr uint64_t lock_note(uint32_t req, uint32_t hist, uint32_t cap, uint32_t bid) {
  return (hist >> 11) | ((cap - 1) >> 10) | (bid >> 22)
             ? kNoNote
             : (uint64_t)(req < kNoteReq ? req : kNoteReq) | ((uint64_t)hist << 11) | ((uint64_t)(cap - 1) << 22) |
                   ((uint64_t)bid << 32);
}
constexpr LockNote lock_note_read(uint64_t v) {
  return LockNote{(uint32_t)v & kNoteReq, (uint32_t)(v >> 11) & 2047u, ((uint32_t)(v >> 22) & 1023u) + 1,
                  (uint32_t)(v >> 32) & 0x3fffffu};
}
static_assert(GFS_MAX_WINDOW_PAGES <= 1024, "the cap, a history of up to one page more, and kNoteReq above both");

/* Whose note it is, in the top ten bits: of the files that share the row, of the tickets that share
 * the place; never 0, which is what cleared memory holds. A holder that finds another's note there
 * leaves the lock to that waiter instead of deciding for it. */
constexpr uint64_t lock_note_tag(uint32_t file, uint64_t n) {
  return 1ull | ((uint64_t)(file / GFS_LOCK_NOTE_ROWS) << 1) | ((n / GFS_LOCK_SLOTS & 31u) << 5);
}
static_assert(GFS_MAX_FILES / GFS_LOCK_NOTE_ROWS <= 16, "a note's file fits its tag");
constexpr uint64_t lock_note_tagged(uint64_t note, uint32_t file, uint64_t n) {
  return note | (lock_note_tag(file, n) << 54);
}
constexpr bool lock_note_is(uint64_t v, uint32_t file, uint64_t n) { return (v >> 54) == lock_note_tag(file, n); }
/* a ticket's place among its file's slots, and among the notes of all files */
constexpr uint64_t lock_slot_index(uint64_t n) { return n & (GFS_LOCK_SLOTS - 1); }
constexpr uint64_t lock_note_index(uint32_t file, uint64_t n) {
  return (uint64_t)(file % GFS_LOCK_NOTE_ROWS) * GFS_LOCK_SLOTS + lock_slot_index(n);
}

}  // namespace gfsd

#endif /* GFS_LOCK_H */
