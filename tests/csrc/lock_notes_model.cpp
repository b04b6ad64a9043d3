// CPU thread model of the notes in which waiters of the per-file miss lock leave what a holder
// needs to decide for them, on the device's own encodings (gfs_lock.h), run under ThreadSanitizer
// by the CPU tests. Several files keep their notes in one row, so that a waiter's note may be
// written over by another file's waiter, and files are closed and opened again, which starts their
// tickets and clears their slots but not their notes.
//
// Threads stand in for blocks (the same number for every file). Each takes tickets of one file, writes its note (read length, cached
// history, largest window, block: different each time), announces its page, and is granted the
// lock, or finds an outcome. A holder looks at the slots behind its ticket, then reads the notes of
// those that wait, takes them, and decides for each from its note up to the first whose note is
// another's; that one and the taken ones behind it wait again before the lock is passed on. With
// every outcome the holder leaves what it decided on, which the waiter compares with its own miss.
// Checked: that comparison, one holder of a file at a time, every thread ends before the deadline.
//
// Modes: notes (as on the device), and planted mistakes which the checks must catch: no-tag (a note
// is believed whosever it is), note-first (the notes are read before the slots, which plain loads
// of one round may do), pass-over (the lock goes past the waiters from a lost note on).
//
// usage: lock_notes_model MODE FILES THREADS MISSES SEED; prints a line ending in "-> ok"
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <deque>
#include <random>
#include <string>
#include <thread>
#include <vector>

#include "gfs_lock.h"

namespace {

using namespace gfsd;
using A64 = std::atomic<uint64_t>;
constexpr auto ACQ = std::memory_order_acquire, REL = std::memory_order_release, AR = std::memory_order_acq_rel,
               RLX = std::memory_order_relaxed;

struct File {
  uint32_t id = 0;
  A64 next{0};
  A64 slot[GFS_LOCK_SLOTS] = {};
  LockNote used[GFS_LOCK_SLOTS] = {};   // what a holder decided on, ordered by the slot
  std::atomic<int> holders{0};
};
std::deque<File> g_files;
A64 g_note[GFS_LOCK_SLOTS];   // the row that the files share
std::atomic<bool> g_failed{false};
A64 g_for_others{0}, g_lost{0}, g_own{0};
bool g_tags = true, g_slot_first = true, g_pass_over = false;
std::chrono::steady_clock::time_point g_deadline;

void fail(const char* what, uint64_t a = 0, uint64_t b = 0) {
  if (!g_failed.exchange(true)) fprintf(stderr, "FAILED: %s (%llu, %llu)\n", what, (unsigned long long)a, (unsigned long long)b);
}
bool late() {
  if (g_failed.load(RLX)) return true;
  if (std::chrono::steady_clock::now() < g_deadline) return false;
  fail("deadline");
  return true;
}

A64& note_at(File& f, uint64_t n) { return g_note[lock_note_index(f.id, n) % GFS_LOCK_SLOTS]; }

void hold(File& f, uint64_t t) {
  if (f.holders.fetch_add(1, RLX) != 0) fail("two holders", f.id, t);
  g_own.fetch_add(1, RLX);
  for (int k = 0; k < 8; ++k) std::this_thread::yield();   // waiters gather
  uint64_t v[64], note[64];
  if (!g_slot_first)
    for (uint32_t l = 0; l < 64; ++l) note[l] = note_at(f, t + 1 + l).load(ACQ);
  if (!g_slot_first) std::this_thread::yield();
  for (uint32_t l = 0; l < 64; ++l) v[l] = f.slot[lock_slot_index(t + 1 + l)].load(ACQ);
  uint32_t end = 0;
  while (end < GFS_LOCK_BATCH - 1 && (v[end] >> 63) && (uint32_t)v[end] == (uint32_t)(t + 1 + end) << 2 &&
         (uint32_t)(v[end] >> 32) != (0x80000000u | kNoPage))
    ++end;
  if (t % 4 == 0) std::this_thread::yield();   // notes get lost
  if (g_slot_first)
    for (uint32_t l = 0; l < end; ++l) note[l] = note_at(f, t + 1 + l).load(ACQ);
  for (uint32_t l = 0; l < end; ++l) {
    uint64_t x = v[l];
    if (!f.slot[lock_slot_index(t + 1 + l)].compare_exchange_strong(x, lock_taken(t + 1 + l), AR)) fail("a waiter left", t + 1 + l);
  }
  uint32_t keep = 0;
  while (keep < end && (!g_tags || lock_note_is(note[keep], f.id, t + 1 + keep))) ++keep;
  if (keep < end) {
    g_lost.fetch_add(1, RLX);
    for (uint32_t l = keep; l < end; ++l) f.slot[lock_slot_index(t + 1 + l)].store(v[l], REL);
  }
  for (uint32_t l = 0; l < keep; ++l) {
    f.used[lock_slot_index(t + 1 + l)] = lock_note_read(note[l]);
    f.slot[lock_slot_index(t + 1 + l)].store(lock_decided(t + 1 + l, 0, 1, 0, false), REL);
  }
  f.holders.fetch_sub(1, RLX);
  const uint64_t next = t + 1 + (g_pass_over ? end : keep);
  f.slot[lock_slot_index(next)].store(lock_granted(next), REL);
}

void block(File* fp, uint32_t me, int misses, uint64_t seed) {
  File& f = *fp;
  std::mt19937_64 r(seed * 1000003 + me);
  for (int k = 0; k < misses && !late(); ++k) {
    const uint32_t req = 1 + (uint32_t)(r() % 4000), hist = (uint32_t)(r() % 1026), cap = 1 + (uint32_t)(r() % 1024);
    const uint64_t mine = lock_note(req, hist, cap, me);
    // files go on together, so that their tickets meet in the row
    while (!late()) {
      uint64_t least = ~0ull;
      for (auto& o : g_files) least = std::min(least, o.next.load(RLX));
      if (f.next.load(RLX) <= least + 8) break;
      std::this_thread::yield();
    }
    const uint64_t t = f.next.fetch_add(1, RLX);
    A64& sl = f.slot[lock_slot_index(t)];
    uint64_t v = sl.load(ACQ);
    if (t != 0 && v != lock_granted(t)) {
      note_at(f, t).store(lock_note_tagged(mine, f.id, t), REL);
      while (v != lock_granted(t) && !sl.compare_exchange_weak(v, lock_waiting(t, t & 0xffff), AR, ACQ)) {
      }
      while (v != lock_granted(t)) {
        v = sl.load(ACQ);
        if (v >> 62 == 1 && (uint32_t)v == (uint32_t)lock_covered(t)) break;
        if (late()) return;
        std::this_thread::yield();
      }
    }
    if (t == 0 || v == lock_granted(t)) {
      hold(f, t);
      continue;
    }
    g_for_others.fetch_add(1, RLX);
    const LockNote n = f.used[lock_slot_index(t)];
    if (n.req != (req < kNoteReq ? req : kNoteReq) || n.hist != hist || n.cap != cap || n.bid != me)
      fail("decided on another miss", t, n.bid);
  }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const std::string mode = argv[1];
  const uint32_t files = (uint32_t)atoi(argv[2]), threads = (uint32_t)atoi(argv[3]);
  const int misses = atoi(argv[4]);
  if (files < 1 || files > 16 || threads % files || threads == 0 || (uint64_t)threads * misses / files > GFS_LOCK_SLOTS / 2) return 2;
  if (mode == "no-tag") g_tags = false;
  else if (mode == "note-first") g_slot_first = false;
  else if (mode == "pass-over") g_pass_over = true;
  else if (mode != "notes") return 2;
  for (uint32_t req : {1u, 2046u, 2047u, 2048u, ~0u})
    for (uint32_t hist : {0u, 1025u})
      for (uint32_t cap : {1u, 1024u}) {
        const LockNote n = lock_note_read(lock_note_tagged(lock_note(req, hist, cap, 0x3fffffu), GFS_MAX_FILES - 1, ~0ull));
        if (n.req != (req < 2047 ? req : 2047) || n.hist != hist || n.cap != cap || n.bid != 0x3fffffu) fail("encoding", req, cap);
      }
  if (lock_note(1, 0, 1, 0x400000u) != kNoNote || lock_note(1, 2048, 1, 0) != kNoNote) fail("a note that does not fit");
  if (lock_note_is(0, 0, 0)) fail("cleared memory is a note");
  const char* dl = getenv("LNM_DEADLINE_S");
  g_deadline = std::chrono::steady_clock::now() + std::chrono::seconds(dl ? atoi(dl) : 60);
  for (uint32_t i = 0; i < files; ++i) g_files.emplace_back();
  for (uint32_t i = 0; i < files; ++i) g_files[i].id = 3 + i * GFS_LOCK_NOTE_ROWS;   // one row
  for (int round = 0; round < 4 && !g_failed; ++round) {
    for (auto& f : g_files) {   // opened again: tickets and slots start over
      f.next = 0;
      for (auto& s : f.slot) s = 0;
    }
    std::vector<std::thread> t;
    for (uint32_t i = 0; i < threads; ++i)
      t.emplace_back(block, &g_files[i % files], i, misses, (uint64_t)atoll(argv[5]) * 16 + (uint64_t)round);
    for (auto& x : t) x.join();
  }
  printf("%s: %llu decided for, %llu held, %llu notes lost %s\n", mode.c_str(), (unsigned long long)g_for_others.load(),
         (unsigned long long)g_own.load(), (unsigned long long)g_lost.load(), g_failed ? "-> FAILED" : "-> ok");
  return g_failed ? 1 : 0;
}
