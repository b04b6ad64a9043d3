// CPU thread model of the device's per-file miss lock (a FIFO ticket lock whose holder also
// decides for waiters behind it), on the library's slot encoding, run under ThreadSanitizer by
// the CPU tests. Threads stand in for blocks. Each thread misses pages of one file, takes a
// ticket, announces its page, and either holds the lock, is decided for by a holder, is told
// that a holder's window covers its page, or leaves the queue when its page shows up. The
// detector's state is plain memory here, so that ThreadSanitizer checks that one holder's use
// of it happens before the next one's; the window claims and the table are atomics as on the
// device. A block with a window reserves its absent pages, each of which must still be absent
// (no two windows may hold one page at once), then clears the claim; pages are dropped again at
// random, so that misses go on. Checked: one holder at a time, every decided window holds its
// page and overlaps no running claim, every page is reserved by one block, every thread ends
// before the deadline, and the state counts every decision once.
//
// A slot is used again GFS_LOCK_SLOTS tickets later. On the device a waiter looks at its slot
// every few microseconds, in which that many tickets cannot pass; here a thread may not run for
// long, so a new ticket is taken only when every thread's last one is recent enough.
//
// Modes: batch (as on the device), single (room for no waiter: every ticket holds the lock),
// and a planted mistake the checks must catch, drop-taken: a holder forgets the outcome of the
// last waiter it took (that waiter can no longer leave, and waits for ever).
//
// usage: miss_lock_model MODE THREADS MISSES PAGES SEED; prints a line ending in "-> ok"
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <random>
#include <string>
#include <thread>
#include <vector>

#include "gfs_layout.h"

namespace {

using A64 = std::atomic<uint64_t>;
constexpr auto ACQ = std::memory_order_acquire, REL = std::memory_order_release, AR = std::memory_order_acq_rel,
               RLX = std::memory_order_relaxed;

A64 g_next{0};
A64 g_slot[GFS_LOCK_SLOTS], g_note[GFS_LOCK_SLOTS], g_claim[GFS_CLAIMS];
std::vector<std::atomic<uint32_t>> g_table;   // 0 absent, 1 reserved, 2 there
std::atomic<int> g_holders{0};
std::atomic<bool> g_failed{false};
uint32_t g_room = GFS_LOCK_BATCH - 1;
bool g_drop = false;
std::chrono::steady_clock::time_point g_deadline;

constexpr int kMaxThreads = 256;
A64 g_live[kMaxThreads];   // each thread's ticket in use, + 1
thread_local int g_me = 0;

struct State {          // plain: the lock orders it
  uint64_t clock = 0, last = 0;
} g_state;
A64 g_decisions{0}, g_for_others{0}, g_covered{0}, g_left{0};

void fail(const char* what, uint64_t a = 0, uint64_t b = 0) {
  if (!g_failed.exchange(true)) fprintf(stderr, "FAILED: %s (%llu, %llu)\n", what, (unsigned long long)a, (unsigned long long)b);
}
bool late() {
  if (g_failed.load(RLX)) return true;
  if (std::chrono::steady_clock::now() < g_deadline) return false;
  fail("deadline");
  return true;
}

uint64_t granted(uint64_t n) { return (uint32_t)n << 2 | 1u; }
uint64_t left(uint64_t n) { return (uint32_t)n << 2 | 2u; }
uint64_t covered(uint64_t n) { return (uint32_t)n << 2 | 3u; }
uint64_t waiting(uint64_t n, uint64_t page) { return 1ull << 63 | page << 32 | (uint32_t)((uint32_t)n << 2); }
uint64_t taken(uint64_t n) { return 1ull << 62 | (uint32_t)((uint32_t)n << 2); }
uint64_t decided(uint64_t n, uint32_t below, uint32_t above, uint32_t claim) {
  return 1ull << 62 | (uint64_t)(below | above << 10 | claim << 21) << 32 | covered(n);
}
A64& slot(uint64_t n) { return g_slot[n & (GFS_LOCK_SLOTS - 1)]; }

struct Claim {
  bool on;
  uint64_t lo, hi;
};
Claim claim_of(uint64_t v) { return {(v & 1) != 0, v >> 32, (v >> 32) + ((v & 0xffffffffull) >> 1)}; }

void unlock(uint64_t n, const std::vector<Claim>& windows) {
  bool look = !windows.empty();
  while (true) {
    if (look) {
      while (true) {
        uint64_t v = slot(n).load(ACQ);
        bool in = false;
        for (auto& w : windows) in |= ((v >> 32) & 0x7fffffffu) >= w.lo && ((v >> 32) & 0x7fffffffu) < w.hi;
        if (v == left(n) || v == covered(n)) {
          ++n;
        } else if ((v >> 63) && (uint32_t)v == (uint32_t)n << 2 && in) {
          slot(n).compare_exchange_strong(v, covered(n), AR, ACQ);
          ++n;
        } else {
          break;
        }
      }
    }
    g_holders.fetch_sub(1, RLX);   // before the grant: the next holder counts itself after it
    if (slot(n).exchange(granted(n), AR) != left(n)) return;
    g_holders.fetch_add(1, RLX);
    ++n;
    look = true;
  }
}

// one decision on the state: the window around page p
Claim decide(uint64_t p, uint32_t want) {
  g_state.clock += 1;
  g_state.last = p;
  uint64_t lo = p - (g_state.clock % 3 < p ? g_state.clock % 3 : 0), hi = p + want;
  if (hi > g_table.size()) hi = g_table.size();
  return {true, lo, hi};
}

enum { RETRY, WINDOW, STOP };

// a ticket, once none in use is about to be lapped
uint64_t take_ticket() {
  while (!late()) {
    const uint64_t n = g_next.load(RLX);
    bool ok = true;
    for (auto& x : g_live) {
      const uint64_t v = x.load(RLX);
      ok = ok && (v == 0 || n - (v - 1) < GFS_LOCK_SLOTS - 2 * kMaxThreads);
    }
    if (ok) break;
    std::this_thread::yield();
  }
  g_live[g_me].store(g_next.load(RLX) + 1, RLX);   // no later than the ticket taken next
  const uint64_t t = g_next.fetch_add(1, RLX);
  return t;
}

int miss(uint64_t p, uint32_t want, Claim* win, uint32_t* cj) {
  const uint64_t t = take_ticket();
  struct Done {
    ~Done() { g_live[g_me].store(0, RLX); }
  } done;
  if (t != 0) {
    uint64_t v = slot(t).load(ACQ);
    if (v != granted(t)) {
      g_note[t & (GFS_LOCK_SLOTS - 1)].store(want, RLX);
      while (v != granted(t) && !slot(t).compare_exchange_weak(v, waiting(t, p), AR, ACQ)) {
      }
    }
    for (uint32_t n = 0; v != granted(t); ++n) {
      v = slot(t).load(ACQ);
      if (v == granted(t)) break;
      if ((uint32_t)v == (uint32_t)covered(t)) {
        if (v >> 62) {
          const uint32_t w = (uint32_t)(v >> 32);
          *win = {true, p - (w & 0x3ff), p + (w >> 10 & 0x7ff)};
          *cj = w >> 21 & 31;
          g_for_others.fetch_add(1, RLX);
          return WINDOW;
        }
        g_covered.fetch_add(1, RLX);
        while (g_table[p].load(ACQ) == 0 && !late()) {
          bool any = false;
          for (auto& c : g_claim) {
            const Claim k = claim_of(c.load(ACQ));
            any |= k.on && k.lo <= p && p < k.hi;
          }
          if (!any) break;
          std::this_thread::yield();
        }
        return RETRY;
      }
      if ((n & 7) == 7 && g_table[p].load(ACQ) != 0) {
        uint64_t x = slot(t).load(ACQ);
        while (x != granted(t) && x != taken(t) && (uint32_t)x != (uint32_t)covered(t)) {
          if (slot(t).compare_exchange_weak(x, left(t), AR, ACQ)) {
            g_left.fetch_add(1, RLX);
            return RETRY;
          }
        }
      }
      if (late()) return STOP;
      std::this_thread::yield();
    }
  }
  if (g_holders.fetch_add(1, RLX) != 0) fail("two holders");
  // the claims, then (ordered after them) the table
  Claim cl[GFS_CLAIMS];
  uint32_t nfree = 0;
  for (uint32_t i = 0; i < GFS_CLAIMS; ++i) {
    cl[i] = claim_of(g_claim[i].load(ACQ));
    nfree += cl[i].on ? 0 : 1;
  }
  struct Item {
    uint64_t ticket, page;
    uint32_t want;
  };
  std::vector<Item> items{{t, p, want}};
  const uint32_t room = nfree ? (nfree - 1 < g_room ? nfree - 1 : g_room) : 0;
  uint64_t end = t + 1;
  for (; end < t + 65; ++end) {
    uint64_t v = slot(end).load(ACQ);
    if (v == left(end) || v == covered(end)) continue;
    if (!(v >> 63) || (uint32_t)v != (uint32_t)end << 2) break;   // not announced
    if (items.size() > room) break;
    const uint64_t page = v >> 32 & 0x7fffffff;
    if (slot(end).compare_exchange_strong(v, taken(end), AR, ACQ))
      items.push_back({end, page, (uint32_t)g_note[end & (GFS_LOCK_SLOTS - 1)].load(RLX)});
  }
  std::vector<Claim> windows;
  std::vector<uint64_t> outcome(items.size());
  int own = RETRY;
  std::vector<uint32_t> fresh;
  for (size_t i = 0; i < items.size(); ++i) {
    const uint64_t q = items[i].page;
    bool cov = false;
    int32_t f = -1;
    for (uint32_t c = 0; c < GFS_CLAIMS; ++c) {
      cov |= cl[c].on && cl[c].lo <= q && q < cl[c].hi;
      if (!cl[c].on && f < 0) f = (int32_t)c;
    }
    outcome[i] = covered(items[i].ticket);
    if (cov || f < 0 || g_table[q].load(ACQ) != 0) continue;
    Claim w = decide(q, items[i].want);
    for (auto& k : cl) {
      if (!k.on) continue;
      if (k.hi <= q) w.lo = w.lo > k.hi ? w.lo : k.hi;
      else w.hi = w.hi < k.lo ? w.hi : k.lo;
    }
    if (!(w.lo <= q && q < w.hi)) fail("window without its page", q, w.lo);
    cl[f] = w;
    fresh.push_back((uint32_t)f);
    windows.push_back(w);
    g_decisions.fetch_add(1, RLX);
    if (i == 0) {
      own = WINDOW;
      *win = w;
      *cj = (uint32_t)f;
    } else {
      outcome[i] = decided(items[i].ticket, (uint32_t)(q - w.lo), (uint32_t)(w.hi - q), (uint32_t)f);
    }
  }
  for (uint32_t f : fresh) g_claim[f].store(cl[f].lo << 32 | (cl[f].hi - cl[f].lo) << 1 | 1, REL);
  for (size_t i = 1; i < items.size(); ++i)
    if (!(g_drop && i + 1 == items.size())) slot(items[i].ticket).store(outcome[i], REL);
  unlock(end, windows);
  return own;
}

void block(int id, int misses, uint64_t seed) {
  g_me = id;
  std::mt19937_64 r(seed * 1000003 + (uint64_t)id);
  for (int k = 0; k < misses && !late(); ++k) {
    // blocks read near each other, so that windows meet
    const uint64_t p = ((uint64_t)k * 4 + r() % 48) % g_table.size();
    while (g_table[p].load(ACQ) == 0 && !late()) {
      Claim w;
      uint32_t cj = 0;
      const int st = miss(p, 1 + (uint32_t)(r() % 16), &w, &cj);
      if (st == STOP) return;
      if (st == RETRY) continue;
      if (!(w.lo <= p && p < w.hi)) fail("outcome without its page", p, w.lo);
      for (uint64_t q = w.lo; q < w.hi; ++q) {
        uint32_t z = 0;
        if (g_table[q].load(ACQ) == 0 && !g_table[q].compare_exchange_strong(z, 1, AR)) fail("page reserved twice", q, p);
      }
      g_claim[cj].store(0, REL);
      for (uint64_t q = w.lo; q < w.hi; ++q) {
        uint32_t one = 1;
        g_table[q].compare_exchange_strong(one, 2, AR);
      }
    }
    // drop some pages, as eviction does
    for (int e = 0; e < 24; ++e) {
      uint32_t two = 2;
      g_table[r() % g_table.size()].compare_exchange_strong(two, 0, AR);
    }
  }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const std::string mode = argv[1];
  const int threads = atoi(argv[2]), misses = atoi(argv[3]);
  if (threads < 1 || threads > kMaxThreads) return 2;
  g_table = std::vector<std::atomic<uint32_t>>((size_t)atoi(argv[4]));
  if (mode == "single") g_room = 0;
  else if (mode == "drop-taken") g_drop = true;
  else if (mode != "batch") return 2;
  const char* dl = getenv("MLM_DEADLINE_S");
  g_deadline = std::chrono::steady_clock::now() + std::chrono::seconds(dl ? atoi(dl) : 60);
  std::vector<std::thread> t;
  for (int i = 0; i < threads; ++i) t.emplace_back(block, i, misses, (uint64_t)atoll(argv[5]));
  for (auto& x : t) x.join();
  if (!g_failed && g_state.clock != g_decisions.load()) fail("decisions lost", g_state.clock, g_decisions.load());
  for (auto& c : g_claim)
    if (!g_failed && c.load()) fail("claim left over");
  printf("%s: %llu decisions, %llu of them for waiters, %llu covered, %llu left %s\n", mode.c_str(),
         (unsigned long long)g_decisions.load(), (unsigned long long)g_for_others.load(),
         (unsigned long long)g_covered.load(), (unsigned long long)g_left.load(), g_failed ? "-> FAILED" : "-> ok");
  return g_failed ? 1 : 0;
}
