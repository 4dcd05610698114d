// Host-side checks of liblsq's C ABI that need no GPU, meant to be built with AddressSanitizer and
// UndefinedBehaviorSanitizer on the host code (tests/test_host_sanitizers.py does that): header parsing, the
// max-shape memory plan and every error path that must return before any device work, fed with valid,
// truncated, corrupted and randomly damaged model headers.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <utility>
#include <vector>

#include "../include/lsq.h"
#include "../paper_2010_13887_amd/csrc/die_count.h"

namespace lsq { bool stack_twice(int arch, int M, int d, int beam, int pos, int src); }   // kernels_stack.hip

static int failures = 0;
#define EXPECT(cond)                                                        \
  do {                                                                      \
    if (!(cond)) { std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); ++failures; } \
  } while (0)

// a header as the blob format defines it (256 bytes, little endian), total = what the shapes add up to when asked
static std::vector<unsigned char> header(int arch, int n_enc, int n_dec, int d, int H, int F, int V, int dtype,
                                         uint64_t total) {
  std::vector<unsigned char> h(256, 0);
  std::memcpy(h.data(), "LSQBLOB1", 8);
  int32_t f[17] = {1, arch, n_enc, n_dec, d, H, F, V, 64, arch, arch, dtype, 0, 1, 2, 50, arch ? 8 : 0};
  std::memcpy(h.data() + 8, f, sizeof f);
  float alpha = 1.0f, eps = 1e-5f, topp = 0.f;
  std::memcpy(h.data() + 76, &alpha, 4);
  std::memcpy(h.data() + 80, &eps, 4);
  std::memcpy(h.data() + 84, &topp, 4);
  uint64_t seed = 1234;
  std::memcpy(h.data() + 88, &seed, 8);
  std::memcpy(h.data() + 96, &total, 8);
  return h;
}

// A launch with a group of rows per die, by where its workgroups find themselves: every group of the launch is complete, or it has a workgroup that
// waits for one that is missing (and gives up), or the last workgroup of the launch sees that it has none.
static void placements() {
  using namespace lsq;
  constexpr int N = kDies * kDieGroup;
  uint32_t x = 1;
  auto random = [&] { return (x = x * 1664525u + 1013904223u) >> 8; };
  bool complete_seen = false, missed_seen = false;
  for (int it = 0; it < 4000; ++it) {
    int die[N], order[N];
    const int first = random() % kDies, kind = it % 4;
    for (int b = 0; b < N; ++b) {
      order[b] = b;
      die[b] = (b + first) % kDies;                                        // in turn, from any die
      if (kind == 1 && random() % 64 == 0) die[b] = random() % kDies;      // a few of them astray
      if (kind == 2) die[b] = random() % (1 + random() % kDies);           // anyhow
      if (kind == 3) die[b] = die[b] == first ? (first + 1) % kDies : die[b];   // a die that gets nothing
    }
    if (it % 64 == 2)
      for (int& d : die) d = first;
    for (int b = N - 1; b > 0; --b) std::swap(order[b], order[random() % (b + 1)]);   // the order in which they leave
    bool has[kDies][kDieGroup] = {};
    for (int b = 0; b < N; ++b) has[die[b]][b / kDies] = true;
    for (int G = 1; G <= kDies; ++G) {
      bool complete = true, waits = false;
      for (int g = 0; g < G; ++g) {
        int places = 0;
        for (bool h : has[g]) places += h;
        complete = complete && places == kDieGroup;
        waits = waits || (places > 0 && places < kDieGroup);
      }
      uint64_t word = 0;
      int ends = 0;
      bool there = false;
      for (int b : order) {
        const uint64_t mine = die_word(die[b], b / kDies);
        const bool last = die_launch_ends(word);
        word += mine;
        if (last) { ++ends; there = die_groups_there(word, G); }
      }
      EXPECT(ends == 1 && die_launch_ends(word - 1));
      if (complete) EXPECT(there);
      else EXPECT(waits || !there);
      if (kind == 0) EXPECT(complete);
      complete_seen = complete_seen || complete;
      missed_seen = missed_seen || (!complete && !waits);
    }
  }
  EXPECT(complete_seen && missed_seen);
}

// The workgroups of dies to spare, which go on behind their words: whatever the others do between any two of their steps, each wavefront
// works on the set that the launch began with, and the columns are dealt out once each.  Wavefronts that look for themselves
// behind the word, as they may when nothing is handed on, must be seen to miss it: otherwise this could not tell.
static void spare_workgroups() {
  using namespace lsq;
  constexpr int N = kDies * kDieGroup;
  uint32_t x = 7;
  auto random = [&] { return (x = x * 1664525u + 1013904223u) >> 8; };
  int64_t missed = 0;
  for (int it = 0; it < 2000; ++it) {
    const int G = 1 + it % (kDies - 1), first = it / 7 & 1;
    int order[N], next = 0, seq = first, tickets = 0;
    uint64_t count = 0;
    bool taken[N] = {};
    for (int b = 0; b < N; ++b) order[b] = b;
    for (int b = N - 1; b > 0; --b) std::swap(order[b], order[random() % (b + 1)]);
    auto run = [&](auto&& self) -> void {
      if (next == N) return;
      const int b = order[next++], die = b % kDies;
      auto others = [&] { while (random() % 3 == 0 && next < N) self(self); };
      auto leave = [&] {
        others();
        const bool last = die_launch_ends(count);
        count += die_word(die, b / kDies);
        if (last) seq ^= 1;
        others();
      };
      others();
      if (die < G) {   // a working group's: looked long ago
        leave();
        return;
      }
      int handed = -1, columns = -1;
      die_spare_signs_off([&] { const int seen = seq; others(); return seen; }, [&] { const int mine = tickets++; others(); return mine; },
                          [&](int launch, int mine) { handed = launch; columns = mine; others(); }, leave);
      EXPECT(handed == first);
      EXPECT(columns >= 0 && columns < (kDies - G) * kDieGroup && !taken[columns]);
      if (columns >= 0 && columns < N) taken[columns] = true;
      missed += seq != first;
    };
    while (next < N) run(run);
    EXPECT(tickets == (kDies - G) * kDieGroup && seq == (first ^ 1));
  }
  EXPECT(missed > 0);
}

// Two launches of the stack kernel: only for rows that one cannot hold.
static void two_launches() {
  using lsq::stack_twice;
  for (int M : {1, 20, 66, 128})
    for (int pos : {0, 5, 100, 300, 2000})
      for (int beam : {1, 2, 4}) EXPECT(!stack_twice(0, M, 1024, beam, pos, 30));
  EXPECT(stack_twice(0, 132, 1024, 4, 5, 30) && stack_twice(0, 208, 1024, 4, 5, 30) && stack_twice(0, 130, 1024, 2, 5, 30));
  EXPECT(!stack_twice(0, 212, 1024, 4, 5, 30) && !stack_twice(0, 208, 1024, 4, 91, 30) && !stack_twice(0, 132, 1024, 1, 5, 30));
  EXPECT(!stack_twice(1, 132, 1024, 4, 5, 30) && !stack_twice(0, 132, 768, 4, 5, 30));
}

int main() {
  placements();
  spare_workgroups();
  two_launches();
  size_t n = 0;
  // null / short / wrong magic
  EXPECT(lsq_workspace_bytes(nullptr, 0, 2, 4, 8, &n) == LSQ_E_ARG);
  auto h = header(0, 1, 1, 64, 4, 256, 1000, 0, 0);
  EXPECT(lsq_workspace_bytes(h.data(), 100, 2, 4, 8, &n) == LSQ_E_BLOB);
  EXPECT(lsq_workspace_bytes(h.data(), h.size(), 2, 4, 8, nullptr) == LSQ_E_ARG);
  // the size the shapes add up to: ask the library through a wrong total first (it reports the right one in its message)
  EXPECT(lsq_workspace_bytes(h.data(), h.size(), 2, 4, 8, &n) == LSQ_E_BLOB);
  unsigned long long want = 0;
  const char* msg = lsq_last_error();
  const char* at = std::strstr(msg, "add up to ");
  EXPECT(at != nullptr);
  if (at) std::sscanf(at, "add up to %llu", &want);
  EXPECT(want > 256);
  for (int arch = 0; arch < 2; ++arch)
    for (int dtype = 0; dtype < 2; ++dtype) {
      auto g = header(arch, arch ? 0 : 2, 3, 128, 2, 264, 1003, dtype, 0);
      int rc = lsq_workspace_bytes(g.data(), g.size(), 3, arch ? 1 : 4, 32, &n);
      EXPECT(rc == LSQ_E_BLOB);
      at = std::strstr(lsq_last_error(), "add up to ");
      EXPECT(at != nullptr);
      if (!at) continue;
      std::sscanf(at, "add up to %llu", &want);
      g = header(arch, arch ? 0 : 2, 3, 128, 2, 264, 1003, dtype, want);
      size_t a = 0, b = 0, c = 0;
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 3, arch ? 1 : 4, 32, &a) == LSQ_OK);
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 6, arch ? 1 : 4, 32, &b) == LSQ_OK);
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 3, arch ? 1 : 4, 64, &c) == LSQ_OK);
      EXPECT(a > want && b > a && c > a);          // the plan holds the weights and grows with every maximum
      // limits
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 0, 1, 32, &a) == LSQ_E_ARG);
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 3, LSQ_MAX_BEAM + 1, 32, &a) == LSQ_E_ARG);
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 3, 1, 0, &a) == LSQ_E_ARG);
      EXPECT(lsq_workspace_bytes(g.data(), g.size(), 3, 1, 1 << 20, &a) == LSQ_E_ARG);
      // every single header byte damaged in turn: an error or a plan, never a crash or an overflow
      for (size_t i = 0; i < 104; ++i)
        for (unsigned char v : {(unsigned char)0x00, (unsigned char)0x7f, (unsigned char)0x80, (unsigned char)0xff}) {
          auto bad = g;
          bad[i] = v;
          size_t out = 0;
          int r = lsq_workspace_bytes(bad.data(), bad.size(), 3, arch ? 1 : 4, 32, &out);
          EXPECT(r == LSQ_OK || r == LSQ_E_BLOB || r == LSQ_E_ARG);
        }
    }
  // a pseudo-random walk over whole headers
  uint32_t x = 12345;
  for (int it = 0; it < 20000; ++it) {
    auto g = header(0, 1, 1, 64, 4, 256, 1000, 0, 0);
    for (int k = 0; k < 6; ++k) {
      x = x * 1664525u + 1013904223u;
      g[8 + (x >> 8) % 96] = (unsigned char)(x >> 24);
    }
    size_t out = 0;
    int r = lsq_workspace_bytes(g.data(), g.size(), 1 + (int)(x % 7), 1 + (int)((x >> 3) % 8), 1 + (int)((x >> 6) % 200), &out);
    EXPECT(r == LSQ_OK || r == LSQ_E_BLOB || r == LSQ_E_ARG);
  }
  // calls out of order: state errors, no device work
  lsq_free();
  EXPECT(lsq_decode_step() == LSQ_E_STATE);
  EXPECT(lsq_decode_steps(3) == LSQ_E_STATE);
  int32_t ids[4] = {4, 5, 6, 7}, lens[1] = {4};
  EXPECT(lsq_encode(ids, lens, 1, 4) == LSQ_E_STATE);
  float sc[4];
  int32_t ol[4];
  EXPECT(lsq_get_beams(ids, ol, sc) == LSQ_E_STATE);
  EXPECT(lsq_init(h.data(), h.size(), 2, 4, 8) == LSQ_E_STATE);
  EXPECT(lsq_set_workspace(nullptr, 0, nullptr) == LSQ_E_ARG);
  EXPECT(lsq_set_workspace((void*)3, 1024, nullptr) == LSQ_E_ARG);
  EXPECT(lsq_set_diversity(0, 0.f) == LSQ_E_ARG);
  EXPECT(lsq_set_diversity(2, -1.f) == LSQ_E_ARG);
  EXPECT(lsq_set_diversity(1, 0.f) == LSQ_OK);
  EXPECT(lsq_set_cache_refresh(7) == LSQ_E_ARG);
  EXPECT(lsq_debug_read(LSQ_DBG_SCORE, sc, sizeof sc) == LSQ_E_STATE);
  int64_t counts[4];
  EXPECT(lsq_debug_stack_launches(counts) == LSQ_E_STATE);
  EXPECT(lsq_debug_small_launches(counts) == LSQ_E_STATE);
  EXPECT(lsq_debug_forget_dies() == LSQ_E_STATE);
  EXPECT(lsq_k_packed_weight_bytes(64, 24) == 0);
  EXPECT(lsq_k_packed_weight_bytes(33, 32) == 64u * 32 * 2);
  EXPECT(lsq_k_gemm_add_layernorm_scratch(1, 512, 1024, 4096) >= 512u * 1024 * 4);
  EXPECT(lsq_k_gemm(1, nullptr, nullptr, nullptr, nullptr, 1, 1, 8, 0, nullptr) == LSQ_E_ARG);
  lsq_free();
  std::printf(failures ? "host checks: %d FAILED\n" : "host checks: all passed\n", failures);
  return failures ? 1 : 0;
}
