// Runs meet_splits (csrc/meet.hpp) for the workgroups of a tile through orders of their steps on the word: every order for
// two to four workgroups (four: a wait of one look), random ones for more.  Each share has to be taken exactly once, and
// only when all have arrived.  Prints "orders departures takeovers" or what went wrong.
#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "meet.hpp"

static constexpr int kMax = 16, kStack = 64 << 10;
static ucontext_t scheduler, contexts[kMax];
static std::vector<char> stacks[kMax];
static uint32_t word, taken[kMax];
static bool done[kMax];
static int self_, expected, sharers, patience;

// the choices of one run: from `path` while it lasts, then the first possible one (or a random one)
struct Choice { int taken, of; };
static std::vector<Choice> path;
static size_t at;
static std::mt19937 *dice;
static int choose(int of) {
  if (at == path.size()) path.push_back({dice ? (int)((*dice)() % of) : 0, of});
  return path[at++].taken;
}

struct Word {   // every change and every look is a step of its own
  int looks = 0;
  void step() { const int me = self_; swapcontext(&contexts[me], &scheduler); }
  uint32_t add(int n) { step(); const uint32_t old = word; word += n; return old; }
  uint32_t load() { step(); ++looks; return word; }
  uint32_t set(uint32_t bits) { step(); const uint32_t old = word; word |= bits; return old; }
  void start_clock() {}
  bool late() { return looks >= patience || choose(2) == 1; }
  void nap() {}
};

static void workgroup() {
  const int me = self_;
  Word w;
  const uint32_t take = ts::meet_splits(w, expected, me, me < sharers);
  if (take != 0 && (int)(word & 255u) != expected) { printf("a share is taken before all have arrived\n"); exit(1); }
  taken[me] = take;
  done[me] = true;
  swapcontext(&contexts[me], &scheduler);
}

static long orders, departures, takeovers;
static void run() {
  word = 0;
  at = 0;
  for (int i = 0; i < expected; ++i) {
    done[i] = false;
    getcontext(&contexts[i]);
    contexts[i].uc_stack.ss_sp = stacks[i].data();
    contexts[i].uc_stack.ss_size = kStack;
    contexts[i].uc_link = &scheduler;
    makecontext(&contexts[i], workgroup, 0);
    self_ = i;
    swapcontext(&scheduler, &contexts[i]);   // up to its first step
  }
  for (;;) {
    int alive[kMax], n = 0;
    for (int i = 0; i < expected; ++i)
      if (!done[i]) alive[n++] = i;
    if (n == 0) break;
    self_ = alive[n > 1 ? choose(n) : 0];
    swapcontext(&scheduler, &contexts[self_]);
  }
  for (int s = 0; s < sharers; ++s) {
    int times = 0;
    for (int i = 0; i < expected; ++i) {
      times += taken[i] >> s & 1u;
      takeovers += i != s && (taken[i] >> s & 1u);
    }
    departures += word >> (8 + s) & 1u;
    if (times != 1) { printf("share %d of %d workgroups is taken %d times\n", s, expected, times); exit(1); }
  }
  ++orders;
}

int main() {
  for (auto &s : stacks) s.resize(kStack);
  for (expected = 2; expected <= 4; ++expected)
    for (sharers = 1; sharers <= expected; ++sharers) {
      patience = expected < 4 ? 2 : 1;
      path.clear();
      for (;;) {   // depth first over the choices
        run();
        while (!path.empty() && path.back().taken + 1 == path.back().of) path.pop_back();
        if (path.empty()) break;
        ++path.back().taken;
      }
    }
  std::mt19937 random(5);
  dice = &random;
  for (int i = 0; i < 200000; ++i) {
    expected = 5 + random() % 12;
    sharers = 1 + random() % expected;
    patience = 1 + random() % 4;
    path.clear();
    run();
  }
  printf("%ld %ld %ld\n", orders, departures, takeovers);
  return 0;
}
