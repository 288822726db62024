// Model of the exchange of the in-register tridiagonal reduction, on the host:
// workgroups that follow the rules of tridiag_steps.hpp (or, as a check of
// the model itself, the faulty rule of leaving a step later) under schedules
// chosen to go wrong.  A workgroup's reads are one reader per column, each of
// which looks at the slot when it is scheduled and needs the step's epoch; the
// workgroup publishes (one word at a time) and goes on when all have it.
//
//   model RULE N [SEED SCHEDULES]
//
// RULE 0: tridiag_leaves; 1: the workgroup also reads in its last step.
// For every workgroup and step, its readers (all, the first or the last column)
// are held until nobody else can move; then SCHEDULES random schedules, in which
// workgroups get very different shares of the time.  Prints the number of
// runs and of those in which somebody waits for ever; exits 1 if there are any.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "tridiag_steps.hpp"

using namespace bitsmoe;

struct Model {
  int rule, n, wgs;
  std::vector<int> ex[2];  // epochs of the words
  struct Wg {
    int i = 0, pub = 0;       // step; next row to publish (n: done)
    bool done = false;
    std::vector<char> have;   // columns read in this step
  };
  std::vector<Wg> wg;

  Model(int rule_, int n_) : rule(rule_), n(n_), wgs((n_ + kTridiagRows - 1) / kTridiagRows), wg(wgs) {
    ex[0].assign(n, 0);
    ex[1].assign(n, 0);
    for (int g = 0; g < wgs; ++g) start(g);
  }
  int r0(int g) const { return g * kTridiagRows; }
  void start(int g) {
    wg[g].pub = r0(g);
    wg[g].have.assign(n, 0);
  }
  // Moves workgroup g by one word, or one look at every word that it still
  // needs (first < 0); `held` columns are not read.  False if it cannot move.
  template <class Held>
  bool move(int g, int first, Held held) {
    Wg& w = wg[g];
    if (w.done) return false;
    const int i = w.i, end = std::min(n, r0(g) + kTridiagRows);
    if (!tridiag_exchanges(n, i)) {
      w.done = true;
      return true;
    }
    while (w.pub < end && !tridiag_word_live(n, i, w.pub)) ++w.pub;
    if (w.pub < end) {
      ex[i & 1][w.pub++] = i + 1;
      return true;
    }
    if (rule == 0 && tridiag_leaves(n, i, r0(g))) {
      w.done = true;
      return true;
    }
    bool all = true, got = false;
    for (int k = 0; k < n; ++k) {  // a reader that finds its word, from column `first` on
      const int c = first < 0 ? k : (first + k) % n;
      if (!tridiag_word_live(n, i, c) || w.have[c]) continue;
      all = false;
      if (held(c)) continue;
      if (ex[i & 1][c] == i + 1) {
        w.have[c] = 1;
        got = true;
        if (first >= 0) break;
      }
    }
    if (!all) return got;
    ++w.i;
    if (rule != 0 && r0(g) + kTridiagRows <= w.i + 1 && r0(g) + kTridiagRows < n)
      w.done = true;
    else
      start(g);
    return true;
  }
  bool finished() const {
    for (const Wg& w : wg)
      if (!w.done) return false;
    return true;
  }
};

int main(int argc, char** argv) {
  const int rule = std::atoi(argv[1]), n = std::atoi(argv[2]);
  const unsigned seed = argc > 3 ? std::atoi(argv[3]) : 0;
  const int schedules = argc > 4 ? std::atoi(argv[4]) : 0;
  long runs = 0, stuck = 0;
  auto run_all = [&](Model& m) {  // everybody, until nobody moves
    for (bool moved = true; moved;) {
      moved = false;
      for (int g = 0; g < m.wgs; ++g)
        while (m.move(g, -1, [](int) { return false; })) moved = true;
    }
    ++runs;
    stuck += !m.finished();
  };
  const int wgs = (n + kTridiagRows - 1) / kTridiagRows;
  for (int x = 0; x < wgs; ++x)
    for (int step = 0; tridiag_exchanges(n, step); ++step)
      for (int kind = 0; kind < 3; ++kind) {
        Model m(rule, n);
        auto held = [&](int c) { return kind == 0 || (kind == 1 ? c == step + 1 : c == n - 1); };
        for (bool moved = true; moved;) {
          moved = false;
          for (int g = 0; g < wgs; ++g)
            while (m.move(g, -1, [&](int c) { return g == x && m.wg[g].i == step && held(c); })) moved = true;
        }
        run_all(m);
      }
  std::mt19937 rng(seed);
  for (int s = 0; s < schedules; ++s) {
    Model m(rule, n);
    std::vector<int> share(wgs);
    for (long t = 0, idle = 0; !m.finished() && idle < 4000; ++t) {
      if (t % 512 == 0)  // new shares now and then: one in three nearly stopped
        for (int& v : share) v = rng() % 3 == 0 ? 1 : 1 + rng() % 200;
      const int g = rng() % wgs;
      bool moved = false;
      for (int k = rng() % (1 + share[g]); k >= 0; --k) moved |= m.move(g, rng() % n, [](int) { return false; });
      idle = moved ? 0 : idle + 1;
    }
    run_all(m);
  }
  std::printf("%ld %ld\n", runs, stuck);
  return stuck != 0;
}
