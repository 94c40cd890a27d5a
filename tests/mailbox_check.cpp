// Model of the camera loops' mailbox exchange (mail_put, mail_take) and check
// of its wait's bound (WaitBound).
//
// Wavefronts own cameras strided over them and go through K iterations; in
// each, for each of its cameras in turn, a wavefront waits for the records of
// the camera's neighbours, `lanes` of them a pass, each pass in rounds that
// read every word of the pass once, and then publishes the camera's next
// record.  A record is `words` tagged words, two records a camera, alternated
// by iteration.  Words are stored and read one by one: a stored word lands at
// any later time and in any order (in program order for one address).
//
// Checked: every value taken is the neighbour's value of that iteration, every
// wavefront finishes, under random schedules and, for small graphs, under
// every schedule; a wavefront that never publishes ends the others within the
// bound.  The mistakes planted in the model (one record a camera; a tag that
// an earlier launch left) must be found.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <string>
#include <vector>

#include "wait_bound.h"

struct Word {
  int tag = 0, value = 0;
};

struct Graph {
  int N;
  std::vector<std::vector<int>> nb;   // neighbours, the pairs listed at both of their cameras
};

static Graph band(int N, int reach, bool ring) {
  Graph g{N, std::vector<std::vector<int>>(N)};
  for (int i = 0; i < N; ++i)
    for (int k = 1; k <= reach; ++k) {
      const int j = i + k;
      if (j >= N && !ring) continue;
      g.nb[i].push_back(j % N);
      g.nb[j % N].push_back(i);
    }
  return g;
}

struct Config {
  Graph g;
  int waves, lanes, words, K;
  int records = 2;      // 1: the planted mistake
  bool stale = false;   // records of an earlier launch not cleared
  int silent = -1;      // this wavefront publishes nothing after its first records
};

static int value_of(int cam, int k, int w) { return 1 + w + 10 * (k + 100 * cam); }

// One wavefront's place in the program.
struct Wave {
  int k = 0, cam = 0, pass = 0, pos = 0;   // pos: the next word of the round
  bool ok = true;                          // every word of the round so far carried the tag
  bool done = false, dead = false;
};

struct Store {
  int addr;
  Word w;
};

struct State {
  std::vector<Word> mem;
  std::vector<std::vector<Store>> flight;   // per wavefront, in program order
  std::vector<Wave> waves;
  bool wrong = false;

  std::string key() const {
    std::string s;
    auto put = [&](int v) { s.append(reinterpret_cast<const char*>(&v), sizeof v); };
    for (const Word& w : mem) put(w.tag), put(w.value);
    for (const auto& f : flight) {
      put((int)f.size());
      for (const Store& x : f) put(x.addr), put(x.w.tag), put(x.w.value);
    }
    for (const Wave& w : waves) put(w.k), put(w.cam), put(w.pass), put(w.pos), put(w.ok), put(w.done);
    return s;
  }
};

static int addr(const Config& c, int k, int cam, int w) {
  return ((c.records == 2 ? k & 1 : 0) * c.g.N + cam) * c.words + w;
}

static void publish(const Config& c, State& s, int wave, int cam, int k) {
  for (int w = 0; w < c.words; ++w) s.flight[wave].push_back({addr(c, k, cam, w), Word{k + 1, value_of(cam, k, w)}});
}

static State start(const Config& c) {
  State s;
  s.mem.resize(2 * c.g.N * c.words);
  if (c.stale)
    for (int cam = 0; cam < c.g.N; ++cam)
      for (int w = 0; w < c.words; ++w) s.mem[addr(c, 1, cam, w)] = Word{2, -1};
  s.flight.resize(c.waves);
  s.waves.resize(c.waves);
  for (int v = 0; v < c.waves; ++v) {
    for (int cam = v; cam < c.g.N; cam += c.waves) publish(c, s, v, cam, 0);
    s.waves[v].cam = v;
    if (v >= c.g.N) s.waves[v].done = true;
  }
  return s;
}

// The next read of wavefront v (or, at the end of a pass, what follows it).
// Returns whether a wait's round ended without its words.
static bool step(const Config& c, State& s, int v) {
  Wave& w = s.waves[v];
  const std::vector<int>& nb = c.g.nb[w.cam];
  const int first = w.pass * c.lanes, count = std::min(c.lanes, (int)nb.size() - first);
  if (count > 0 && w.pos < count * c.words) {
    const int other = nb[first + w.pos / c.words], word = w.pos % c.words;
    const Word& x = s.mem[addr(c, w.k, other, word)];
    w.ok = w.ok && x.tag == w.k + 1;
    // (the value counts only if the round succeeds: a word whose tag matches
    // holds it)
    if (x.tag == w.k + 1 && x.value != value_of(other, w.k, word)) s.wrong = true;
    ++w.pos;
    return false;
  }
  if (!w.ok) {   // again
    w.pos = 0;
    w.ok = true;
    return true;
  }
  w.pos = 0;
  if (count > 0 && first + count < (int)nb.size()) {
    ++w.pass;
    return false;
  }
  w.pass = 0;
  if (v != c.silent && w.k + 1 < c.K) publish(c, s, v, w.cam, w.k + 1);
  w.cam += c.waves;
  if (w.cam >= c.g.N) {
    w.cam = v;
    if (++w.k == c.K) w.done = true;
  }
  return false;
}

static void land(State& s, int v, int i) {
  s.mem[s.flight[v][i].addr] = s.flight[v][i].w;
  s.flight[v].erase(s.flight[v].begin() + i);
}

// A store may land unless one to the same address is ahead of it.
static bool may_land(const State& s, int v, int i) {
  for (int j = 0; j < i; ++j)
    if (s.flight[v][j].addr == s.flight[v][i].addr) return false;
  return true;
}

// Every schedule of a small configuration: false if a value is wrong or a
// state that no schedule leaves is reached before the end.
static bool every_schedule(const Config& c, long* states) {
  // forward search over all states; then every state must reach an end, which
  // is checked backwards over the recorded edges
  std::vector<State> all;
  std::vector<std::vector<int>> back;
  std::vector<char> good;
  std::map<std::string, int> index;
  auto id = [&](const State& s) {
    const int n = (int)all.size();
    const auto at = index.emplace(s.key(), n);
    if (!at.second) return at.first->second;
    all.push_back(s);
    back.emplace_back();
    good.push_back(0);
    return n;
  };
  id(start(c));
  std::vector<int> ends;
  for (int n = 0; n < (int)all.size(); ++n) {
    const State cur = all[n];
    if (cur.wrong) return false;
    bool done = true;
    for (int v = 0; v < c.waves; ++v) {
      if (!cur.waves[v].done) {
        done = false;
        State s = cur;
        step(c, s, v);
        const int m = id(s);
        back[m].push_back(n);
      }
      for (int i = 0; i < (int)cur.flight[v].size(); ++i)
        if (may_land(cur, v, i)) {
          State s = cur;
          land(s, v, i);
          const int m = id(s);
          back[m].push_back(n);
        }
    }
    if (done) ends.push_back(n), good[n] = 1;
    if (all.size() > 3000000) std::printf("too many states\n"), std::exit(1);
  }
  for (size_t q = 0; q < ends.size(); ++q)
    for (int p : back[ends[q]])
      if (!good[p]) good[p] = 1, ends.push_back(p);
  *states = (long)all.size();
  for (char g : good)
    if (!g) return false;
  return true;
}

// A random schedule: false on a wrong value or if the wavefronts do not finish.
static bool random_schedule(const Config& c, unsigned seed) {
  std::mt19937 rng(seed);
  State s = start(c);
  const int slow = rng() % c.waves;   // now and then one wavefront hardly runs
  const unsigned mode = rng() % 3, delay = 1 + rng() % 8;
  for (long n = 0; n < 4000000; ++n) {
    bool done = true;
    for (const Wave& w : s.waves) done = done && w.done;
    if (s.wrong) return false;
    if (done) return true;
    int v = rng() % c.waves;
    if (mode == 1 && v == slow && rng() % 50) continue;
    if (rng() % delay == 0 && !s.flight[v].empty()) {
      const int i = rng() % s.flight[v].size();
      if (may_land(s, v, i)) land(s, v, i);
    } else if (!s.waves[v].done) {
      step(c, s, v);
    }
  }
  return false;
}

// One wavefront never publishes: every wavefront ends, the failure is raised
// and no wait lasts more than the bound and the rounds between two looks.
static bool expiry(Config c, unsigned seed, unsigned long long ticks_per_round) {
  std::mt19937 rng(seed);
  c.silent = rng() % c.waves;
  State s = start(c);
  std::vector<WaitBound> wb(c.waves);
  std::vector<unsigned long long> clock(c.waves, 0), wait(c.waves, 0);
  bool failed = false;
  // whole rounds at a time: step() until the round ends or the wait does
  for (long n = 0; n < 200000000; ++n) {
    bool done = true;
    for (const Wave& w : s.waves) done = done && w.done;
    if (done) return failed;
    const int v = rng() % c.waves;
    while (!s.flight[v].empty()) land(s, v, 0);
    if (s.waves[v].done) continue;
    const Wave before = s.waves[v];
    bool again = false;
    do again = step(c, s, v);
    while (!again && !s.waves[v].done && s.waves[v].pos > 0);
    if (!again) {
      const Wave& w = s.waves[v];
      if (w.k != before.k || w.cam != before.cam || w.pass != before.pass) wb[v] = WaitBound(), wait[v] = 0;
      continue;
    }
    clock[v] += ticks_per_round;
    wait[v] += ticks_per_round;
    if (wait[v] > kWaitTicks + 2 * kWaitCheck * ticks_per_round) return false;
    if (!wb[v].go_on([&] { return clock[v]; }, [&] { return failed; })) {
      failed = true;
      s.waves[v].dead = s.waves[v].done = true;   // untraced: the loop is left
    }
  }
  return false;
}

// go_on itself: no look before kWaitCheck rounds, the end at the bound or at
// the first look after a failure, clocks that wrap included.
static bool bound() {
  for (unsigned long long base : {0ull, ~0ull - kWaitTicks / 2}) {
    WaitBound w;
    unsigned long long t = base;
    long looks = 0, rounds = 0;
    const unsigned long long per = kWaitTicks / 10000;
    while (w.go_on([&] { ++looks; return t; }, [] { return false; })) t += per, ++rounds;
    if (looks != (rounds + 1) / kWaitCheck) return false;
    const unsigned long long took = t - base;
    if (took < kWaitTicks || took > kWaitTicks + 2 * kWaitCheck * per) return false;
  }
  WaitBound w;
  unsigned rounds = 1;
  while (w.go_on([] { return 7ull; }, [] { return true; })) ++rounds;
  return rounds == kWaitCheck;
}

static int fail(const char* what, int a = 0, int b = 0) {
  std::printf("FAIL %s (%d, %d)\n", what, a, b);
  return 1;
}

int main() {
  if (!bound()) return fail("bound");
  // every schedule: one and two cameras a wavefront, a pass each
  long states = 0, total = 0;
  for (const Config& c : {Config{band(2, 1, false), 2, 4, 1, 4}, Config{band(3, 1, false), 3, 4, 1, 3},
                          Config{band(3, 1, true), 2, 4, 1, 3}, Config{band(4, 1, false), 2, 1, 1, 3},
                          Config{band(2, 1, false), 2, 4, 2, 3}}) {
    if (!every_schedule(c, &states)) return fail("every schedule", c.g.N, c.waves);
    total += states;
  }
  // random schedules: up to four cameras a wavefront and four passes a camera
  int runs = 0;
  for (int N : {2, 5, 12, 24})
    for (int waves : {1, 3, 6, 24})
      for (int lanes : {1, 2, 8})
        for (bool ring : {false, true}) {
          const Config c{band(N, std::min(N - 1, 4) / (ring ? 2 : 1) + (N == 2 && ring), ring), waves, lanes, 3, 6};
          for (unsigned seed = 0; seed < 6; ++seed, ++runs)
            if (!random_schedule(c, seed)) return fail("random schedule", N, waves);
        }
  for (unsigned seed = 0; seed < 8; ++seed) {
    const Config c{band(8, 2, false), seed % 2 ? 8 : 3, 2, 3, 6};
    if (!expiry(c, seed, 100 + 1500 * (seed % 3))) return fail("expiry", (int)seed);
  }
  // planted mistakes
  int found = 0;
  for (unsigned seed = 0; seed < 20; ++seed) {
    Config c{band(6, 2, false), 3, 2, 3, 6};
    c.records = 1;
    found += !random_schedule(c, seed);
  }
  if (!found) return fail("one record a camera not found");
  Config one{band(2, 1, false), 2, 4, 1, 4};
  one.records = 1;
  if (every_schedule(one, &states)) return fail("one record a camera not found in every schedule");
  Config stale{band(2, 1, false), 2, 4, 1, 4};
  stale.stale = true;
  if (every_schedule(stale, &states)) return fail("stale tags not found");
  std::printf("OK states %ld schedules %d\n", total, runs);
  return 0;
}
