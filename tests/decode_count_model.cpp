// Host model of one decode step on one sequence: waves that read the tables, workgroups that count, the last of
// which moves the tables - every order in which they can start and come to count, by the arithmetic of the kernels
// (bc_decode_count.h).  Prints for every shape the number of states seen and of ends in which something is wrong.
//   argv[1] == "uncounted": the model with a mistake planted, workgroups without rows count nowhere.
#include <cstdio>
#include <cstring>
#include <set>
#include <string>
#include <vector>

#include "bc_decode_count.h"

using namespace bc;

namespace {

constexpr int kSplitRows = 33, kChunkRows = 32;      // whole up to 32 rows, then a chunk for every 32

struct Shape {
  int Hkv, max_chunks, waves, forced;
  bool ticket_per_wave;     // of a workgroup with rows: one for each wave, or one
  int L_old, c;             // resident rows and ratio (P = L_old - w; w = c - 1 closes the window)
  bool evicts;
};

struct View { int nb, w; };

struct State {
  std::vector<int> read;         // per wave: 0 not started, 1 tables as before the step, 2 as behind it
  std::vector<int> ticketed;     // per wave of a whole sequence
  std::vector<int> done;         // per workgroup: 1 has counted, 2 drew its pair's ticket (or has none to draw)
  std::vector<int> written, arrivals, folded;
  int tickets = 0, moved = 0;
  bool broken = false;
  std::string key() const {
    std::string k;
    for (auto* v : {&read, &ticketed, &done, &written, &arrivals, &folded})
      for (int x : *v) k += char('0' + x);
    return k + char('0' + tickets) + char('0' + moved) + char('0' + broken);
  }
};

struct Model {
  Shape s;
  bool plant;
  std::set<std::string> seen;
  long bad = 0;

  int groups() const { return s.Hkv * s.max_chunks; }
  // what a wave that found the tables so makes of them
  void derive(int found, int chunk, int& nchunks, bool& has) const {
    int L = s.L_old + 1;
    if (found == 2) L = s.evicts ? s.L_old + 1 - s.c + 1 + 1 : s.L_old + 2;
    const SequenceCut cut = cut_sequence(L, s.forced, s.max_chunks, kSplitRows, kChunkRows);
    nchunks = cut.nchunks;
    has = chunk < nchunks;
  }
  int own() const { return s.ticket_per_wave ? s.waves : 1; }
  int tickets_wanted(int nchunks) const {
    return plant ? (nchunks > 1 ? s.Hkv : s.Hkv * own()) : tickets_due(s.Hkv, own(), nchunks, s.max_chunks);
  }
  int arrivals_wanted(int nchunks) const { return plant ? nchunks : arrivals_due(true, nchunks, s.max_chunks); }
  void draw(State& t, int nchunks) const {
    if (++t.tickets < tickets_wanted(nchunks)) return;
    if (t.tickets > tickets_wanted(nchunks)) { t.broken = true; return; }
    t.tickets = 0;
    ++t.moved;
  }

  std::vector<State> next(const State& t) const {
    std::vector<State> out;
    for (int g = 0; g < groups(); ++g) {
      const int kvh = g / s.max_chunks, chunk = g % s.max_chunks;
      bool all_read = true, same = true;
      for (int i = 0; i < s.waves; ++i) {
        const int wv = g * s.waves + i;
        if (t.read[wv] == 0) {
          all_read = false;
          State u = t;
          u.read[wv] = u.moved ? 2 : 1;
          out.push_back(u);
          continue;
        }
        same = same && t.read[wv] == t.read[g * s.waves];
        int n; bool has;
        derive(t.read[wv], chunk, n, has);
        if (n == 1 && has && s.ticket_per_wave && !t.ticketed[wv]) {
          State u = t;
          u.ticketed[wv] = 1;
          draw(u, n);
          out.push_back(u);
        }
      }
      if (!all_read || t.done[g] == 2) continue;
      State u = t;
      int n; bool has;
      derive(t.read[g * s.waves], chunk, n, has);
      if (!same) {                      // waves of a workgroup that do not agree on what they are
        u.broken = true; u.done[g] = 2;
        out.push_back(u);
        continue;
      }
      if (t.done[g] == 1) {             // the pair's ticket, behind the fold
        draw(u, n); u.done[g] = 2;
        out.push_back(u);
        continue;
      }
      const CloseBy move = plant && !has ? CloseBy::nothing : closing_move(true, has, n);
      u.done[g] = 2;
      if (move == CloseBy::ticket) {
        if (!(has && s.ticket_per_wave)) draw(u, n);
      } else if (move == CloseBy::arrival) {
        if (has) u.written[g] = 1;
        if (++u.arrivals[kvh] == arrivals_wanted(n)) {
          u.arrivals[kvh] = 0;
          for (int ch = 0; ch < n; ++ch) u.broken = u.broken || !u.written[kvh * s.max_chunks + ch];
          ++u.folded[kvh];
          u.done[g] = 1;
        }
      }
      out.push_back(u);
    }
    return out;
  }
  void run() {
    State t;
    t.read.assign(groups() * s.waves, 0); t.ticketed = t.read;
    t.done.assign(groups(), 0); t.written = t.done;
    t.arrivals.assign(s.Hkv, 0); t.folded = t.arrivals;
    std::vector<State> work{t};
    seen.insert(t.key());
    while (!work.empty()) {
      const State u = work.back();
      work.pop_back();
      const std::vector<State> more = next(u);
      if (more.empty()) {               // all is done: one step of the tables, one fold, counters at zero
        int n; bool has;
        derive(1, 0, n, has);
        bool ok = !u.broken && u.moved == 1 && u.tickets == 0;
        for (int x : u.arrivals) ok = ok && x == 0;
        for (int x : u.folded) ok = ok && x == (n > 1 ? 1 : 0);
        bad += !ok;
      }
      for (const State& v : more)
        if (seen.insert(v.key()).second) work.push_back(v);
    }
  }
};

}  // namespace

int main(int argc, char** argv) {
  const bool plant = argc > 1 && !strcmp(argv[1], "uncounted");
  for (int Hkv : {1, 2})
    for (int chunks : {1, 2, 3})
      for (int waves : {1, 2})
        for (int per_wave : {0, 1})
          for (int forced : {0, 64})
            for (int L : {1, 30, 31, 32, 33, 63, 64, 65, 95})
              for (int evicts : {0, 1}) {
                if (Hkv * chunks * waves > 6 || L + 1 > (forced ? forced : 32) * chunks) continue;
                if (evicts && L < 8) continue;
                Model m{Shape{Hkv, chunks, waves, forced, per_wave != 0, L, 4, evicts != 0}, plant, {}, 0};
                m.run();
                printf("Hkv=%d chunks=%d waves=%d per_wave=%d forced=%d L=%d evicts=%d states=%zu bad=%ld\n", Hkv, chunks,
                       waves, per_wave, forced, L, evicts, m.seen.size(), m.bad);
              }
  return 0;
}
