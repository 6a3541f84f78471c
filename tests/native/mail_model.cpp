// The mailboxes of a team in the on-chip form (csrc/sos_mail.h), run through every
// order of the members' steps. A member walks through its subdomains; a sweep is:
// write the edges to each neighbour, publish the sums, then (in either order)
// read the neighbours' edges of this sweep and wait for every member's sums. A
// store becomes visible some time after it was issued, in order per mailbox.
// Prints the number of states, or the first state from which nobody moves on.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <string>
#include <vector>

#include "sos_mail.h"

namespace {

struct Model {
  int members;
  std::vector<int> jobs;  // sweeps of each subdomain
  bool counts_skipped;    // the faulty rule: a subdomain without a sweep takes a number too
  uint32_t first;

  struct Member {
    int job = 0, sweep = 0, published = 0, read = 0, met = 0;  // read: bit per side
    uint32_t seq = 0;
    std::vector<uint32_t> flying[4];  // [side][parity]: issued, not yet visible
  };
  struct State {
    std::vector<Member> m;
    std::vector<uint32_t> box;        // [member][side][parity]: visible words
    std::vector<int> sums;            // [member]: meetings published so far
  };

  std::string key(const State& s) const {
    std::string k;
    auto put = [&](uint32_t v) { k.append((const char*)&v, 4); };
    for (auto& m : s.m) {
      for (int v : {m.job, m.sweep, m.published, m.read, m.met}) put((uint32_t)v);
      put(m.seq);
      for (auto& f : m.flying) {
        put((uint32_t)f.size());
        for (uint32_t v : f) put(v);
      }
    }
    for (uint32_t v : s.box) put(v);
    for (int v : s.sums) put((uint32_t)v);
    return k;
  }
  bool has(int i, int side) const { return side == 0 ? i > 0 : i + 1 < members; }
  // Enters the sweep at (job, sweep), or the next subdomain that has one.
  void enter(Member& m, int i) const {
    while (m.job < (int)jobs.size() && m.sweep >= jobs[m.job]) {
      if (jobs[m.job] > 0) m.seq = sos::mail_next_job(m.seq - 1);  // (seq was moved past the last sweep)
      else if (counts_skipped) ++m.seq;
      ++m.job;
      m.sweep = 0;
    }
    m.published = m.met = 0;
    m.read = 0;
    if (m.job >= (int)jobs.size()) return;
    for (int side = 0; side < 2; ++side)
      if (has(i, side)) m.flying[2 * side + (m.seq & 1)].push_back(m.seq);
  }
  int run() const {
    State s;
    s.m.resize(members);
    s.box.assign(4 * members, 0);
    s.sums.assign(members, 0);
    for (int i = 0; i < members; ++i) {
      s.m[i].seq = first;
      enter(s.m[i], i);
    }
    std::set<std::string> seen{key(s)};
    std::vector<State> todo{s};
    long states = 0;
    while (!todo.empty()) {
      State at = todo.back();
      todo.pop_back();
      ++states;
      int moves = 0, done = 0;
      auto visit = [&](const State& n) {
        ++moves;
        if (seen.insert(key(n)).second) todo.push_back(n);
      };
      for (int i = 0; i < members; ++i) {
        const Member& m = at.m[i];
        for (int f = 0; f < 4; ++f)
          if (!m.flying[f].empty()) {
            State n = at;
            n.box[4 * i + f] = m.flying[f].front();
            n.m[i].flying[f].erase(n.m[i].flying[f].begin());
            visit(n);
          }
        if (m.job >= (int)jobs.size()) {
          ++done;
          continue;
        }
        if (!m.published) {
          State n = at;
          n.m[i].published = 1;
          ++n.sums[i];
          visit(n);
          continue;
        }
        for (int side = 0; side < 2; ++side) {
          if (!has(i, side) || (m.read >> side & 1)) continue;
          const int from = side == 0 ? i - 1 : i + 1;
          if (at.box[4 * from + 2 * (1 - side) + (m.seq & 1)] != m.seq) continue;
          State n = at;
          n.m[i].read |= 1 << side;
          visit(n);
        }
        if (!m.met) {
          bool all = true;
          for (int j = 0; j < members; ++j) all = all && at.sums[j] >= at.sums[i];
          if (all) {
            State n = at;
            n.m[i].met = 1;
            visit(n);
          }
        }
        const int want = (has(i, 0) ? 1 : 0) | (has(i, 1) ? 2 : 0);
        if (m.met && m.read == want) {
          State n = at;
          ++n.m[i].sweep;
          ++n.m[i].seq;
          enter(n.m[i], i);
          visit(n);
        }
      }
      if (!moves && done < members) {
        for (int i = 0; i < members; ++i)
          printf("stuck: member %d at subdomain %d, sweep %d, number %u, met %d, read %d\n", i, at.m[i].job, at.m[i].sweep,
                 at.m[i].seq, at.m[i].met, at.m[i].read);
        return 1;
      }
    }
    printf("states %ld\n", states);
    return 0;
  }
};

}  // namespace

// members counts_skipped first sweeps...
// numbers jobs teams max_inner launch: span, launches between two clears, first number of the launch
int main(int argc, char** argv) {
  if (argc == 6 && !strcmp(argv[1], "numbers")) {
    const uint32_t span = sos::mail_span(atoll(argv[2]), atoll(argv[3]), atoll(argv[4]));
    printf("%u %u %u\n", span, sos::mail_launches(span), sos::mail_first((uint32_t)strtoul(argv[5], nullptr, 10), span));
    return 0;
  }
  if (argc < 5) return 2;
  Model m{atoi(argv[1]), {}, atoi(argv[2]) != 0, (uint32_t)strtoul(argv[3], nullptr, 10)};
  for (int i = 4; i < argc; ++i) m.jobs.push_back(atoi(argv[i]));
  return m.run();
}
