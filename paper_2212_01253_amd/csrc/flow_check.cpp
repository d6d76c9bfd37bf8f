// Host-only check of the dataflow schedule's ordering (msl_flow.hpp) and of its rule of residency (flow_admits).
//
// Follows the wavefronts of a launch through its passes, on every grid the schedule serves, and keeps
// for each the set of events that are ordered before its current point: by its own
// program order, by its workgroup's barriers, by its waits for its own stores, and by the elements it
// has read (what their producer's wavefront knew when it stored them).  No kernel boundary and no
// timing counts.  The exchange fields are safe if
//  * a share of X[(i - 1) % 4] is reset in pass i after everybody has read what they need of it in pass i - 1;
//  * a new element of that field is stored in pass i + 2 after every reset of pass i is complete;
//  * a wavefront looks for it in pass i + 3 after every reset of pass i is complete.
//
// Build: hipcc --offload-host-only -std=c++17 -I include -o flow_check flow_check.cpp
// Run:   ./flow_check [late|early]   (the order of all grids instead of each grid's own); prints the grids
//        that are not safe, "OK" and exit status 0 if there are none
#include <cstdio>
#include <cstring>
#include <vector>

#include "msl_flow_host.hpp"

namespace {

constexpr int kPasses = 9;   // two turns of the rotation and one pass more

using Set = std::vector<uint64_t>;

void join(Set& a, const Set& b) {
  for (size_t i = 0; i < a.size(); ++i) a[i] |= b[i];
}

struct Axis {
  int n, L, lines, units;   // points and lanes of a line, lines per workgroup, workgroups
};

struct Model {
  int waves, groups;
  Axis ax[2];               // row pass, column pass
  std::vector<Set> know;    // per (group, wavefront), at its current point
  std::vector<Set> out[2];  // ... when it stored the output of a pass (the last two passes)
  std::vector<bool> open;   // resets issued, not yet waited for
  int bad = 0;

  // events: kind 0 (has read its input) or 1 (its resets are complete) of (pass, group, wavefront)
  size_t event(int kind, int pass, int g, int w) const { return (((size_t)kind * kPasses + pass) * groups + g) * waves + w; }
  static void add(Set& s, size_t e) { s[e >> 6] |= 1ull << (e & 63); }
  static bool has(const Set& s, size_t e) { return (s[e >> 6] >> (e & 63)) & 1; }
  int id(int g, int w) const { return g * waves + w; }
  const Axis& of(int pass) const { return ax[pass & 1 ? 0 : 1]; }   // pass 0 is a column pass

  void need(const Set& s, int kind, int pass) {
    for (int g = 0; g < of(pass).units; ++g)
      for (int w = 0; w < waves; ++w)
        if (!has(s, event(kind, pass, g, w))) {
          ++bad;
          return;
        }
  }
  void meet(int g) {   // a workgroup barrier
    for (int w = 1; w < waves; ++w) join(know[id(g, 0)], know[id(g, w)]);
    for (int w = 1; w < waves; ++w) know[id(g, w)] = know[id(g, 0)];
  }
  // the wavefront that holds element e of a line of axis a at a pass's ends (FlowEnds)
  int holder(const Axis& a, int e) const { return waves == 1 ? 0 : (e % a.L) * a.lines / 64; }
  void complete(int pass, int g, int w) { add(know[id(g, w)], event(1, pass, g, w)); }

  int run(int nz, int ny, bool early) {
    waves = msl::flow_threads(nz, ny) / 64;
    ax[0] = Axis{nz, nz / msl::flow_pts(nz), msl::flow_lines(nz, ny, nz), msl::flow_row_units(nz, ny)};
    ax[1] = Axis{ny, ny / msl::flow_pts(ny), msl::flow_lines(nz, ny, ny), msl::flow_col_units(nz, ny)};
    groups = ax[0].units > ax[1].units ? ax[0].units : ax[1].units;
    const size_t words = (2ull * kPasses * groups * waves + 63) / 64;
    know.assign(groups * waves, Set(words, 0));
    open.assign(groups * waves, false);
    std::vector<int> reset_in(groups * waves, 0);
    for (int i = 0; i < kPasses; ++i) {
      const Axis &a = of(i), &p = of(i + 1);   // this pass's axis and the pass before's
      std::vector<Set>& mine = out[i & 1];
      const std::vector<Set>& theirs = out[(i + 1) & 1];
      mine.assign(groups * waves, Set());
      for (int g = 0; g < a.units; ++g) {
        for (int w = 0; w < waves; ++w) {
          Set& k = know[id(g, w)];
          if (i >= 4) need(k, 1, i - 3);   // its first look at its input: the old values are gone
          if (i >= 1)                      // it has read all of it
            for (int line = g * a.lines; line < (g + 1) * a.lines; ++line)
              for (int e = 0; e < a.n; ++e)
                if (holder(a, e) == w) join(k, theirs[id(e / p.lines, holder(p, line))]);
          if (i >= 1) add(k, event(0, i, g, w));
          if (open[id(g, w)]) {            // late resets: waited for before the pass is computed
            complete(reset_in[id(g, w)], g, w);
            open[id(g, w)] = false;
          }
        }
        meet(g);   // first exchange
        auto issue = [&]() {
          for (int w = 0; w < waves; ++w) {
            if (i >= 2) need(know[id(g, w)], 0, i - 1);
            open[id(g, w)] = true;
            reset_in[id(g, w)] = i;
          }
        };
        if (early && i >= 1) {
          issue();
          for (int w = 0; w < waves; ++w) {
            complete(i, g, w);
            open[id(g, w)] = false;
          }
        }
        meet(g);   // last exchange
        for (int w = 0; w < waves; ++w) {
          if (i >= 3) need(know[id(g, w)], 1, i - 2);
          mine[id(g, w)] = know[id(g, w)];
        }
        if (!early && i >= 1) issue();
      }
    }
    return bad;
  }
};

// Launches that the rule admits, dealt to compute units in the worst way: workgroups of the given
// shares of a compute unit, each to the fullest one that would still take the smallest, until none takes the next.
// Returns whether all of `queues` launches of every mix of two kinds found room.
bool all_fit(int queues, int cus, int per_a, int grid_a, int per_b, int grid_b) {
  if (!msl::flow_admits(queues, cus, per_a, grid_a) || !msl::flow_admits(queues, cus, per_b, grid_b)) return true;
  const int unit = per_a * per_b;   // a compute unit's resource; a workgroup of a takes per_b of it, of b per_a
  for (int na = 0; na <= queues; ++na) {
    int left[2] = {na * grid_a, (queues - na) * grid_b};
    const int share[2] = {per_b, per_a};
    std::vector<int> used(cus, 0);
    for (int c = 0; c < cus; ++c)   // as many units as possible spoiled with a remainder too small for the larger
      for (int k : {share[0] < share[1] ? 0 : 1, share[0] < share[1] ? 1 : 0}) {
        const int big = share[0] > share[1] ? share[0] : share[1];
        while (left[k] > 0 && used[c] + share[k] <= unit && unit - used[c] >= big) {
          used[c] += share[k];
          --left[k];
        }
      }
    for (int k = 0; k < 2; ++k)
      for (int c = 0; c < cus; ++c)
        while (left[k] > 0 && used[c] + share[k] <= unit) {
          used[c] += share[k];
          --left[k];
        }
    if (left[0] + left[1] > 0) return false;
  }
  return true;
}

}  // namespace

int main(int argc, char** argv) {
  int unsafe = 0;
  for (int nz = 16; nz <= 512; nz *= 2)
    for (int ny = 16; ny <= 512; ny *= 2) {
      bool early = msl::flow_resets_early(nz, ny);
      if (argc > 1) early = std::strcmp(argv[1], "early") == 0;
      Model m;
      if (m.run(nz, ny, early) > 0) {
        std::printf("%d x %d: not ordered\n", ny, nz);
        ++unsafe;
      }
    }
  for (int queues : {4, 5, 8, 12, 16, 24, 32})
    for (int cus : {32, 64, 128, 256})
      for (int pa = 4; pa <= 16; ++pa)
        for (int pb = pa; pb <= 16; ++pb)
          for (int ga = 16; ga <= 256; ga *= 2)
            for (int gb = 16; gb <= 256; gb *= 2)
              if (!all_fit(queues, cus, pa, ga, pb, gb)) {
                std::printf("%d queues, %d compute units: %d workgroups at %d and %d at %d do not fit\n", queues, cus, ga, pa,
                            gb, pb);
                ++unsafe;
              }
  if (unsafe) return 1;
  std::printf("OK\n");
  return 0;
}
