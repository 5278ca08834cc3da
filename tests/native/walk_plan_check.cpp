// CPU driver of the walk form's item list (build_walk_plan in host_core.cpp):
// reads nn; anc[nn]; prob[nn]; nc max_chain max_path max_pieces from argv[1]
// and checks, item by item in launch order, what the kernel relies on. Prints
// "ok <items> <chain> <path>", or the first rule that does not hold.
#include <algorithm>
#include <cstdio>
#include <fstream>
#include <vector>

#include "../../paper_2212_01110_amd/csrc/host_core.h"

#define RULE(c)                                        \
  do {                                                 \
    if (!(c)) {                                        \
      std::printf("item %d: not (%s)\n", k, #c);       \
      return 1;                                        \
    }                                                  \
  } while (0)

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  std::ifstream in(argv[1]);
  int nn = 0, nc = 1, max_chain = 1, max_path = 0, max_pieces = 0, k = -1;
  in >> nn;
  std::vector<int32_t> anc(nn);
  std::vector<double> prob(nn);
  for (auto& a : anc) in >> a;
  for (auto& p : prob) in >> p;
  in >> nc >> max_chain >> max_path >> max_pieces;
  spk::Tree T;
  RULE(spk::build_tree(nn, anc.data(), prob.data(), T) == SPOCK_OK);
  spk::WalkPlan F;
  RULE(spk::build_walk_plan(T, nc, 64, max_chain, max_path, max_pieces, F) == SPOCK_OK);
  RULE(F.rs >= 4 && F.rs <= 64 && (int)F.items.size() == F.nitems * F.rs);
  std::vector<char> q(T.nl, 0), d(T.nl, 0), x(T.nn, 0), sent(T.nn, 0), u(T.nl, 0);
  std::vector<int> parts(T.nl, 0);
  sent[0] = 1;  // (the root state comes with the call)
  for (k = 0; k < F.nitems; ++k) {
    const int* r = &F.items[(size_t)k * F.rs];
    const int i = r[0] / 64, j = r[0] % 64;
    if (k < F.nbwd) {
      RULE(r[2] == T.fc[i] && r[3] == T.nch[i] && j == parts[i]);  // chunks in order
      const int c1 = std::min(T.nch[i], (j + 1) * nc);
      for (int c = j * nc; c < c1; ++c) RULE(T.fc[i] + c >= T.nl || q[T.fc[i] + c]);
      ++parts[i];
      RULE(r[1] >= 1 && r[1] <= std::max(1, max_chain) && r[1] <= F.chain && 3 + r[1] <= F.rs);
      RULE(r[1] == 1 || c1 == T.nch[i]);
      if (c1 < T.nch[i]) continue;
      for (int l = 0, f = i; l < r[1]; ++l) {
        if (l > 0) {
          RULE(r[3 + l] == T.anc[f] && T.nch[T.anc[f]] == 1);
          f = r[3 + l];
        }
        RULE(!d[f]);
        d[f] = 1;
        q[f] = l + 1 == r[1];  // inside a chain q is not published
      }
    } else if (r[1] > 0) {
      const int m = r[1], own = r[2];
      RULE(m >= 2 && m <= F.path && 5 + m <= F.rs && own >= 0 && own <= m);
      RULE(sent[r[4]]);
      for (int l = 0; l <= m; ++l) {
        const int v = r[4 + l];
        if (l > 0) RULE(T.anc[v] == r[3 + l]);
        if (l < m) RULE(d[v]);
        if (l > 0) RULE((l >= own) == !x[v]);  // the first piece through a node writes it
        if (l < m) RULE((l >= own) == !u[v]);
        x[v] = 1;
        if (l < m) u[v] = 1;
      }
      sent[r[4 + m]] = 1;
    } else {
      RULE(sent[i] && d[i]);
      if (j == 0) {
        RULE(!u[i]);
        u[i] = 1;
      }
      for (int c = T.fc[i] + j * nc; c < std::min(T.fc[i] + T.nch[i], T.fc[i] + (j + 1) * nc); ++c) {
        RULE(!x[c]);
        x[c] = sent[c] = 1;
      }
    }
  }
  k = F.nitems;
  for (int i = 0; i < T.nl; ++i) RULE(d[i] && u[i]);
  for (int c = 1; c < T.nn; ++c) RULE(x[c]);
  std::printf("ok %d %d %d\n", F.nitems, F.chain, F.path);
  return 0;
}
