// Dependencies of the nodes of a graph that a three-stream walk (walk.hpp) is
// added to node by node.  Pure host code; Node is whatever names a node.
//
// Nodes form three sequences, each ordered in itself: the chain (kernels, and
// transfers that a kernel moves), the copy nodes of the upload stream and those
// of the spill stream.  What a stream's next node has to follow, and what an
// event stands for, is then one place in each sequence, and joining two of them
// takes the later place.  No node is added only to join others, and a chain
// node follows the chain node before it and copy nodes only: a graph without
// copy nodes is a plain sequence, whatever the passes and events.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "walk.hpp"

namespace cdag {

template <class Node>
class GraphOrder {
 public:
  GraphOrder(int64_t steps, int64_t passes) {
    for (int r = 0; r < kStreams; ++r) {
      event_[r].resize((size_t)steps);
      pass_[r].resize((size_t)passes);
    }
  }
  void wait(int to, int from, int64_t g) { at_[to].join(event_[from][(size_t)g]); }
  void record(int r, int64_t g) { event_[r][(size_t)g] = at_[r]; }
  void wait_pass(int to, int from, int64_t k) { at_[to].join(pass_[from][(size_t)k]); }
  void record_pass(int r, int64_t k) { pass_[r][(size_t)k] = at_[r]; }
  // What stream r's next node, a chain node or a copy node, depends on.
  void deps_of(int r, bool in_chain, std::vector<Node>* deps) const {
    Place p = at_[r];
    if (in_chain) {
      p.join(at_[S_COMP]);
      p.n[CHAIN] = seq_[CHAIN].size();
    }
    deps->clear();
    for (int q = 0; q < kStreams; ++q)
      if (p.n[q] > 0) deps->push_back(seq_[q][p.n[q] - 1]);
  }
  // `n` was added as stream r's next node; it stands for all that it follows.
  void added(int r, bool in_chain, Node n) {
    const int q = in_chain ? (int)CHAIN : r;
    seq_[q].push_back(n);
    Place p;
    p.n[q] = seq_[q].size();
    at_[r] = p;
    if (in_chain) at_[S_COMP] = p;
  }
  bool copies() const { return !seq_[S_H2D].empty() || !seq_[S_D2H].empty(); }

 private:
  enum { CHAIN = S_COMP };         // the sequences: the chain, copies by stream
  struct Place {                   // how many nodes of each sequence come before
    size_t n[kStreams] = {0, 0, 0};
    void join(const Place& o) {
      for (int q = 0; q < kStreams; ++q) n[q] = std::max(n[q], o.n[q]);
    }
  };
  std::vector<Node> seq_[kStreams];
  Place at_[kStreams];
  std::vector<Place> event_[kStreams], pass_[kStreams];   // per global step, per pass
};

}  // namespace cdag
