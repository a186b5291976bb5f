// The autotuners' decision on planted times (tests/test_tuner.py): what beats no
// choice is entered, what does not is left to it.
#include <cstdio>

#include "host/kplan.hpp"

using namespace cdag;

namespace {
int g_fail = 0;
void expect(bool ok, const char* what) {
  if (!ok) {
    std::printf("FAILED: %s\n", what);
    g_fail = 1;
  }
}
TuneRow row(double choices, double none, int best, double t_best, int variant = 0) {
  TuneRow r;
  for (int ch = 0; ch < kNumChoices; ++ch) r.t[ch] = choices;
  if (best >= 0) r.t[best] = t_best;
  r.t[kNoChoice] = none;
  r.default_variant = variant;
  return r;
}
}  // namespace

int main() {
  const std::pair<int, int> k22{K22, 72}, k32{K32, 72}, k33{K33, 72};
  const auto key = [](const std::pair<int, int>& s) { return std::make_tuple(1, s.first, s.second); };
  TileTable t{{key(k22), 3}, {key(k33), 4}, {std::make_tuple(0, (int)K22, 72), 5}};
  // per shape: no choice is fastest; a choice is; nothing ran; only choices ran
  int64_t n = store_choices({{k22, row(2.0, 1.0, 7, 1.5)}, {k32, row(2.0, 1.0, 9, 0.8)}, {k33, TuneRow{}},
                             {{C1, 8}, row(2.0, kNotTimed, 11, 1.9)}}, 1, false, &t);
  expect(n == 3, "three shapes decided");
  expect(t.count(key(k22)) == 0, "no entry where no choice is fastest");
  expect(t.at(key(k32)) == 9, "the fastest choice");
  expect(t.at(key(k33)) == 4, "nothing timed: the entry stays");
  expect(t.at(key({C1, 8})) == 11, "no choice did not run");
  expect(t.at(std::make_tuple(0, (int)K22, 72)) == 5, "another precision's entry stays");
  t.clear();
  store_choices({{k22, row(2.0, 1.0, 7, 1.0)}}, 1, false, &t);
  expect(t.empty(), "no faster than no choice");
  // uniform: one choice for every shape, by weight; no choice only as one variant
  TuneRow a = row(2.0, 1.0, 3, 1.2, 30), b = row(2.0, 1.0, 5, 1.3, 30);
  a.weight = 10.0;
  n = store_choices({{k22, a}, {k32, b}}, 1, true, &t);
  expect(n == 2 && t.empty(), "uniform: no choice is one variant and fastest");
  b.default_variant = 36;
  n = store_choices({{k22, a}, {k32, b}}, 1, true, &t);
  expect(n == 2 && t.at(key(k22)) == 3 && t.at(key(k32)) == 3, "uniform: the weighted choice");
  b.t[3] = kNotTimed;
  n = store_choices({{k22, a}, {k32, b}}, 1, true, &t);
  expect(t.at(key(k22)) == 5 && t.at(key(k32)) == 5, "uniform: a choice has to run on every shape");
  expect(store_choices({{k22, TuneRow{}}}, 1, true, &t) == 0 && t.at(key(k22)) == 5, "uniform: nothing timed");
  expect(store_choices({}, 1, true, &t) == 0, "uniform: no shapes");
  // what a candidate runs: no choice with the K splits of the reported tile
  HecDesc h{}, d{};
  expect(decompose_candidate({72, 72, 5184}, 8, kNoChoice, 3, K33, 72, &h) == kExtraVariantId, "128 x 128, split BF16");
  decompose({72, 72, 5184}, 8, default_tile(3, K33, 72), 3, &d);
  expect(h.splits == d.splits && h.k_split == d.k_split, "K splits");
  expect(h.tiles_m == 1 && h.tiles_n == 1 && h.tile_count == 8 * h.splits, "tiles");
  expect(decompose_candidate({5184, 72, 72}, 8, kNoChoice, 0, K32, 72, &h) == kExtraVariantId + kNumTiles, "64 x 80");
  if (!g_fail) std::printf("tuner driver: ok\n");
  return g_fail;
}
