// Corner records of the rotate-back on grains whose first segment has no
// node (its one slot, slot 0, is written by no sweep): every slot that a
// record leads to is a node's.  Built and run by tests/test_host_records.py.
#include <cmath>
#include <cstdio>
#include <vector>

#include "plan.hpp"

namespace {

int fails = 0;

qc::Shape regular(int n, double side, double turn, double cx) {
  qc::Shape s;
  s.kind = 1;
  const double rc = side / (2.0 * std::sin(M_PI / n));
  for (int m = 0; m < n; ++m) {
    const double a = -0.5 * M_PI - M_PI / n + 2.0 * M_PI * m / n + 2.0 * M_PI * turn;
    s.vx.push_back(cx + rc * std::cos(a));
    s.vy.push_back(rc * std::sin(a));
  }
  return s;
}

void run(const char* name, int nx, int ny, qc::Shape shape) {
  qc::Plan p;
  p.nx = nx;
  p.ny = ny;
  p.h = 0.4;
  p.x0 = -0.5 * nx * p.h;
  p.y0 = -0.5 * ny * p.h;
  p.n_theta = 8;
  p.n_poles = 2;
  p.t = 0.4;
  p.ncomp = 1;
  p.tc_rel = {1.0};
  for (int k = 0; k < p.n_theta; ++k) p.eta.push_back(1.0);
  p.shapes = {shape};
  qc::build_plan(p);
  std::vector<char> node(static_cast<size_t>(p.nslot), 0);
  for (int64_t s = 0; s < p.nseg; ++s)
    for (int t = 0; t < p.seg_n[s]; ++t) node[static_cast<size_t>(p.seg_slot0[s] + t)] = 1;
  if (node[0]) {
    std::printf("FAIL: %s: the first segment has a node\n", name);
    ++fails;
  }
  int64_t missing = 0, bad = 0;
  for (const std::vector<int32_t>* rb : {&p.rb4, &p.rb4_pair})
    for (size_t i = 0; i + 3 < rb->size(); i += 4) {
      const int32_t* r = &(*rb)[i];
      for (int q = 0; q < 4; ++q) {
        missing += r[q] < 0;
        const int32_t sl = r[q] < 0 ? qc::record_node(r[0], r[1], r[2], r[3]) : r[q];
        bad += sl < 0 || sl >= p.nslot || !node[static_cast<size_t>(sl)];
      }
    }
  if (missing == 0 || bad > 0) {
    std::printf("FAIL: %s: %lld corners that are no nodes, %lld slots that no sweep writes\n", name,
                static_cast<long long>(missing), static_cast<long long>(bad));
    ++fails;
  }
}

}  // namespace

int main() {
  run("turned square", 12, 12, regular(4, 0.93 * 12 * 0.4, 0.1, 0.0));
  run("turned square without pairs", 30, 30, regular(4, 0.93 * 30 * 0.4, 0.07, 0.0));
  run("pentagon", 13, 14, regular(5, 2.4, 0.17, 0.1));
  std::printf(fails ? "FAILED\n" : "OK\n");
  return fails ? 1 : 0;
}
