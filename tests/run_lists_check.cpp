// The tile lists that launches run in place of the plan's own (Launch::run_*),
// checked on the plan built for one weight set: every 128-tile of the update
// list is covered once by the 256-tiles that run, each of its trace slots is
// the one that the run tile's slot and Pp / 128 name, and entries stay on one XCD's
// queue with padding at its end; and the launches' operands and factors, run in
// scalar arithmetic, give the table's polynomials. Input as for plan_check.cpp (stdin); built
// by tests/test_run_lists.py.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <iostream>
#include <map>
#include <set>
#include <tuple>

#include "plan.hpp"

using namespace slorr;

int main() {
  int dtype, kind, iters, ncoef, n;
  unsigned flags;
  if (!(std::cin >> dtype >> kind >> iters >> flags >> ncoef)) return 2;
  Plan p;
  p.dtype = dtype;
  p.kind = kind;
  p.iters = iters;
  p.flags = flags;
  if (ncoef) {
    p.coeffs.resize(size_t(3) * iters);
    for (double &c : p.coeffs) std::cin >> c;
  }
  std::cin >> n;
  p.n = n;
  for (int i = 0; i < n; ++i) {
    slorr_shape_t s;
    std::cin >> s.rows >> s.cols;
    p.shapes.push_back(s);
  }
  int grad_dtype;
  if (std::cin >> grad_dtype) p.grad_dtype = grad_dtype;     // optional; fp32 otherwise
  if (!(std::cin >> p.eps)) p.eps = 0.0f;                    // optional
  p.mats.resize(size_t(n));
  build_plan(p);
  int bad = 0;
  auto fail = [&](const char *m, int a, int b, int c) {
    if (++bad < 20) std::printf("FAIL %s: %d %d %d\n", m, a, b, c);
  };
  std::map<std::tuple<int, int, int>, int> slot_of;      // 128-tile -> its slot in the plan's list
  for (int e = 0; e < p.pq[kCfg128].count; ++e) {
    const Tile &t = p.tiles[p.pq[kCfg128].first + e];
    if (t.mat >= 0) slot_of[{t.mat, t.tm, t.tn}] = t.slot;
  }
  if (p.upd.count) {
    if (p.upd.count % kXcds) fail("entries per XCD", p.upd.count, 0, 0);
    if (p.upd.first < 0 || size_t(p.upd.first) + p.upd.count > p.tiles.size()) fail("list range", p.upd.first, p.upd.count, 0);
    bool pad[kXcds] = {};
    std::map<std::tuple<int, int, int>, int> seen;
    for (int e = 0; e < p.upd.count; ++e) {
      const Tile &t = p.tiles[p.upd.first + e];
      if (t.mat < 0) {
        pad[e % kXcds] = true;
        continue;
      }
      if (pad[e % kXcds]) fail("tile after padding", e, 0, 0);
      const MatDesc &d = p.mats[t.mat];
      for (int qm = 0; qm < 2; ++qm)
        for (int qn = 0; qn < 2; ++qn) {
          const int tm = 2 * t.tm + qm, tn = 2 * t.tn + qn;
          if (tm * kTile >= d.Pp || tn * kTile >= d.Qp) {
            if (qm + qn == 0) fail("run tile outside its matrix", t.mat, t.tm, t.tn);
            continue;
          }
          seen[{t.mat, tm, tn}]++;
          auto it = slot_of.find({t.mat, tm, tn});
          if (it == slot_of.end()) fail("no such 128-tile", t.mat, tm, tn);
          else if (it->second != t.slot + qn * (d.Pp / kTile) + qm) fail("slot", it->second, t.slot, d.Pp);
        }
    }
    for (const auto &kv : slot_of) {
      auto it = seen.find(kv.first);
      if (it == seen.end() || it->second != 1)
        fail("128-tile not covered once", std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first));
    }
  }
  // a matrix's buffers follow each other without gaps, at multiples of 256
  bool quintic = false;
  for (int t = 0; t < p.iters; ++t) quintic |= p.coeffs[3 * t + 2] != 0.0;
  for (int i = 0; i < p.n; ++i) {
    const MatDesc &d = p.mats[i];
    if (d.empty) continue;
    const size_t px = size_t(d.Pp) * d.Qp * p.iter_bytes(), pa = size_t(d.Pp) * d.Pp * p.iter_bytes();
    if (d.x[0] % 256 || (d.x[0] >> 8) >> 32 || d.x[1] != d.x[0] + px || d.x[2] != d.x[1] + px || d.a != d.x[2] + px ||
        d.b != d.a + (quintic ? pa : 0))
      fail("buffers", i, d.Pp, d.Qp);
  }
  // the symmetric outputs as 64-tiles: every upper tile once, padding at the
  // end of each XCD's queue, at most two per CU; and a queue, two tiles on each
  // of its 32 CUs at a time, ends by 1.3 times the longest tile (k and 500)
  for (const TileRange &r : {p.gram64, p.pp64}) {
    if (!r.count) continue;
    bool pad[kXcds] = {};
    std::map<std::tuple<int, int, int>, int> seen;
    std::multiset<double> end[kXcds];
    double longest = 0.0;
    for (int x = 0; x < kXcds; ++x)
      for (int i = 0; i < 64; ++i) end[x].insert(0.0);
    for (int e = 0; e < r.count; ++e) {
      const Tile &t = p.tiles[r.first + e];
      if (t.mat < 0) continue;
      const MatDesc &d = p.mats[t.mat];
      const double c = 500.0 + (p.gram64.count && r.first == p.gram64.first ? d.Qp : d.Pp);
      const double start = *end[e % kXcds].begin();
      end[e % kXcds].erase(end[e % kXcds].begin());
      end[e % kXcds].insert(start + c);
      longest = std::max(longest, c);
    }
    for (int x = 0; x < kXcds; ++x)
      if (*end[x].rbegin() > 1.3 * longest) fail("64-tile queue", x, int(*end[x].rbegin()), int(longest));
    for (int e = 0; e < r.count; ++e) {
      const Tile &t = p.tiles[r.first + e];
      if (t.mat < 0) {
        pad[e % kXcds] = true;
        continue;
      }
      if (pad[e % kXcds] || t.k1 != 0) fail("64-tile entry", e, t.mat, t.k1);
      if (t.tm > t.tn || t.tn * kSmallTile >= p.mats[t.mat].Pp) fail("64-tile", t.mat, t.tm, t.tn);
      seen[{t.mat, t.tm, t.tn}]++;
    }
    size_t want = 0;
    for (const MatDesc &d : p.mats) want += d.empty ? 0 : size_t(d.Pp / kSmallTile) * (d.Pp / kSmallTile + 1) / 2;
    if (seen.size() != want || want > size_t(2 * kCus)) fail("64-tiles", int(seen.size()), int(want), 0);
    for (const auto &kv : seen)
      if (kv.second != 1) fail("64-tile not covered once", std::get<0>(kv.first), std::get<1>(kv.first), kv.second);
  }
  int run = 0;
  for (const Launch &l : p.launches) {
    const TileRange &r64 = l.op == Op::Gram ? p.gram64 : p.pp64;
    if ((l.op == Op::Gram || l.op == Op::Poly) && r64.count) {
      if (l.run_cfg != kCfg64 || l.run_first != r64.first || l.run_grid != r64.count || l.cfg != kCfg128)
        fail("64-tile run list", l.cfg, l.run_cfg, l.run_grid);
    } else if (l.op == Op::Gram && p.gsplit.count && p.gram_parts == p.gred.count) {
      // one part per tile: the whole tiles
      if (l.run_cfg != kCfg128 || l.run_first != p.gram[kCfg128].first || l.run_grid != p.gram[kCfg128].count)
        fail("whole Gram tiles", l.run_cfg, l.run_first, l.run_grid);
    } else if (l.op == Op::Gram || l.op == Op::Poly) {
      if (l.run_cfg != l.cfg || l.run_first != l.tile_first || l.run_grid != l.grid) fail("Gram / poly run list", l.cfg, l.run_cfg, 0);
    } else if (l.op == Op::Update || l.op == Op::Last) {
      const bool big = p.upd.count > 0;
      run += big;
      if (big ? (l.run_cfg != kCfg256 || l.run_first != p.upd.first || l.run_grid != p.upd.count)
              : (l.run_cfg != l.cfg || l.run_first != l.tile_first || l.run_grid != l.grid))
        fail("update run list", l.cfg, l.run_cfg, l.run_grid);
    }
  }
  // the schedule on a 1 x 1 matrix x: every launch's buffers and factors in
  // scalar arithmetic, against the table's polynomials
  const bool scaled = p.dtype == SLORR_BF16 || p.split;
  const double sx = scaled ? kScaleX16 : 1.0;
  // (eps > 0: X_0 a factor 2^-h smaller, the iterates held in powers of two)
  for (int h : {0, 1, 3, 9, 30})
  for (double x0 : {0.02, 0.3, 0.8}) {
    if (p.prep.count == 0) break;             // no matrix with elements
    if (h && p.growth.empty()) break;
    if (!p.growth.empty() && p.growth.size() != size_t(iters) + 1) fail("growth entries", int(p.growth.size()), iters, 0);
    const double nan = std::nan(""), kappa = 1.25;
    double x[3] = {sx * x0, nan, nan}, A = nan, B = nan, part = nan;
    for (const Launch &l : p.launches) {
      const double c = l.kap || l.poly_kap ? kappa : 1.0;
      const int h0 = l.rescale ? std::max(0, h - l.grow0) : 0, h1 = l.rescale ? std::max(0, h - l.grow1) : 0;
      const double k = std::ldexp(c, -h0), m = std::ldexp(c, h1 - h0), k2 = k * k;
      if (l.rescale != (p.growth.empty() ? 0 : l.op == Op::Poly || (l.run == kRunShort && l.op != Op::Gram) || l.use_a))
        fail("rescale", int(l.op), l.run, l.rescale);
      if (l.run == kRunShort && !p.short_set) fail("short-set flag", l.run, int(l.op), 0);
      if (l.run == kNothing) {
        continue;
      } else if (l.run == kRunShort) {        // one slice: X stays in the buffer of X_T from step 1 on
        const int last = iters == 0 ? 0 : 1 + ((iters - 1) & 1);
        double &X = x[l.op == Op::Gram || l.xin == 0 ? 0 : last];
        if (l.op != Op::Gram) {
          const double G = l.gram_alpha * part;
          x[last] = l.alpha * (l.poly_beta * k2 * m * G + l.poly_alpha * k2 * k2 * m * G * G + l.poly_gamma * m) * X;
        }
        part = x[l.op == Op::Gram ? 0 : last] * x[l.op == Op::Gram ? 0 : last];
      } else if (l.op == Op::Gram) {
        const bool parts = p.gsplit.count && p.gram_parts != p.gred.count;
        (parts ? part : A) = (parts ? 1.0 : double(l.alpha)) * x[l.xin] * x[l.xin];
      } else if (l.op == Op::GramReduce && l.run != kNothing) {
        A = l.alpha * part;
      } else if (l.op == Op::Poly) {
        B = l.beta * k2 * m * A + l.alpha * k2 * k2 * m * A * A + l.gamma * m;
        if (scaled && !(std::fabs(B) < 65504.0)) fail("B beyond fp16", int(B), h, 0);
      } else if (l.op == Op::Update || l.op == Op::Last) {
        const double v = double(l.alpha) * (l.use_a ? A : B) * x[l.xin];
        x[l.xout] = l.fold ? v : l.beta * m * x[l.xin] + v * k2 * m;
        if (scaled && !(std::fabs(x[l.xout]) < 65504.0)) fail("X beyond fp16", int(x[l.xout]), h, 0);
        // held no smaller than a step's ordinary iterate, or as large as its bound allows
        if (h1 && !(std::fabs(x[l.xout]) >= 0.02 * x0 * sx)) fail("X held too small", int(1e6 * x[l.xout]), h, h1);
      }
    }
    double want = std::ldexp(kappa * x0, -h);
    for (int t = 0; t < iters; ++t) {
      const double z = want * want;
      want *= p.coeffs[3 * t] + z * (p.coeffs[3 * t + 1] + z * p.coeffs[3 * t + 2]);
    }
    const int hT = p.growth.empty() ? 0 : std::max(0, h - p.growth.back());
    const double got = std::ldexp(x[iters == 0 ? 0 : 1 + ((iters - 1) & 1)] / sx, -hT);
    if (!(std::fabs(got - want) <= 1e-4 * std::fabs(want) + (h ? 0.0 : 1e-6))) fail("schedule's value", int(1e6 * got), int(1e6 * want), int(100 * x0));
  }
  if (bad) return 1;
  std::printf("OK split=%d run256=%d short=%d small=%d%d lean=%d ws=%zu\n", p.split ? 1 : 0, run, p.short_set ? 1 : 0, p.gram64.count > 0,
              p.pp64.count > 0, p.lean ? 1 : 0, p.ws_bytes);
  return 0;
}
