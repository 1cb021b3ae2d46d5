// Plan building: validation of the static arguments, canonical orientation,
// shape grouping, launch schedule, tile/chunk lists and workspace layout.
#include "plan.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <queue>
#include <stdexcept>
#include <utility>

namespace slorr {

namespace {

constexpr int64_t kMaxShort = 16384;
constexpr int64_t kMaxLong = 1 << 20;
constexpr int64_t kMaxElems = (int64_t(1) << 31) - 1;
// the GEMM kernels address each operand matrix (padded canonical shape, in
// the iterate type) through a buffer resource with 32-bit byte offsets
constexpr int64_t kMaxIterBytes = int64_t(1) << 31;
constexpr int64_t kMinBigTiles = 2 * kCus;  // two 256-tiles per CU
constexpr double kMaxEdgeWaste = 1.25;      // work of 256-tiles with edges over that of 128-tiles
constexpr int64_t kMinGramUnits = 2 * kCus; // Gram blocks wanted per launch (two per CU)
constexpr int kMaxGramParts = 16;           // k parts per Gram tile at most
// split only Gram tiles this many k-slabs long, into parts of at least this
// many slabs: fp16 slabs (64 values of k) are bound by their load latency
// (about 0.7 us on a 128-tile), fp32 slabs (32 values) by their MFMAs (0.75 us
// in split form, 1.7 us on fp32 MFMA), and a reduce launch costs about 7 us
constexpr int kMinSplitSlabs16 = 32, kMinPartSlabs16 = 8;
// sets of short matrices: slices per matrix, and Gram partials read per step
constexpr int kMaxShortSlices = 8, kMaxShortReads = 1600;
constexpr int64_t kMaxSmallTiles = 2 * kCus;   // 64-tiles of a launch
// a 64-tile's start and end in values of k, and the time of an XCD's queue of
// them over that of the longest tile, up to which they are used
constexpr double kSmallTileFixed = 500.0, kMaxQueueSpan = 1.3;
constexpr int kMinSplitSlabs32 = 8, kMinPartSlabs32 = 4;

Tile make_tile(int32_t mat, int32_t tm, int32_t tn, int32_t slot) {
  Tile t{};
  t.mat = mat;
  t.tm = tm;
  t.tn = tn;
  t.slot = slot;
  return t;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int32_t round_up(int32_t x, int32_t m) { return (x + m - 1) / m * m; }

// X buffer holding the iterate after t steps: X_0 stays in x[0] (the last
// step's trace reads it), later iterates alternate between x[1] and x[2].
int32_t xbuf(int t) { return t == 0 ? 0 : 1 + ((t - 1) & 1); }

// Whether every intermediate of an fp32 set's iteration fits the split form's
// fp16 range, from the coefficient table alone: u bounds the singular values
// of the iterate (X_0' = W / 2^e has none above 1, and the first step's
// polynomial sees kappa X_0' = X_0, also <= 1), so |X_ij| <= u, |A_ij| <= u^2
// and |B_ij| <= max |a + b x^2 + c x^4| on [0, u] (times kappa < 2 in the
// first step). The scales (4096, 4096, 1024) leave fp16 (65504) room for
// u <= 3.5 and |B_ij| <= 58. The built-in schedules stay below 2.1 and 9;
// an explicit table that may exceed the range keeps the fp32 MFMA kernels. So
// does one whose linear terms, which the small singular values follow, shrink
// the iterate below half of X_0 on the way (or at the end): it would come near
// the split form's smallest value, 2^-36, which fp32 does not have (1e-4 times
// X_0 and back by the next steps, 200 x 300: gradient off by 1.0e-5 against
// 2.6e-7). The built-in linear terms are all above 1.
// `growth` receives g_0 .. g_T: 2^g_t bounds ||X_t|| over the power of two that
// Scalars::shift takes out of X_0 (the product of the steps' |B|, which is 2^-h
// kappa ||X_0'|| at the start, kappa < 2 in the first step's).
bool split_fits(const std::vector<double> &coeffs, int iters, std::vector<int32_t> *growth = nullptr) {
  constexpr double kMaxX = 3.5, kMaxB = 58.0;
  double u = 1.0, grown = 0.0, linear = 1.0;
  if (growth) growth->assign(1, 0);
  for (int t = 0; t < iters; ++t) {
    const double a = coeffs[3 * t], b = coeffs[3 * t + 1], c = coeffs[3 * t + 2];
    auto g = [&](double z) { return std::fabs(a + z * (b + z * c)); };   // |p(x) / x|, z = x^2
    const double z1 = u * u;
    double gmax = std::max(g(0.0), g(z1));
    if (c != 0.0 && -b / (2 * c) > 0.0 && -b / (2 * c) < z1) gmax = std::max(gmax, g(-b / (2 * c)));
    gmax *= t == 0 ? 2.0 : 1.0;
    if (gmax > kMaxB) return false;
    linear *= std::fabs(a);
    if (!(linear >= 0.5)) return false;
    grown += std::log2(std::max(gmax, 1e-300));
    if (growth) growth->push_back(int32_t(std::ceil(grown)));
    // extrema of p on [0, u]: a + 3 b z + 5 c z^2 = 0
    double pmax = u * g(z1);
    const double disc = 9 * b * b - 20 * a * c;
    if (c == 0.0) {
      if (b != 0.0 && -a / (3 * b) > 0.0 && -a / (3 * b) < z1) pmax = std::max(pmax, std::sqrt(-a / (3 * b)) * g(-a / (3 * b)));
    } else if (disc >= 0.0) {
      for (double r : {-3 * b + std::sqrt(disc), -3 * b - std::sqrt(disc)}) {
        const double z = r / (10 * c);
        if (z > 0.0 && z < z1) pmax = std::max(pmax, std::sqrt(z) * g(z));
      }
    }
    u = pmax * 1.001;                  // rounding of the iterate
    if (!(u <= kMaxX)) return false;
  }
  return true;
}

}  // namespace

double Plan::product_flops(Op op) const {
  double f = 0.0;
  for (const MatDesc &d : mats) {
    const double P = d.P, Q = d.Q;
    if (op == Op::Poly) f += 2.0 * P * P * P;
    else if (op == Op::Gram || op == Op::Update || op == Op::Last) f += 2.0 * P * P * Q;
  }
  return f;
}

size_t Plan::dyn_bytes() const { return off_call + sizeof(CallParams) - off_dyn; }

void build_plan(Plan &p) {
  if (p.n < 0) throw std::invalid_argument("n must be >= 0");
  if (p.dtype != SLORR_F32 && p.dtype != SLORR_BF16) throw std::domain_error("unsupported dtype");
  if (p.kind != SLORR_HOYER && p.kind != SLORR_NUCLEAR) throw std::domain_error("unsupported kind");
  if (p.iters < 1 || p.iters > 1000) throw std::invalid_argument("iters must be in [1, 1000]");
  if (p.degree != 3 && p.degree != 5) throw std::domain_error("degree must be 3 or 5");
  if (!(p.ell > 0.0 && p.ell < 1.0)) throw std::invalid_argument("ell must be in (0, 1)");
  if (!(p.eps >= 0.0f) || !std::isfinite(p.eps)) throw std::invalid_argument("eps must be finite and >= 0");
  if (p.flags & ~uint32_t(SLORR_ACCUMULATE | SLORR_VALUES_ONLY | SLORR_NO_GRAPH | SLORR_AUX |
                          SLORR_DEFER_GRAD))
    throw std::invalid_argument("unknown flag bits");
  if ((p.flags & SLORR_VALUES_ONLY) && (p.flags & SLORR_DEFER_GRAD))
    throw std::invalid_argument("SLORR_VALUES_ONLY and SLORR_DEFER_GRAD exclude each other");
  if (p.grad_dtype != SLORR_F32 && p.grad_dtype != SLORR_BF16)
    throw std::domain_error("unsupported gradient dtype");
  if (!(p.safety >= 0.0 && p.safety < 1.0)) throw std::invalid_argument("safety must be in [0, 1)");
  if (p.coeffs.empty()) {
    // the built-in schedule, stabilised: every step but the last evaluates its
    // polynomial at x / (1 + safety), i.e. (a / s, b / s^3, c / s^5), so that a
    // singular value the iterate's rounding pushes slightly past the step's
    // interval stays inside the next one (explicit tables are used as given)
    p.coeffs.resize(size_t(p.iters) * 3);
    greedy_schedule(p.ell, p.degree, p.iters, p.coeffs.data());
    const double s = 1.0 + p.safety;
    for (int t = 0; t + 1 < p.iters; ++t) {
      p.coeffs[3 * t] /= s;
      p.coeffs[3 * t + 1] /= s * s * s;
      p.coeffs[3 * t + 2] /= s * s * s * s * s;
    }
  }
  if (p.coeffs.size() != size_t(p.iters) * 3) throw std::invalid_argument("coefficient table size");
  for (double c : p.coeffs)
    if (!std::isfinite(c)) throw std::invalid_argument("non-finite coefficient");

  const bool f16 = p.dtype == SLORR_BF16;
  // Gradients rounded to bf16 keep the fp32 MFMA kernels: both forms are off
  // by the same 1.7e-3 there (bf16's own rounding), but their fp32 gradients
  // differ by 5e-6, which moves 1 gradient in 700 to the next bf16 number
  // (2e-4 of the gradient, 40 times the forms' difference), and such sets'
  // results stay bit for bit.
  std::vector<int32_t> growth;
  p.split = p.dtype == SLORR_F32 && p.grad_dtype == SLORR_F32 && split_fits(p.coeffs, p.iters, &growth);
  p.growth.clear();
  if (p.split && p.eps > 0.0f) p.growth = growth;
  const bool scaled = f16 || p.split;      // 16-bit MFMA operands
  const float sx = scaled ? kScaleX16 : 1.0f, sa = scaled ? kScaleA16 : 1.0f, sb = scaled ? kScaleB16 : 1.0f;
  bool any_quintic = false;
  for (int t = 0; t < p.iters; ++t) any_quintic |= p.coeffs[3 * t + 2] != 0.0;

  // canonical shapes, groups
  p.mats.assign(p.n, MatDesc{});
  std::map<std::pair<int32_t, int32_t>, int> groups;
  p.paper_flops = p.mfma_flops = p.weight_bytes = 0;
  for (int i = 0; i < p.n; ++i) {
    const int64_t r = p.shapes[i].rows, c = p.shapes[i].cols;
    if (r < 0 || c < 0) throw std::invalid_argument("negative matrix dimension");
    MatDesc &d = p.mats[i];
    d.rows = int32_t(r);
    d.cols = int32_t(c);
    d.empty = (r == 0 || c == 0);
    if (d.empty) continue;
    const int64_t P = std::min(r, c), Q = std::max(r, c);
    if (P > kMaxShort || Q > kMaxLong) throw std::domain_error("matrix dimension beyond the limits");
    d.tall = r > c;
    d.P = int32_t(P);
    d.Q = int32_t(Q);
    d.Pp = round_up(d.P, kTile);
    d.Qp = round_up(d.Q, kTile);
    if (r * c > kMaxElems || int64_t(d.Pp) * d.Qp > kMaxElems)
      throw std::domain_error("matrix has more than 2^31 - 1 elements");
    if (int64_t(d.Pp) * d.Qp * int64_t(p.iter_bytes()) >= kMaxIterBytes)
      throw std::domain_error("matrix of 2 GiB or more in the iterate type (padded canonical shape)");
    groups[{d.P, d.Q}]++;
    p.paper_flops += p.iters * (4.0 * P * P * Q + 2.0 * P * P * P);
    p.weight_bytes += double(r) * c * p.elem_bytes();
  }
  p.groups = int32_t(groups.size());
  const int T = p.iters;

  std::vector<int> order;                 // non-empty matrices
  for (int i = 0; i < p.n; ++i)
    if (!p.mats[i].empty) order.push_back(i);
  auto tsize = [](int cfg) { return cfg == kCfg128 ? kTile : kBigTile; };
  p.tiles.clear();
  size_t entries = 64;                    // about what the lists below hold together
  for (int i : order) {
    const size_t nm = size_t(p.mats[i].Pp / kTile), nn = size_t(p.mats[i].Qp / kTile);
    entries += 6 * nm * nn + 4 * nm * (nm + 1);
  }
  p.tiles.reserve(entries);

  // XCD-aware order. Workgroup b of a launch runs on XCD b % kXcds, so list
  // entry b is taken from XCD (b % kXcds)'s own sequence: every matrix's tiles
  // stay on one XCD (its operand panels are fetched into one L2), matrices are
  // spread over the XCDs by longest-processing-time on their MFMA work, and
  // each XCD runs its longest tiles first. Short sequences are padded with
  // empty tiles (mat = -1), which exit at once.
  struct Job {
    int mat;
    double cost;                 // per tile (proportional to its k extent)
    std::vector<Tile> tiles;
  };
  auto emit = [&](std::vector<Job> whole) {
    TileRange r;
    r.first = int32_t(p.tiles.size());
    if (whole.empty()) return r;
    // a set of few large matrices would leave XCDs idle: cut every matrix into
    // jobs of at most 1/16 of the launch's tiles (contiguous runs of its tile order)
    size_t total = 0;
    for (const Job &j : whole) total += j.tiles.size();
    const size_t cap = std::max<size_t>(1, (total + 2 * kXcds - 1) / (2 * kXcds));
    std::vector<Job> jobs;
    for (Job &j : whole) {
      for (size_t b = 0; b < j.tiles.size(); b += cap) {
        Job part{j.mat, j.cost, {}};
        part.tiles.assign(j.tiles.begin() + b, j.tiles.begin() + std::min(j.tiles.size(), b + cap));
        jobs.push_back(std::move(part));
      }
    }
    std::stable_sort(jobs.begin(), jobs.end(), [](const Job &a, const Job &b) {
      return a.cost * a.tiles.size() > b.cost * b.tiles.size();
    });
    std::vector<std::vector<const Job *>> bins(kXcds);
    std::vector<double> load(kXcds, 0.0);
    for (const Job &j : jobs) {
      const int x = int(std::min_element(load.begin(), load.end()) - load.begin());
      bins[x].push_back(&j);
      load[x] += j.cost * j.tiles.size();
    }
    std::vector<std::vector<Tile>> seq(kXcds);
    size_t longest = 0;
    for (int x = 0; x < kXcds; ++x) {
      std::stable_sort(bins[x].begin(), bins[x].end(),
                       [](const Job *a, const Job *b) { return a->cost > b->cost; });
      for (const Job *j : bins[x]) seq[x].insert(seq[x].end(), j->tiles.begin(), j->tiles.end());
      longest = std::max(longest, seq[x].size());
    }
    for (size_t i = 0; i < longest; ++i)
      for (int x = 0; x < kXcds; ++x)
        p.tiles.push_back(i < seq[x].size() ? seq[x][i] : make_tile(-1, 0, 0, 0));
    r.count = int32_t(p.tiles.size()) - r.first;
    return r;
  };

  // Symmetric-output products of the Gram and poly launches: upper-
  // triangle tiles only; the kernel also stores the transpose of off-diagonal
  // tiles. `prods` lists the products of one launch as (matrix, k extent);
  // the 256-tile is used for every product of the launch when all of them
  // allow it and the launch has at least `min_big` such tiles (it halves the
  // operand traffic per flop of the 128-tile but gives 4x fewer blocks).
  struct Prod {
    int mat;
    int32_t k;
  };
  auto sym_list = [&](const std::vector<Prod> &prods, int64_t min_big, TileRange *out) {
    int64_t big = 0;
    bool all_big = !prods.empty();
    for (const Prod &q : prods) {
      const int nb = p.mats[q.mat].Pp / kBigTile;
      all_big &= p.mats[q.mat].Pp % kBigTile == 0;
      big += int64_t(nb) * (nb + 1) / 2;
    }
    const int cfg = (all_big && big >= min_big) ? kCfg256 : kCfg128;
    std::vector<Job> jobs;
    for (const Prod &q : prods) {
      Job j{q.mat, double(q.k), {}};
      const int nt = p.mats[q.mat].Pp / tsize(cfg);
      for (int tm = 0; tm < nt; ++tm)
        for (int tn = tm; tn < nt; ++tn) {
          j.tiles.push_back(make_tile(q.mat, tm, tn, 0));
        }
      jobs.push_back(std::move(j));
    }
    for (int c = 0; c < kNumCfg; ++c) out[c] = TileRange{};
    out[cfg] = emit(std::move(jobs));
  };
  // A = X X^T: long k ranges (K = Qp), so the 256-tile pays as soon as the set
  // has one upper-triangle 256-tile per CU. The P x P products (K = Pp, the
  // shortest) take it only with two per CU.
  {
    std::vector<Prod> g0, pl;
    for (int i : order) {
      const MatDesc &d = p.mats[i];
      g0.push_back({i, d.Qp});
      pl.push_back({i, d.Pp});
    }
    sym_list(g0, kCus, p.gram);
    sym_list(pl, kMinBigTiles, p.pp);
  }
  // Split-K Gram. A set with few Gram tiles (small P) but long K = Qp would
  // leave most CUs idle: every tile's k range is cut into parts (multiples of
  // kTile) so that the launch has about kMinGramUnits blocks; each part writes
  // an fp32 partial tile, and a reduce launch adds the parts in order.
  p.gsplit = TileRange{};
  p.gred = TileRange{};
  p.gram_parts = 0;
  // The parts and the reduce launch cost more than they save unless the
  // tiles are long: only sets whose longest Gram tile has enough k-slabs of
  // the kernel (64 fp16 / 32 fp32 values of k) are split, into parts of a
  // minimum number of slabs.
  const int slab_k = f16 ? 64 : 32;
  const int kMinSplitSlabs = f16 ? kMinSplitSlabs16 : kMinSplitSlabs32;
  const int kMinPartSlabs = f16 ? kMinPartSlabs16 : kMinPartSlabs32;
  int max_slabs = 0;
  for (int i : order) max_slabs = std::max(max_slabs, p.mats[i].Qp / slab_k);
  if (p.gram[kCfg256].count == 0 && max_slabs >= kMinSplitSlabs) {
    int64_t ntiles = 0;
    for (int i : order) ntiles += int64_t(p.mats[i].Pp / kTile) * (p.mats[i].Pp / kTile + 1) / 2;
    if (ntiles > 0 && ntiles < kMinGramUnits) {
      const int want = int(std::max<int64_t>(1, std::min<int64_t>(kMaxGramParts, kMinGramUnits / ntiles)));
      const int per_min = std::max(1, kMinPartSlabs * slab_k / kTile);   // k blocks of kTile per part
      std::vector<Job> jobs;
      std::vector<Tile> reds;
      for (int i : order) {
        const MatDesc &d = p.mats[i];
        const int nblk = d.Qp / kTile;                     // k blocks of kTile
        const int per = std::max(per_min, (nblk + std::min(want, nblk) - 1) / std::min(want, nblk));
        const int parts = (nblk + per - 1) / per;
        Job j{i, double(per * kTile), {}};
        const int nt = d.Pp / kTile;
        for (int tm = 0; tm < nt; ++tm)
          for (int tn = tm; tn < nt; ++tn) {
            Tile r = make_tile(i, tm, tn, p.gram_parts);
            r.parts = parts;
            reds.push_back(r);
            for (int q = 0; q < parts; ++q) {
              Tile t = make_tile(i, tm, tn, p.gram_parts++);
              t.k0 = q * per * kTile;
              t.k1 = std::min(nblk, (q + 1) * per) * kTile;
              j.tiles.push_back(t);
            }
          }
        jobs.push_back(std::move(j));
      }
      p.gsplit = emit(std::move(jobs));
      p.gred.first = int32_t(p.tiles.size());
      p.tiles.insert(p.tiles.end(), reds.begin(), reds.end());
      p.gred.count = int32_t(reds.size());
    }
  }
  // Symmetric outputs of few tiles on 16-bit operands run as 64-tiles, up to
  // two per CU: a tile's k range is serial work on one CU, a quarter of it on a
  // 64-tile, whose fetches (twice the bytes per product) such launches have
  // room for. Per call, 128-tiles -> P x P products -> Gram on 64-tiles too:
  // ResNet-18 in fp32 (61 tiles, 211 64-tiles; its Gram is split) 711 -> 656 us,
  // ViT-Ti (144, 480) 228 -> 213 -> 203. With up to four per CU: ViT-S (288, 1008)
  // 487 -> 501 -> 512.
  // And only while the longest XCD's queue (a matrix's tiles stay together, so
  // queues are uneven) ends soon after its longest tile: a second round costs more
  // than the quarter saves. At a span of at most 1.2 times the longest tile (a
  // tile takes about as long to start and end as 500 values of k) all of 324
  // lists of random sets gained, 1 to 13 % of a call; between 1.4 and 1.6 one of
  // 6 lost; from 1.6 all but one of 44 lost, up to 14 % (bf16: 51 matrices of 256
  // x 768, 70 tiles in a queue, 271 -> 310 us; 9 of 640 x 1920 432 -> 536).
  p.gram64 = p.pp64 = TileRange{};
  if (scaled && !p.lean) {
    int64_t tiles = 0;
    std::vector<Job> jobs;
    for (int i : order) {
      Job j{i, double(p.mats[i].Pp), {}};
      const int nt = p.mats[i].Pp / kSmallTile;
      tiles += int64_t(nt) * (nt + 1) / 2;
      if (tiles > kMaxSmallTiles) break;
      for (int tm = 0; tm < nt; ++tm)
        for (int tn = tm; tn < nt; ++tn) j.tiles.push_back(make_tile(i, tm, tn, 0));
      jobs.push_back(std::move(j));
    }
    auto emit64 = [&]() {                       // costs per matrix as set in jobs
      const TileRange r = emit(jobs);
      std::vector<double> cost(size_t(p.n), 0.0);
      for (const Job &j : jobs) cost[size_t(j.mat)] = j.cost + kSmallTileFixed;
      double span = 0.0, longest = 0.0;
      for (int x = 0; x < kXcds; ++x) {
        // when each of the blocks that the XCD holds ends, the first on top
        std::priority_queue<double, std::vector<double>, std::greater<double>> end(
            std::greater<double>(), std::vector<double>(2 * kCus / kXcds, 0.0));
        for (int e = x; e < r.count; e += kXcds) {
          const Tile &t = p.tiles[size_t(r.first) + e];
          if (t.mat < 0) continue;
          const double at = end.top() + cost[size_t(t.mat)];
          end.pop();
          end.push(at);
          span = std::max(span, at);
          longest = std::max(longest, cost[size_t(t.mat)]);
        }
      }
      if (span <= kMaxQueueSpan * longest) return r;
      p.tiles.resize(size_t(r.first));
      return TileRange{};
    };
    if (tiles <= kMaxSmallTiles) {
      p.pp64 = emit64();
      if (!p.gsplit.count && p.gram[kCfg128].count) {
        for (Job &j : jobs) j.cost = p.mats[j.mat].Qp;
        p.gram64 = emit64();
      }
    }
  }
  // Update launches: X' = B X (P x Q, full output). The tiles of the last
  // update own one trace slot each, contiguous per matrix (the same list
  // serves every step). The tiles of one matrix form one job, dispatched
  // column panel by column panel: the Pp / ts tiles that read one panel of X
  // run together on one XCD, so the panel is fetched into its L2 once. The
  // 256-tile needs 256-aligned padded dims and is used when the launch has at
  // least two such tiles per CU; fp32 sets use the 128-tile (the fp32 256-tile
  // update with the trace epilogue does not fit the register file).
  int32_t slot = 0;
  {
    int64_t big = 0;
    bool all_big = !order.empty() && f16;
    for (int i : order) {
      const MatDesc &d = p.mats[i];
      all_big &= d.Pp % kBigTile == 0 && d.Qp % kBigTile == 0;
      big += int64_t(d.Pp / kBigTile) * (d.Qp / kBigTile);
    }
    const int cfg = (all_big && big >= kMinBigTiles) ? kCfg256 : kCfg128;
    const int ts = tsize(cfg);
    std::vector<Job> jobs;
    for (int i : order) {
      MatDesc &d = p.mats[i];
      Job j{i, double(d.Pp), {}};
      d.trace_begin = slot;
      for (int tn = 0; tn < d.Qp / ts; ++tn)
        for (int tm = 0; tm < d.Pp / ts; ++tm) j.tiles.push_back(make_tile(i, tm, tn, slot++));
      d.trace_end = slot;
      jobs.push_back(std::move(j));
    }
    for (int c = 0; c < kNumCfg; ++c) p.pq[c] = TileRange{};
    p.pq[cfg] = emit(std::move(jobs));
    // The 128-tile list again as 256-tiles for the persistent update kernel
    // (split sets, and fp16 sets whose padded dims are not all multiples of
    // 256: their tiles at the right and lower edge cover half a tile's work).
    // Each 256-tile names the trace slot of its first 128-tile (a column of
    // 128-tiles has Pp / 128 slots). As for whole tiles, from two per CU;
    // and while the edge tiles' empty part stays below kMaxEdgeWaste of the
    // work: the 256-tile kernel runs at about 1.3 times the 128-tile's rate
    // (1280 x 3456 bf16 sets: 1045 against 795 TFLOP/s). Split tables with a
    // cubic step stay on 128-tiles (the 256-tile's a X term does not fit the
    // registers next to the split trace).
    p.upd = TileRange{};
    bool run_big = (p.split || f16) && cfg == kCfg128 && !order.empty();
    for (int t = 0; p.split && t < T; ++t) run_big &= p.coeffs[3 * t + 2] != 0.0;
    int64_t nrun = 0;
    double work = 0.0, run_work = 0.0;
    for (int i : order) {
      const MatDesc &d = p.mats[i];
      const int64_t tiles = int64_t((d.Pp + kTile) / kBigTile) * ((d.Qp + kTile) / kBigTile);
      nrun += tiles;
      run_work += double(tiles) * kBigTile * kBigTile * d.Pp;
      work += double(d.Pp) * d.Qp * d.Pp;
    }
    if (run_big && nrun >= kMinBigTiles && run_work <= kMaxEdgeWaste * work) {
      jobs.clear();
      for (int i : order) {
        const MatDesc &d = p.mats[i];
        Job j{i, double(d.Pp), {}};
        const int col = d.Pp / kTile;                       // slots per column
        for (int tn = 0; tn * kBigTile < d.Qp; ++tn)
          for (int tm = 0; tm * kBigTile < d.Pp; ++tm) {
            j.tiles.push_back(make_tile(i, tm, tn, d.trace_begin + 2 * tn * col + 2 * tm));
          }
        jobs.push_back(std::move(j));
      }
      p.upd = emit(std::move(jobs));
    }
  }
  p.trace_slots = slot;

  // Sets of short matrices run one launch per step (k_short): every matrix has
  // one tile of rows and at most kMaxShortSlices of columns, every step is
  // quintic, and a step reads at most kMaxShortReads Gram partials (each block
  // all of its matrix's): beyond, the reads and the poly product that every
  // block forms cost more than the launches they save. Per call, launch per
  // product -> per step, at partials read, T = 6:
  //   fp32  384 (24 of 128 x 512) 259 -> 137 us    1600 (100 of them) 426 -> 313
  //         1920 (30 of 128 x 1024) 317 -> 312     16384 (256 of them) 974 -> 1907
  //   bf16  384: 163 -> 87    1600: 193 -> 188     4096 (256 of 128 x 512) 298 -> 335
  // Their partials lie behind the matrices; a set that fits the static scratch
  // of the no-allocation entry without them and not with them goes step by
  // step.
  p.short_set = scaled && !order.empty();
  int64_t reads = 0;
  for (int i : order) {
    const int64_t slices = p.mats[i].Qp / kTile;
    p.short_set &= p.mats[i].Pp == kTile && slices <= kMaxShortSlices;
    reads += slices * slices;
  }
  p.short_set &= reads <= kMaxShortReads;
  for (int t = 0; t < T; ++t) p.short_set &= p.coeffs[3 * t + 2] != 0.0;

  // canonical 64 x 64 tiles: the norm (one partial slot each, contiguous per
  // matrix in canonical row-major tile order, which is the order they are
  // summed in), the normalisation and the gradient; element runs of the
  // original layout for the decoupled update. The list walks each matrix along
  // W's own rows (tall W: down the canonical columns), so that the 4 waves of
  // a block read adjacent 128-byte pieces of the same rows of W.
  p.chunks.clear();
  p.prep.first = int32_t(p.tiles.size());
  int32_t nslot = 0;
  for (int i = 0; i < p.n; ++i) {
    MatDesc &d = p.mats[i];
    if (d.empty) continue;
    d.norm_begin = nslot;
    const int ntm = d.Pp / kPrepTile, ntn = d.Qp / kPrepTile;
    if (d.tall) {
      for (int tn = 0; tn < ntn; ++tn)
        for (int tm = 0; tm < ntm; ++tm) p.tiles.push_back(make_tile(i, tm, tn, nslot + tm * ntn + tn));
    } else {
      for (int tm = 0; tm < ntm; ++tm)
        for (int tn = 0; tn < ntn; ++tn) p.tiles.push_back(make_tile(i, tm, tn, nslot + tm * ntn + tn));
    }
    nslot += ntm * ntn;
    d.norm_end = nslot;
    const int64_t total = int64_t(d.rows) * d.cols;
    for (int64_t b = 0; b < total; b += kChunk)
      p.chunks.push_back({i, int32_t(b), int32_t(std::min<int64_t>(kChunk, total - b)), 0});
  }
  p.prep.count = int32_t(p.tiles.size()) - p.prep.first;
  p.norm_slots = nslot;

  // workspace layout
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + std::max<size_t>(bytes, 1));
    return o;
  };
  p.off_mats = take(sizeof(MatDesc) * p.n);
  p.off_dyn = take(sizeof(DynDesc) * p.n);
  off = p.off_dyn + sizeof(DynDesc) * p.n;          // call params follow the dyn table
  p.off_call = take(sizeof(CallParams));
  p.off_tiles = take(sizeof(Tile) * p.tiles.size());
  p.off_chunks = take(sizeof(Chunk) * p.chunks.size());
  p.off_scal = take(sizeof(Scalars) * p.n);
  p.off_sumsq = take(sizeof(double) * size_t(p.norm_slots));
  p.off_trace = take(sizeof(double) * p.trace_slots);
  p.off_gpart = take(sizeof(float) * size_t(kTile) * kTile * size_t(p.gram_parts));
  p.off_static_end = off;
  const size_t es = p.iter_bytes();
  for (int i = 0; i < p.n; ++i) {
    MatDesc &d = p.mats[i];
    if (d.empty) continue;
    const size_t pq = size_t(d.Pp) * d.Qp * es, pp = size_t(d.Pp) * d.Pp * es;
    d.x[0] = take(pq);
    d.x[1] = take(pq);
    d.x[2] = take(pq);
    d.a = take(pp);
    d.b = any_quintic ? take(pp) : d.a;
    d.xt = d.x[xbuf(T)];                      // step t reads x[xbuf(t)], writes x[xbuf(t + 1)]
  }
  p.off_short = off;
  if (p.short_set) {
    const size_t with = off + align256(2 * sizeof(float) * size_t(kTile) * kTile * size_t(p.trace_slots));
    if (off <= size_t(SLORR_SCRATCH_BYTES) && with > size_t(SLORR_SCRATCH_BYTES)) p.short_set = false;
    else off = with;
  }
  p.ws_bytes = off;
  // a set that fits the static scratch without the 64-tile lists goes without
  // (p.off_short: the size without the partials of short matrices, which such a
  // set goes without too if need be)
  const size_t lists = sizeof(Tile) * size_t(p.gram64.count + p.pp64.count);
  if (lists && p.off_short > size_t(SLORR_SCRATCH_BYTES) && p.off_short - lists - 256 <= size_t(SLORR_SCRATCH_BYTES)) {
    p.lean = true;
    build_plan(p);                            // (with the table built above)
    return;
  }
  // host image of the table region, for the entry point that allocates nothing
  p.image.assign(p.off_scal, 0);
  if (p.n) std::memcpy(p.image.data() + p.off_mats, p.mats.data(), sizeof(MatDesc) * p.n);
  if (!p.tiles.empty()) std::memcpy(p.image.data() + p.off_tiles, p.tiles.data(), sizeof(Tile) * p.tiles.size());
  if (!p.chunks.empty()) std::memcpy(p.image.data() + p.off_chunks, p.chunks.data(), sizeof(Chunk) * p.chunks.size());
  p.spans.clear();
  p.spans.reserve(size_t(2) * p.n);

  // launch schedule
  p.launches.clear();
  auto plain = [](Op op, int32_t grid, int32_t first = 0) {
    Launch l{};
    l.op = op;
    l.grid = grid;
    l.tile_first = first;
    return l;
  };
  if (p.prep.count) p.launches.push_back(plain(Op::SumSq, p.prep.count, p.prep.first));
  if (p.n > 0) p.launches.push_back(plain(Op::NormFin, (p.n + kThreads / 64 - 1) / (kThreads / 64)));
  if (p.prep.count) p.launches.push_back(plain(Op::Prep, p.prep.count, p.prep.first));
  auto gemm = [&](Op op, const TileRange *r, Launch l) {
    for (int cfg = kNumCfg - 1; cfg >= 0; --cfg) {
      if (!r[cfg].count) continue;
      l.op = op;
      l.grid = r[cfg].count;
      l.tile_first = r[cfg].first;
      l.cfg = cfg;
      l.run_cfg = cfg;
      l.run_first = l.tile_first;
      l.run_grid = l.grid;
      const TileRange &r64 = op == Op::Gram ? p.gram64 : p.pp64;
      if ((op == Op::Gram || op == Op::Poly) && r64.count) {
        l.run_cfg = kCfg64;
        l.run_first = r64.first;
        l.run_grid = r64.count;
      }
      if ((op == Op::Update || op == Op::Last) && p.upd.count) {
        l.run_cfg = kCfg256;
        l.run_first = p.upd.first;
        l.run_grid = p.upd.count;
      }
      p.launches.push_back(l);
    }
  };
  const float prod = float(1.0 / sb);           // (B_s X_s) / s_b keeps X's scale
  auto rescale = [&](Launch &l, int t) {
    if (p.growth.empty()) return;
    l.rescale = 1;
    l.grow0 = p.growth[size_t(t)];
    l.grow1 = p.growth[size_t(t) + 1];
  };
  for (int t = 0; t < T; ++t) {
    const double a = p.coeffs[3 * t], b = p.coeffs[3 * t + 1], c = p.coeffs[3 * t + 2];
    const int32_t xi = xbuf(t), xo = xbuf(t + 1);
    const bool quintic = c != 0.0;
    // the first step runs on X_0' = W / 2^e: its coefficients are scaled per
    // matrix by kappa, kappa^3, kappa^5 (kappa = 2^e / (f + eps), read by the
    // kernels), so that it computes p_1(X_0) with X_0 = kappa X_0'
    const int32_t kap = t == 0 ? 1 : 0;
    // A_s = s_a A with A = X X^T = (X_s X_s^T) / s_x^2
    Launch g{};
    g.xin = xi;
    g.alpha = float(sa / (double(sx) * sx));
    if (p.short_set) g.run = t == 0 ? kRunShort : kNothing;
    if (p.gsplit.count) {
      g.op = Op::Gram;
      g.grid = p.gsplit.count;
      g.tile_first = p.gsplit.first;
      g.cfg = g.run_cfg = kCfg128;
      g.run_first = g.tile_first;
      g.run_grid = g.grid;
      // one part per tile: the tiles are stored whole, the reduce launch would
      // copy (ViT-S in fp32, 288 tiles: 1136 -> 1096 us a call)
      const bool whole = p.gram_parts == p.gred.count;
      if (whole) {
        g.run_first = p.gram[kCfg128].first;
        g.run_grid = p.gram[kCfg128].count;
      }
      p.launches.push_back(g);                // fp32 partials
      Launch l = plain(Op::GramReduce, p.gred.count * kRedStripes, p.gred.first);
      l.alpha = g.alpha;
      if (p.short_set || whole) l.run = kNothing;
      p.launches.push_back(l);
    } else {
      gemm(Op::Gram, p.gram, g);
    }
    const Op op = (t == T - 1) ? Op::Last : Op::Update;
    if (quintic) {
      // B_s = s_b (b A + c A A + a I) = s_b (b A_s / s_a + c (A_s A_s) / s_a^2 + a I):
      // the step X' = a X + (b A + c A A) X becomes X' = B X (a_t I folded in)
      Launch l{};
      l.xin = xi;
      l.kap = kap;
      rescale(l, t);
      l.alpha = float(double(sb) * c / (double(sa) * sa));
      l.beta = float(double(sb) * b / sa);
      l.gamma = float(double(sb) * a);
      if (p.short_set) l.run = kNothing;
      gemm(Op::Poly, p.pp, l);
      // X'_s = (B_s X_s) / s_b
      Launch u{};
      u.xin = xi;
      u.xout = xo;
      u.fold = 1;
      u.alpha = prod;
      if (p.short_set) {
        u.run = kRunShort;
        u.gram_alpha = g.alpha;
        u.poly_alpha = l.alpha;
        u.poly_beta = l.beta;
        u.poly_gamma = l.gamma;
        u.poly_kap = kap;
        rescale(u, t);
      }
      gemm(op, p.pq, u);
    } else {
      // cubic step: X'_s = a X_s + b (A_s X_s) / s_a
      Launch u{};
      u.xin = xi;
      u.xout = xo;
      u.use_a = 1;
      u.kap = kap;
      rescale(u, t);
      u.alpha = float(b / sa);
      u.beta = float(a);
      gemm(op, p.pq, u);
    }
  }
  if (p.n > 0) p.launches.push_back(plain(Op::Finalize, p.n));
  // The gradient, once s1 and s2 are known, by the gradient kernel from the
  // stored X_T. A deferred gradient runs the same launch later, from the X_T
  // and the factors the forward left in the workspace. The set total (the
  // values added in index order) is written by the gradient launch's first
  // block when the call computes the gradient, else by a launch of its own.
  const bool grad_now = !(p.flags & (SLORR_VALUES_ONLY | SLORR_DEFER_GRAD)) && p.prep.count;
  if (!grad_now) p.launches.push_back(plain(Op::SetSum, 1));
  p.grad_launches.clear();
  if (!(p.flags & SLORR_VALUES_ONLY)) {
    const size_t first = p.launches.size();
    if (p.prep.count) p.launches.push_back(plain(Op::Grad, p.prep.count, p.prep.first));
    p.grad_launches.assign(p.launches.begin() + first, p.launches.end());
    if (p.flags & SLORR_DEFER_GRAD) p.launches.resize(first);
    else if (grad_now) p.launches.back().set_sum = 1;
  }

  // the kernel of each launch
  p.kernels.clear();
  for (const Launch &l : p.launches) {
    static const char *const simple[] = {"k_sumsq", "k_norm_fin", "k_prep", "", "", "", "",
                                         "k_finalize", "k_grad", "k_setsum", "k_gram_reduce"};
    const bool product = l.op == Op::Gram || l.op == Op::Poly || l.op == Op::Update || l.op == Op::Last;
    const char *mode = l.op == Op::Gram ? "gram" : l.op == Op::Poly ? "poly" : l.op == Op::Update ? "update" : "last";
    std::string name;
    if (l.run == kRunShort) {
      name = l.op == Op::Gram ? "k_short<first>" : l.op == Op::Update ? "k_short<step>" : "k_short<last>";
    } else if (l.run != kNothing && product) {
      const std::string edge = l.run_cfg == kCfg64 ? "64" : l.run_cfg == kCfg256 ? "256" : "128";
      if (scaled && l.run_cfg == kCfg256 && l.op != Op::Gram && l.op != Op::Poly) name = std::string("k_upd256<") + mode + ">";
      else name = std::string(scaled ? "k_tile<" : "k_gemm<") + mode + ", " + edge + "x" + edge + ">";
    } else if (l.run != kNothing) {
      name = simple[int(l.op)];
    }
    p.kernels.push_back(name);
  }

  // MFMA work of the schedule's products (padded, symmetric tiles counted once)
  p.mfma_flops = 0;
  for (const Launch &l : p.launches) {
    if (l.op != Op::Gram && l.op != Op::Poly && l.op != Op::Update && l.op != Op::Last) continue;
    const double ts = tsize(l.cfg);
    for (int k = 0; k < l.grid; ++k) {
      const Tile &tl = p.tiles[l.tile_first + k];
      if (tl.mat < 0) continue;
      const MatDesc &d = p.mats[tl.mat];
      double kk = double(d.Pp);
      if (l.op == Op::Gram) kk = tl.k1 > 0 ? double(tl.k1 - tl.k0) : double(d.Qp);
      p.mfma_flops += 2.0 * ts * ts * kk;
    }
  }
}

}  // namespace slorr
