// Host-only driver for the device's work list under AddressSanitizer / UndefinedBehaviorSanitizer: on seeded random operator lists,
// the list made for a launch must cover every output rectangle of the table once (parts that tile it, slices that tile the
// reduction, the same whatever the per-die lists), keep deadlines in order, give every rectangle with slices a workspace of its
// own, and name every LDS tile in the per-die lists once.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <map>
#include <random>
#include <string>
#include <tuple>
#include <vector>

#include "sk_internal.h"

static int fail(const char *what, int seed) {
  std::fprintf(stderr, "work_list_driver: %s (seed %d)\n", what, seed);
  return 1;
}

using Slices = std::vector<std::pair<uint32_t, uint32_t>>;  // k0, k_len

static Slices same(Slices a) {
  std::sort(a.begin(), a.end());
  a.erase(std::unique(a.begin(), a.end()), a.end());
  return a;
}

static std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> blocks(const std::vector<sk_tile> &work) {
  std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> out;
  for (const sk_tile &t : work)
    for (uint32_t m = t.m0 / 64; m <= (t.m0 + t.m_len - 1) / 64; ++m)
      for (uint32_t n = t.n0 / 32; n <= (t.n0 + t.n_len - 1) / 32; ++n) out[{t.problem, m, n}].emplace_back(t.k0, t.k_len);
  return out;
}

// The list against the table: 0, or a message.  `slices`: of every output column block of every operator.
static const char *check(const sk::HostPlan &hp, const sk::WorkList &w, std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> &slices) {
  std::vector<int64_t> count(hp.dev.size(), 0), area(hp.dev.size(), 0);
  std::vector<std::pair<int64_t, int64_t>> used;
  for (size_t i = 0; i < w.work.size(); ++i) {
    const sk_tile &t = w.work[i];
    const sk::DevProblem &d = hp.dev[t.problem];
    if (t.m_len < 1 || t.n_len < 1 || t.k_len < 1 || (int64_t)t.m0 + t.m_len > d.Mg || (int64_t)t.n0 + t.n_len > d.Ng ||
        (int64_t)t.k0 + t.k_len > d.Kg || t.ks_idx >= t.S || t.out_tile_id >= w.ws_off.size())
      return "record leaves its operator";
    ++count[t.problem];
    if (t.ks_idx != 0) {
      const sk_tile &b = w.work[i - 1];
      if (b.problem != t.problem || b.out_tile_id != t.out_tile_id || b.ks_idx + 1 != t.ks_idx || b.k0 + b.k_len != t.k0 || b.m0 != t.m0 ||
          b.n0 != t.n0 || b.m_len != t.m_len || b.n_len != t.n_len || b.S != t.S)
        return "slices that do not follow one another";
    } else {
      if (t.k0 != 0) return "the first slice starts late";
      area[t.problem] += (int64_t)t.m_len * t.n_len;
      if (t.S > 1) {
        const int64_t size = t.cls == sk::CLS_TILE_128x128 ? 4096 : t.cls == sk::CLS_TILE_128x64 ? 2048 : 512 << (t.cls / 3);
        used.emplace_back(w.ws_off[t.out_tile_id], w.ws_off[t.out_tile_id] + size * t.S);
        if (t.n_len > 128 || t.m_len > 128) return "slices of more than one block";
      }
    }
    if (t.ks_idx + 1 == t.S && (int64_t)t.k0 + t.k_len != d.Kg) return "the last slice ends early";
  }
  slices = blocks(w.work);
  if (count != w.count) return "records per operator";
  for (size_t i = 0; i < hp.dev.size(); ++i)
    if (area[i] != (int64_t)hp.dev[i].Mg * hp.dev[i].Ng) return "outputs missing or made twice";
  std::sort(used.begin(), used.end());
  for (size_t i = 0; i < used.size(); ++i)
    if (used[i].second > w.ws_f32x4 || (i && used[i].first < used[i - 1].second)) return "workspaces overlap";
  if (hp.xorder.empty()) return w.xorder.empty() ? nullptr : "lists of a plan without";
  std::vector<int> named(w.work.size(), 0);
  for (uint32_t e : w.xorder) {
    if (e >= w.work.size()) return "an entry of a list names no record";
    ++named[e];
  }
  for (size_t i = 0; i < w.work.size(); ++i)
    if (named[i] != (w.work[i].cls >= sk::CLS_TILE_128x128 ? 1 : 0)) return "an LDS tile that no list, or more than one, names";
  return w.xoff[8] == w.xorder.size() ? nullptr : "offsets of the lists";
}

int main() {
  int cut = 0, sliced = 0, moved = 0;
  for (int seed = 0; seed < 400; ++seed) {
    std::mt19937 g(seed);
    auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + g() % v.size()); };
    const int n = 1 + (int)(g() % 30);
    std::vector<sk_problem> ps((size_t)n);
    uintptr_t addr = 0x10000000;
    for (sk_problem &p : ps) {
      p = sk_problem{};
      p.dtype = pick({SK_F32, SK_BF16, SK_F16});
      if (g() % 2) {
        p.op = SK_GEMM, p.M = pick({1, 16, 33, 64, 65, 129, 300}), p.N = pick({5, 64, 129, 500, 4100}), p.K = pick({40, 64, 129, 1001, 4096, 9001});
      } else {
        p.op = g() % 2 ? SK_CONV2D_NHWC : SK_CONV2D_NCHW, p.Nb = pick({1, 3}), p.H = p.Wd = pick({7, 14, 30}), p.Cin = pick({3, 9, 64, 256});
        p.Cout = pick({20, 64, 200}), p.R = p.S = pick({1, 3}), p.pad_h = p.pad_w = p.R / 2, p.stride = pick({1, 2});
      }
      p.deadline_ms = pick({0, 0, 0, 1, 2});
      p.A = (const void *)addr, p.B = (const void *)(addr + (1u << 28)), p.C = (void *)(addr + (2u << 28));
      addr += (uintptr_t)3 << 28;
    }
    sk_plan_params prm;
    sk_plan_params_default(&prm);
    prm.host_only = 1;
    prm.edf = g() % 4 != 0;
    prm.tail_div = g() % 4 ? 384 : 0;
    prm.tile_bytes_min = pick({4096, 32768});
    const int64_t wgs = pick({1, 60, 512, 512});
    std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> plain;
    for (int part : {0, 4}) {
      prm.xcd_part = part;
      sk::HostPlan hp;
      std::string err;
      if (sk::plan_host(ps.data(), n, &prm, hp, err) != SK_OK) return fail(err.c_str(), seed);
      sk::WorkList w;
      if (!sk::device_list(hp, wgs, false, w)) {  // the table itself
        w.work = hp.tiles, w.count = hp.count, w.ws_off = hp.ws_off, w.ws_f32x4 = hp.ws_f32x4, w.xorder = hp.xorder;
        std::copy(std::begin(hp.xoff), std::end(hp.xoff), std::begin(w.xoff));
      } else if (part == 0) {
        ++cut;
      }
      std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> slices;
      if (const char *what = check(hp, w, slices)) return fail(what, seed);
      size_t before = 0;
      for (size_t i = 1; i < w.work.size(); ++i) {
        const uint32_t a = w.work[i - 1].problem, b = w.work[i].problem;
        if (a == b) continue;
        if (++before >= hp.dev.size()) return fail("an operator's records are not together", seed);
        auto key = [&](uint32_t p) { return ps[p].deadline_ms > 0 ? ps[p].deadline_ms : INFINITY; };
        if (prm.edf ? key(a) > key(b) : a > b) return fail("deadlines out of order", seed);
        if (a > b && key(a) == key(b)) ++moved;
      }
      if (prm.tail_div == 0)
        for (const sk_tile &t : w.work)
          if (t.S != hp.tiles[(size_t)hp.first[t.problem]].S) return fail("slices without the tail rule", seed);
      // slices that only the list makes: all but the last of twelve stages at least (blocks of any alignment eight), and equal
      for (const sk_tile &t : w.work) {
        const sk::DevProblem &d = hp.dev[t.problem];
        if (t.S == hp.tiles[(size_t)hp.first[t.problem]].S || t.ks_idx + 1 == t.S) continue;
        const int64_t stages = t.k_len / (128 / sk::elem_size(d.dtype));
        if (stages < ((d.flags & 3) == 3 ? 12 : 8) || stages % 4 != 0 || t.k0 != (uint64_t)t.ks_idx * t.k_len) return fail("a short slice", seed);
      }
      // the slices are those of a launch that fills the chip, whatever the grid; without new ones they are the table's
      for (int64_t other : {(int64_t)512, (int64_t)33}) {
        sk::WorkList o;
        if (!sk::device_list(hp, other, false, o)) o.work = hp.tiles;
        std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> got;
        if (const char *what = o.count.empty() ? nullptr : check(hp, o, got)) return fail(what, seed);
        if (o.count.empty()) got = blocks(o.work);
        if (got.size() != slices.size()) return fail("blocks on another grid", seed);
        for (const auto &s : slices)
          if (same(got[s.first]) != same(s.second)) return fail("the grid changes the slices", seed);
      }
      sk::WorkList whole;
      if (sk::device_list(hp, wgs, false, whole, false)) {
        std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> ignored;
        if (const char *what = check(hp, whole, ignored)) return fail(what, seed);
        for (const sk_tile &t : whole.work)
          if (t.S != hp.tiles[(size_t)hp.first[t.problem]].S) return fail("slices of a list without", seed);
      }
      if (part == 0) {
        plain = slices;
        for (const sk_tile &t : w.work) sliced += t.S != hp.tiles[(size_t)hp.first[t.problem]].S;
        // the baseline: an operator by itself gets the slices of a plan of that operator
        sk::HostPlan alone;
        if (sk::plan_host_each_alone(hp, wgs, alone, err) != SK_OK) return fail("plan_host_each_alone", seed);
        (void)sk::balance_each_alone(alone, wgs);
        for (int i = 0; i < n; ++i) {
          sk::HostPlan one;
          sk::WorkList o;
          if (sk::plan_host(&ps[(size_t)i], 1, &prm, one, err) != SK_OK) return fail("plan_host", seed);
          const std::vector<sk_tile> &want = sk::device_list(one, wgs, false, o) ? o.work : one.tiles;
          if (o.window) continue;  // (runs of pixels sum in the same order; the baseline keeps the tiles)
          if ((int64_t)want.size() != alone.count[(size_t)i]) return fail("records of an operator alone", seed);
          for (size_t k = 0; k < want.size(); ++k) {
            const sk_tile &a = want[k], &b = alone.tiles[(size_t)alone.first[(size_t)i] + k];
            if (b.problem != (uint32_t)i || a.m0 != b.m0 || a.n0 != b.n0 || a.m_len != b.m_len || a.n_len != b.n_len || a.k0 != b.k0 ||
                a.k_len != b.k_len || a.S != b.S || a.ks_idx != b.ks_idx)
              return fail("a record of an operator alone", seed);
          }
        }
        sk::WorkList all;
        all.work = alone.tiles, all.count = alone.count, all.ws_off = alone.ws_off, all.ws_f32x4 = alone.ws_f32x4;
        std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> ignored;
        if (const char *what = check(hp, all, ignored)) return fail(what, seed);
      } else {
        for (const auto &s : slices) {
          if (same(s.second) != same(plain[s.first])) return fail("the per-die lists change the slices", seed);
        }
      }
    }
  }
  // Runs of pixels: every output of every operator in one record, in order, cut at blocks of 128; and what does not go there.
  for (int seed = 0; seed < 200; ++seed) {
    std::mt19937 g(seed);
    auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + g() % v.size()); };
    std::vector<sk_problem> ps((size_t)(1 + g() % 40));
    uintptr_t addr = 0x10000000;
    const int dt = pick({SK_BF16, SK_F16});
    for (sk_problem &p : ps) {
      p = sk_problem{};
      p.op = SK_CONV2D_NHWC, p.dtype = dt, p.Nb = pick({1, 1, 2, 400}), p.H = pick({9, 20, 56, 300}), p.Wd = pick({9, 56, 63}), p.Cin = 64;
      p.Cout = pick({8, 40, 64}), p.R = p.S = 3, p.pad_h = p.pad_w = 1;
      p.A = (const void *)addr, p.B = (const void *)(addr + (1u << 30)), p.C = (void *)(addr + (2u << 30));
      addr += (uintptr_t)3 << 30;
    }
    sk_plan_params prm;
    sk_plan_params_default(&prm);
    prm.host_only = 1;
    auto window = [&](const std::vector<sk_problem> &list) {
      sk::HostPlan hp;
      std::string err;
      if (sk::plan_host(list.data(), (int)list.size(), &prm, hp, err) != SK_OK) return false;
      for (size_t i = 0; i < list.size(); ++i)
        if (!sk::window_operator(hp, i)) return false;
      return true;
    };
    if (!window(ps)) return fail("not taken for size-keeping convolutions of 64 channels", seed);
    sk::HostPlan hp;
    std::string err;
    if (sk::plan_host(ps.data(), (int)ps.size(), &prm, hp, err) != SK_OK) return fail(err.c_str(), seed);
    const int64_t tiles = (int64_t)hp.tiles.size();
    sk::WorkList w;
    if (sk::device_list(hp, tiles, true, w)) return fail("runs of pixels for no more tiles than workgroups", seed);
    if (tiles < 2) continue;
    if (!sk::device_list(hp, std::min<int64_t>(tiles - 1, pick({1, 16, 512})), g() % 2, w) || !w.window)
      return fail("no runs of pixels for more tiles than workgroups", seed);
    std::vector<int64_t> next(ps.size(), 0), count(ps.size(), 0);
    for (const sk_tile &t : w.work) {
      const sk::DevProblem &d = hp.dev[t.problem];
      if (t.cls != sk::CLS_WINDOW || t.m0 != next[t.problem] || t.m_len < 1 || t.m0 % 128 != 0 || t.n0 != 0 || t.n_len != d.Ng || t.S != 1 || t.k_len != (uint32_t)d.Kg ||
          ((int64_t)t.m0 + t.m_len < d.Mg && t.m_len % 128 != 0))
        return fail("a record of pixels", seed);
      next[t.problem] += t.m_len;
      ++count[t.problem];
    }
    for (size_t i = 0; i < ps.size(); ++i)
      if (next[i] != hp.dev[i].Mg) return fail("pixels missing", seed);
    if (count != w.count || w.ws_f32x4 != 0 || w.ws_off.size() < 1) return fail("counts of the records of pixels", seed);
    std::vector<sk_problem> bad = ps;
    // deadlines of their own: no run longer than a fifth of a workgroup's share (but three steps), or tiles
    std::vector<sk_problem> dated = ps;
    for (size_t i = 0; i < dated.size(); ++i) dated[i].deadline_ms = (double)(dated.size() - i);
    const int64_t grid = std::min<int64_t>(tiles - 1, pick({1, 4, 16, 512}));
    for (int edf : {1, 0}) {
      sk_plan_params by = prm;
      by.edf = edf;
      sk::HostPlan dp;
      if (sk::plan_host(dated.data(), (int)dated.size(), &by, dp, err) != SK_OK) return fail(err.c_str(), seed);
      int64_t steps = 0;
      for (const sk::DevProblem &d : dp.dev) steps += (d.Mg + 127) / 128;
      sk::WorkList dw;
      const bool runs = sk::device_list(dp, grid, true, dw) && dw.window;
      if (edf == 0 || dated.size() == 1) {
        if (!runs) return fail("no runs of pixels where no order is asked for", seed);
        continue;
      }
      if (runs != (steps / grid >= 12)) return fail("runs of pixels by deadline", seed);
      if (!runs) continue;
      for (size_t i = 0; i < dw.work.size(); ++i) {
        if (dw.work[i].m_len > 128 * std::max<int64_t>(3, steps / grid / 5)) return fail("a run that is long for its deadline", seed);
        if (i && dated[dw.work[i - 1].problem].deadline_ms > dated[dw.work[i].problem].deadline_ms) return fail("runs out of order", seed);
      }
    }
    // lists that were asked for stay: no runs
    sk_plan_params asked = prm;
    asked.xcd_part = pick({1, 2, 32});
    sk::HostPlan kept;
    if (sk::plan_host(ps.data(), (int)ps.size(), &asked, kept, err) != SK_OK || kept.xorder.empty()) return fail("lists asked for", seed);
    sk::WorkList k;
    if (sk::device_list(kept, 1, g() % 2, k) && (k.window || k.xorder.size() < kept.xorder.size())) return fail("lists asked for are dropped", seed);
    sk_problem &b = bad[g() % bad.size()];
    switch (g() % 9) {
      case 0: b.Cin = 128; break;
      case 1: b.Cout = 72; break;
      case 2: b.Cout = 4; break;
      case 3: b.Wd = 64; break;
      case 4: b.stride = 2; break;
      case 5: b.pad_w = 0; break;
      case 6: b.op = SK_CONV2D_NCHW; break;
      case 7: b.A = (const char *)b.A + 2; break;
      default: b.C = (char *)b.C + 8; break;
    }
    if (window(bad)) return fail("taken for another operator", seed);
    // beside operators that keep their tiles
    sk::WorkList m;
    if (sk::plan_host(bad.data(), (int)bad.size(), &prm, hp, err) != SK_OK) continue;
    bool fit = hp.xorder.empty();
    for (const sk::DevProblem &d : hp.dev) fit = fit && (d.flags & 3) == 3;
    const bool made = sk::device_list(hp, 1, false, m) && m.window;
    if (bad.size() > 1 && made != fit) return fail("runs of pixels beside other operators", seed);
    if (!made) continue;
    std::vector<int64_t> area(bad.size(), 0);
    for (const sk_tile &t : m.work) {
      if ((t.cls == sk::CLS_WINDOW) != sk::window_operator(hp, t.problem)) return fail("a run of pixels of another operator", seed);
      area[t.problem] += t.ks_idx == 0 ? (int64_t)t.m_len * t.n_len : 0;
    }
    for (size_t i = 0; i < bad.size(); ++i)
      if (area[i] != (int64_t)hp.dev[i].Mg * hp.dev[i].Ng) return fail("outputs beside runs of pixels", seed);
  }
  // Runs of few-channel tiles: in plans of one type, beside long reductions and channel counts of any kind.  Every output once, a run in one image and of
  // one operator that the form takes, never sliced, slices as without lists and on other grids, the operators in the order of their deadlines.
  int joined = 0, beside = 0;
  for (int seed = 0; seed < 150; ++seed) {
    std::mt19937 g(seed);
    auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + g() % v.size()); };
    std::vector<sk_problem> ps((size_t)(8 + g() % 30));
    uintptr_t addr = 0x10000000;
    const int dt = pick({SK_BF16, SK_F16, SK_F32}), deadlines = (int)(g() % 2);
    for (size_t i = 0; i < ps.size(); ++i) {
      sk_problem &p = ps[i];
      p = sk_problem{};
      p.op = SK_CONV2D_NHWC, p.dtype = dt, p.Nb = pick({1, 1, 1, 2}), p.deadline_ms = deadlines * (double)(1 + g() % 4);
      if (i % 4 != 3) {
        p.H = 40 + (int)(g() % 190), p.Wd = 40 + (int)(g() % 190), p.Cin = pick({1, 3, 3, 5}), p.Cout = pick({5, 32, 64, 64, 65});
        p.R = p.S = pick({3, 5, 7}), p.pad_h = p.pad_w = p.R / 2, p.stride = pick({1, 2, 2});
      } else {
        p.op = pick({SK_CONV2D_NHWC, SK_CONV2D_NHWC, SK_CONV2D_NCHW}), p.H = p.Wd = 7 + (int)(g() % 20), p.Cin = 128 + (int)(g() % 1900);
        p.Cout = 128 + (int)(g() % 400), p.R = p.S = 3, p.pad_h = p.pad_w = 1, p.stride = 1;
      }
      p.A = (const void *)addr, p.B = (const void *)(addr + (1u << 28)), p.C = (void *)(addr + (2u << 28));
      addr += (uintptr_t)3 << 28;
    }
    std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> plain;
    for (int part : {0, 4}) {
      sk_plan_params prm;
      sk_plan_params_default(&prm);
      prm.host_only = 1;
      prm.xcd_part = part;
      sk::HostPlan hp;
      std::string err;
      if (sk::plan_host(ps.data(), (int)ps.size(), &prm, hp, err) != SK_OK) return fail(err.c_str(), seed);
      bool marked = false;
      for (const sk::DevProblem &d : hp.dev) marked = marked || (d.flags & sk::FLAG_ROWS) != 0;
      if (marked != hp.rows || (marked && hp.tiles.size() <= 1024)) return fail("marked operators", seed);
      for (int64_t wgs : {(int64_t)512, (int64_t)200, (int64_t)33}) {
        sk::WorkList w;
        if (!sk::device_list(hp, wgs, false, w)) {
          w.work = hp.tiles, w.count = hp.count, w.ws_off = hp.ws_off, w.ws_f32x4 = hp.ws_f32x4, w.xorder = hp.xorder;
          std::copy(std::begin(hp.xoff), std::end(hp.xoff), std::begin(w.xoff));
        }
        std::map<std::tuple<uint32_t, uint32_t, uint32_t>, Slices> slices;
        if (const char *what = check(hp, w, slices)) return fail(what, seed);
        bool run = false, anew = false;
        for (size_t i = 0; i < w.work.size(); ++i) {
          const sk_tile &t = w.work[i];
          const sk::DevProblem &d = hp.dev[t.problem];
          anew = anew || t.S != hp.tiles[(size_t)hp.first[t.problem]].S;
          if (prm.edf && i && ps[w.work[i - 1].problem].deadline_ms > ps[t.problem].deadline_ms) return fail("runs of tiles out of order", seed);
          if (t.m_len <= 128) continue;
          run = true;
          const uint32_t hw = (uint32_t)(d.Ho * d.Wo);
          if (!(d.flags & sk::FLAG_ROWS) || !sk::rows_form(d, (int32_t)sk::elem_size(d.dtype)).ok || part != 0 || t.S != 1 || t.m0 % 128 != 0 ||
              t.m0 / hw != (t.m0 + t.m_len - 1) / hw)
            return fail("a run of tiles", seed);
        }
        joined += run;
        beside += run && anew;
        if (plain.empty()) plain = slices;
        if (plain.size() != slices.size()) return fail("blocks beside runs of tiles", seed);
        for (const auto &s : slices)
          if (same(s.second) != same(plain[s.first])) return fail("slices beside runs of tiles", seed);
      }
    }
  }
  if (joined < 50 || beside < 5) return fail("too few plans with runs of tiles", joined * 1000 + beside);
  // outputs past the caches: all operators of a plan of more than 160 MiB, or none
  for (int n : {1, 3, 40}) {
    for (int k : {1000, 27279, 27280, 80000}) {  // n operators of 2 x (1024 k + k + 1024) bytes
      std::vector<sk_problem> ps((size_t)n);
      for (int i = 0; i < n; ++i) {
        ps[(size_t)i] = sk_problem{};
        ps[(size_t)i].op = SK_GEMM, ps[(size_t)i].dtype = SK_BF16, ps[(size_t)i].M = 1, ps[(size_t)i].N = 1024, ps[(size_t)i].K = k;
        ps[(size_t)i].A = (const void *)0x1000, ps[(size_t)i].B = (const void *)0x100000, ps[(size_t)i].C = (void *)(0x100000000 + 4096 * (uintptr_t)i);
      }
      sk_plan_params prm;
      sk_plan_params_default(&prm);
      prm.host_only = 1;
      sk::HostPlan hp;
      std::string err;
      if (sk::plan_host(ps.data(), n, &prm, hp, err) != SK_OK) return fail(err.c_str(), n);
      const bool want = (int64_t)n * 2 * (1024LL * k + k + 1024) > (160LL << 20);
      for (const sk::DevProblem &d : hp.dev)
        if (((d.flags & sk::FLAG_PAST_CACHES) != 0) != want) return fail("outputs past the caches", n);
    }
  }
  if (cut < 100 || sliced < 100 || moved < 100) return fail("too few plans with a list of their own", cut);
  std::puts("work_list_driver: ok");
  return 0;
}
