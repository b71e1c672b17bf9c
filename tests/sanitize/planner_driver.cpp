// Host-only driver for the planner under AddressSanitizer / UndefinedBehaviorSanitizer:
// seeded random operator lists (odd sizes, strides, all element types, every parameter
// combination the planner accepts, and lists it must reject), planned whole and operator by
// operator.  Checks only what must hold for any input: status codes, table sizes, that every
// record stays inside its operator.  Byte-exact comparison with the reference planner is the
// Python tests' job.
#include <cstdint>
#include <algorithm>
#include <array>
#include <cstdio>
#include <limits>
#include <random>
#include <string>
#include <vector>

#include "sk_internal.h"

static int fail(const char *what, int seed) {
  std::fprintf(stderr, "planner_driver: %s (seed %d)\n", what, seed);
  return 1;
}

int main() {
  for (int seed = 0; seed < 300; ++seed) {
    std::mt19937 g(seed);
    auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + g() % v.size()); };
    const int n = (int)(g() % 40);
    std::vector<sk_problem> ps((size_t)n);
    uintptr_t addr = 0x10000000;
    bool expect_ok = true;
    for (int i = 0; i < n; ++i) {
      sk_problem &p = ps[(size_t)i];
      p = sk_problem{};
      p.dtype = pick({SK_F32, SK_BF16, SK_F16});
      const int es = p.dtype == SK_F32 ? 4 : 2;
      int64_t na, nb, nc;
      if (g() % 5 < 3) {
        p.op = SK_GEMM;
        p.M = pick({1, 2, 7, 16, 17, 33, 64, 65, 129, 300, 1000});
        p.N = pick({1, 5, 31, 32, 33, 127, 128, 129, 500, 4097});
        p.K = pick({1, 3, 8, 63, 64, 65, 256, 1000, 4096, 9000});
        p.lda = g() % 3 ? 0 : p.K + (int)(g() % 9);
        p.ldb = g() % 3 ? 0 : p.K + (int)(g() % 9);
        p.ldc = g() % 3 ? 0 : p.N + (int)(g() % 9);
        na = (int64_t)p.M * (p.lda ? p.lda : p.K);
        nb = (int64_t)p.N * (p.ldb ? p.ldb : p.K);
        nc = (int64_t)p.M * (p.ldc ? p.ldc : p.N);
      } else {
        p.op = SK_CONV2D_NHWC;
        p.Nb = 1 + (int)(g() % 2);
        p.H = 1 + (int)(g() % 40);
        p.Wd = 1 + (int)(g() % 40);
        p.Cin = pick({1, 3, 8, 64, 200});
        p.Cout = pick({1, 7, 64, 130});
        p.R = pick({1, 3, 5, 7});
        p.S = pick({1, 3});
        p.pad_h = (int)(g() % 4);
        p.pad_w = (int)(g() % 2);
        p.stride = (int)(g() % 4);
        if (p.H + 2 * p.pad_h < p.R || p.Wd + 2 * p.pad_w < p.S) expect_ok = false;
        na = (int64_t)p.Nb * p.H * p.Wd * p.Cin;
        nb = (int64_t)p.Cout * p.R * p.S * p.Cin;
        nc = (int64_t)p.Nb * (p.H + 2 * p.pad_h + 1) * (p.Wd + 2 * p.pad_w + 1) * p.Cout;
      }
      p.A = (const void *)addr;
      addr += (uintptr_t)(na * es + 511) / 256 * 256;
      p.B = (const void *)addr;
      addr += (uintptr_t)(nb * es + 511) / 256 * 256;
      p.C = (void *)(addr + (g() % 4 == 0 ? 2 : 0));  // sometimes misaligned
      addr += (uintptr_t)(nc * es + 767) / 256 * 256;
      const double ds[] = {0.0, -1.0, 0.5, 0.5, 3.0, 1e300, std::numeric_limits<double>::infinity(),
                           std::numeric_limits<double>::quiet_NaN()};
      p.deadline_ms = ds[g() % 8];
    }
    sk_plan_params prm;
    sk_plan_params_default(&prm);
    prm.host_only = 1;
    prm.edf = (int)(g() % 2);
    prm.skinny_max_m = pick({0, 8, 16, 32, 64});
    prm.tile_bytes_min = pick({1024, 4096, 32768, 1 << 18});
    prm.tile_bytes_max = prm.tile_bytes_min * pick({1, 2, 16, 64});
    prm.balance_div = pick({1, 7, 64, 512, 2048});
    prm.max_groups = pick({1, 3, 4, 64, 256});
    prm.tail_div = pick({0, 1, 16, 384, 5000});
    sk::HostPlan hp;
    std::string err;
    const sk_status st = sk::plan_host(n ? ps.data() : nullptr, n, &prm, hp, err);
    if (!expect_ok) {
      if (st == SK_OK) return fail("a filter larger than its padded image was accepted", seed);
      continue;
    }
    if (st != SK_OK) {
      std::fprintf(stderr, "%s\n", err.c_str());
      return fail("plan_host failed on a valid list", seed);
    }
    if ((int)hp.dev.size() != n || (int)hp.order.size() != n) return fail("table sizes", seed);
    int64_t sum = 0;
    for (int i = 0; i < n; ++i) sum += hp.count[(size_t)i];
    if (sum != (int64_t)hp.tiles.size()) return fail("tile counts do not add up", seed);
    for (const sk_tile &t : hp.tiles) {
      if ((int)t.problem >= n) return fail("record names a missing operator", seed);
      const sk::DevProblem &d = hp.dev[t.problem];
      if (t.m_len < 1 || t.n_len < 1 || t.k_len < 1 || (int64_t)t.m0 + t.m_len > d.Mg ||
          (int64_t)t.n0 + t.n_len > d.Ng || (int64_t)t.k0 + t.k_len > d.Kg || t.ks_idx >= t.S ||
          t.out_tile_id >= hp.ws_off.size())
        return fail("record leaves its operator", seed);
    }
    // the device's work list: every record once, whole or in parts that tile it; only what may be cut is
    for (int64_t wgs : {(int64_t)1, (int64_t)7, (int64_t)512}) {
      std::vector<sk_tile> work;
      std::vector<int64_t> counts;
      if (!sk::refine_tiles(hp, wgs, work, counts)) {
        if (!work.empty() || !counts.empty()) return fail("a work list that nothing is cut in", seed);
        continue;
      }
      size_t at = 0;
      std::vector<int64_t> seen((size_t)n, 0);
      for (const sk_tile &t : hp.tiles) {
        const sk::DevProblem &d = hp.dev[t.problem];
        const bool vec = (d.flags & (sk::FLAG_VEC_A | sk::FLAG_VEC_B)) == (sk::FLAG_VEC_A | sk::FLAG_VEC_B);
        uint32_t m = t.m0, nn = t.n0;
        int64_t area = 0;
        while (area < (int64_t)t.m_len * t.n_len) {
          if (at == work.size()) return fail("work list ends early", seed);
          const sk_tile &u = work[at++];
          ++seen[t.problem];
          if (u.problem != t.problem || u.cls != t.cls || u.S != t.S || u.ks_idx != t.ks_idx || u.k0 != t.k0 || u.k_len != t.k_len ||
              u.out_tile_id != t.out_tile_id || u.m0 != m || u.n0 != nn || u.m_len < 1 || u.n_len < 1)
            return fail("a part that is not of its record", seed);
          const bool whole = u.m_len == t.m_len && u.n_len == t.n_len;
          if (!whole && (t.S != 1 || d.Kg <= 64 || vec || u.m_len > 64 || u.n_len > 64)) return fail("cut what must stay whole", seed);
          area += (int64_t)u.m_len * u.n_len;
          nn += u.n_len;
          if (nn == t.n0 + t.n_len) nn = t.n0, m += u.m_len;
        }
        if (area != (int64_t)t.m_len * t.n_len) return fail("parts overlap", seed);
      }
      if (at != work.size() || seen != counts) return fail("work list counts", seed);
    }
    sk::HostPlan alone;
    if (sk::plan_host_each_alone(hp, 512, alone, err) != SK_OK) return fail("plan_host_each_alone", seed);
    if (alone.dev.size() != hp.dev.size()) return fail("baseline tables", seed);
  }
  // Convolution operands read through descriptors: the offset of a pixel, the scalar offset of a tap and the element itself must
  // stay below what offsets_below() promises for every pixel and tap, those outside the image too (their offset
  // carries the top bit, and no sum may wrap or lose it); inside the image they must name the element.
  for (int seed = 0; seed < 400; ++seed) {
    std::mt19937 g(seed);
    auto upto = [&](int n) { return (int)(g() % (unsigned)n); };
    sk_problem p{};
    p.op = seed % 2 ? SK_CONV2D_NCHW : SK_CONV2D_NHWC;
    p.dtype = upto(2) ? SK_BF16 : SK_F32;
    const int64_t es = p.dtype == SK_F32 ? 4 : 2;
    do {
      p.Nb = 1 + upto(4), p.H = 1 + upto(6), p.Wd = 1 + upto(6), p.Cin = 1 + upto(9), p.Cout = 3;
      p.R = 1 + upto(7), p.S = 1 + upto(7), p.pad_h = upto(9), p.pad_w = upto(9), p.stride = 1 + upto(3);
    } while (p.H + 2 * p.pad_h < p.R || p.Wd + 2 * p.pad_w < p.S);
    p.A = (const void *)0x10000, p.B = (const void *)0x20000, p.C = (void *)0x30000;
    sk_plan_params prm;
    sk_plan_params_default(&prm);
    prm.host_only = 1;
    sk::HostPlan hp;
    std::string err;
    if (sk::plan_host(&p, 1, &prm, hp, err) != SK_OK) return fail("plan_host failed on a small convolution", seed);
    const sk::DevProblem &d = hp.dev[0];
    int64_t most = 0;  // bytes an offset, a scalar offset and the element reach, over one tile of all images
    const int64_t image = (int64_t)p.H * p.Wd * p.Cin, corner = (int64_t)p.pad_h * p.Wd + p.pad_w;
    for (int64_t b = 0; b < p.Nb; ++b)
      for (int64_t ho = 0; ho < d.Ho; ++ho)
        for (int64_t wo = 0; wo < d.Wo; ++wo)
          for (int64_t r = 0; r < p.R; ++r)
            for (int64_t t = 0; t < p.S; ++t)
              for (int64_t c = 0; c < p.Cin; ++c) {
                const int64_t hs = ho * p.stride, ws = wo * p.stride, h = hs - p.pad_h + r, w = ws - p.pad_w + t;
                const int64_t off = p.op == SK_CONV2D_NCHW ? b * image + hs * p.Wd + ws : ((b * p.H + hs) * p.Wd + ws) * p.Cin;
                const int64_t soff = p.op == SK_CONV2D_NCHW ? (c * p.H + r) * p.Wd + t : (r * p.Wd + t) * p.Cin + c;
                most = std::max(most, (off + soff + 1) * es);
                if (h < 0 || h >= p.H || w < 0 || w >= p.Wd) continue;
                const int64_t place = p.op == SK_CONV2D_NCHW ? ((b * p.Cin + c) * p.H + h) * p.Wd + w : ((b * p.H + h) * p.Wd + w) * p.Cin + c;
                if (off + soff - corner * (p.op == SK_CONV2D_NCHW ? 1 : p.Cin) != place) return fail("an offset misses its element", seed);
              }
    if (!sk::offsets_below(d, p.Nb - 1, es, most + 1) || sk::offsets_below(d, p.Nb - 1, es, most))
      return fail("offsets_below is not the largest offset", seed);
  }
  {
    // sizes at which 32 bits do not hold the products: never below any limit
    sk_problem p{};
    p.op = SK_CONV2D_NHWC, p.dtype = SK_F32, p.Nb = 1, p.H = 1 << 19, p.Wd = 1 << 19, p.Cin = 1 << 10, p.Cout = 1, p.R = 1, p.S = 1;
    p.stride = 1 << 10;
    p.A = (const void *)0x10000, p.B = (const void *)0x20000, p.C = (void *)0x30000;
    sk::HostPlan hp;
    std::string err;
    if (sk::plan_host(&p, 1, nullptr, hp, err) != SK_OK) return fail("plan_host failed on a large convolution", -4);
    if (hp.dev[0].reach != 1u << 31 || sk::offsets_below(hp.dev[0], 0, 4, (int64_t)1 << 31)) return fail("reach of a large image", -4);
  }
  // What is cut, on hand-worked plans.
  {
    sk_plan_params prm;
    sk_plan_params_default(&prm);
    prm.host_only = 1;
    uintptr_t addr = 0x10000000;
    auto place = [&](sk_problem &p) {
      p.A = (const void *)addr, p.B = (const void *)(addr + (1u << 30)), p.C = (void *)(addr + (2u << 30));
      addr += (uintptr_t)3 << 30;
    };
    auto gemm = [&](int dt, int m, int nn, int k) {
      sk_problem p{};
      p.op = SK_GEMM, p.dtype = dt, p.M = m, p.N = nn, p.K = k;
      place(p);
      return p;
    };
    auto conv = [&](int op, int dt, int hw, int ci, int co, int r, int stride, int pad) {
      sk_problem p{};
      p.op = op, p.dtype = dt, p.Nb = 1, p.H = p.Wd = hw, p.Cin = ci, p.Cout = co, p.R = p.S = r, p.stride = stride, p.pad_h = p.pad_w = pad;
      place(p);
      return p;
    };
    auto records = [&](const std::vector<sk_problem> &ps, int64_t wgs) -> int64_t {
      sk::HostPlan hp;
      std::string err;
      if (sk::plan_host(ps.data(), (int)ps.size(), &prm, hp, err) != SK_OK) return -1;
      std::vector<sk_tile> work;
      std::vector<int64_t> counts;
      return sk::refine_tiles(hp, wgs, work, counts) ? (int64_t)work.size() : 0;  // 0: nothing cut
    };
    // 300 x 130 outputs over 1001: 3 x 2 records of 16 stages, (128, 128) 37.6 us, (128, 2) 32, (44, 128) 27.8, (44, 2) 24.2, a part 24.2.
    // All but the last are cut: 2 * 4 + 2 * 2 + 2 + 1.
    const sk_problem odd = gemm(SK_BF16, 300, 130, 1001), odd2 = gemm(SK_F16, 300, 130, 1001);
    if (records({odd}, 512) != 15) return fail("an odd operator by itself", -5);
    // the one-launch-per-operator baseline cuts every operator as if it were alone, whatever the plan waits for
    {
      const std::vector<sk_problem> ps = {odd, gemm(SK_F32, 128, 128, 2040), odd2};
      sk::HostPlan hp, alone;
      std::string err;
      if (sk::plan_host(ps.data(), 3, &prm, hp, err) != SK_OK || sk::plan_host_each_alone(hp, 512, alone, err) != SK_OK)
        return fail("baseline of odd operators", -5);
      if (alone.count != std::vector<int64_t>{15, 1, 15} || alone.first != std::vector<int64_t>{0, 15, 16} || alone.tiles.size() != 31 ||
          alone.dev[2].tile_count != 15 || alone.tiles[30].problem != 2 || alone.tiles[30].out_tile_id != 12)
        return fail("tables of the baseline", -5);
    }
    // ten workgroups start the six records at once, but not the parts of the five that outlast a part: all are cut
    if (records({odd}, 10) != 15) return fail("parts that cannot start at once", -5);
    // two records of 8 stages besides, 22.8 us each: cut where all 23 parts and records start at once, else not
    const sk_problem shorter = gemm(SK_BF16, 256, 128, 449);
    if (records({odd, shorter}, 23) != 23) return fail("a workgroup for every part", -5);
    if (records({odd, shorter}, 20) != 17) return fail("a workgroup for every part that must be", -5);
    // four workgroups: 2 * 110 us of work / 4 is more than the longest record
    if (records({odd}, 4) != 0) return fail("a full chip", -5);
    // beside an fp32 operator of 64 stages (133 us) in aligned pieces
    if (records({odd, gemm(SK_F32, 128, 128, 2040)}, 512) != 0) return fail("a longer record that cannot be cut", -5);
    // at most 64 reduction elements: never
    if (records({gemm(SK_BF16, 300, 130, 63)}, 512) != 0) return fail("a short reduction", -5);
    // the stride-2 layers with the 7x7 stem: records of three stages, for one tenant to six
    std::vector<sk_problem> mix;
    for (int t = 0; t < 6; ++t) {
      for (const auto &l : {std::array<int, 5>{224, 3, 64, 7, 3}, {56, 128, 128, 3, 1}, {56, 256, 512, 1, 0}, {28, 256, 256, 3, 1},
                            {28, 512, 1024, 1, 0}, {14, 512, 512, 3, 1}, {14, 1024, 2048, 1, 0}})
        mix.push_back(conv(SK_CONV2D_NHWC, SK_BF16, l[0], l[1], l[2], l[3], 2, l[4]));
      if (records(mix, 512) != 0) return fail("stems of a few tenants", t);
    }
    // channel-major ResNet layers: the sliced 14 x 14 layer is what one tenant to five wait for
    for (int dt : {SK_F16, SK_F32}) {
      mix.clear();
      for (int t = 0; t < 5; ++t) {
        for (const auto &l : {std::array<int, 4>{56, 64, 256, 1}, {56, 64, 64, 3}, {28, 128, 512, 1}, {28, 128, 128, 3}, {14, 256, 1024, 1},
                              {14, 256, 256, 3}, {7, 512, 2048, 1}, {7, 512, 512, 3}})
          mix.push_back(conv(SK_CONV2D_NCHW, dt, l[0], l[1], l[2], l[3], 1, l[3] / 2));
        if (records(mix, 512) != 0) return fail("channel-major layers of a few tenants", t);
      }
    }
  }
  // Narrow plans: every tile, of the plan and of its operators alone, must satisfy what the device's direct loads ask for (a tile
  // that does not would never be run there); at the limits of that, and where the kernel for them is taken.
  {
    auto lean = [](const sk::DevProblem &d, const sk_tile &t) {
      const int64_t es = sk::elem_size(d.dtype), limit = ((int64_t)1 << 31) - 4096, kb = 128 / es;
      if ((d.flags & (sk::FLAG_VEC_A | sk::FLAG_VEC_B)) != (sk::FLAG_VEC_A | sk::FLAG_VEC_B) || t.cls != sk::CLS_TILE_128x64) return false;
      if (((int64_t)(t.n_len - 1) * d.ldb + d.Kg) * es >= limit) return false;
      if (!d.gather) return ((int64_t)(t.m_len - 1) * d.lda + d.Kg) * es < limit;
      const int64_t hw = (int64_t)d.Ho * d.Wo;
      return !d.nchw && d.Cin % kb == 0 && d.R * d.S <= 31 && sk::offsets_below(d, (t.m0 + t.m_len - 1) / hw - t.m0 / hw, es, limit);
    };
    int narrow = 0;
    for (int seed = 0; seed < 2000; ++seed) {
      std::mt19937 g(seed);
      auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + g() % v.size()); };
      std::vector<sk_problem> ps(1 + g() % 3);
      uintptr_t addr = 0x10000000;
      const int dt = pick({SK_F32, SK_BF16});
      for (sk_problem &p : ps) {
        p = sk_problem{};
        p.dtype = dt;
        if (g() % 2) {
          p.op = SK_GEMM, p.M = pick({65, 128, 200, 5000}), p.N = pick({1, 40, 64, 64, 65}), p.K = pick({8, 64, 1000, 4096, 4100});
          p.lda = pick({0, 0, 1 << 20, 1 << 21, 1 << 22, 1 << 23}), p.ldb = pick({0, 0, 1 << 21, 1 << 22, 1 << 23});
        } else {
          p.op = g() % 8 ? SK_CONV2D_NHWC : SK_CONV2D_NCHW, p.Nb = pick({1, 2, 40}), p.H = pick({1, 9, 56, 2000}), p.Wd = pick({9, 56, 700});
          p.Cin = pick({32, 64, 64, 96, 128}), p.Cout = pick({8, 64}), p.R = pick({1, 3, 5}), p.S = pick({1, 3, 5, 7}), p.pad_h = p.R / 2, p.pad_w = pick({0, 3, 3000});
          p.stride = pick({1, 2, 3});
        }
        p.A = (const void *)addr, p.B = (const void *)(addr + ((uintptr_t)1 << 40)), p.C = (void *)(addr + ((uintptr_t)2 << 40));
        addr += (uintptr_t)3 << 40;
      }
      sk_plan_params prm;
      sk_plan_params_default(&prm);
      prm.host_only = 1;
      prm.tile_bytes_max = prm.tile_bytes_min * pick({1, 64});
      sk::HostPlan hp, alone;
      std::string err;
      if (sk::plan_host(ps.data(), (int)ps.size(), &prm, hp, err) != SK_OK || !sk::narrow_plan(hp)) continue;
      ++narrow;
      if (sk::plan_host_each_alone(hp, 512, alone, err) != SK_OK) return fail("plan_host_each_alone", seed);
      for (const sk::HostPlan *h : {&hp, &alone})
        for (const sk_tile &t : h->tiles)
          if (!lean(h->dev[t.problem], t)) return fail("a tile of a narrow plan that the direct loads cannot serve", seed);
    }
    if (narrow < 100) return fail("hardly any narrow plan", narrow);
    auto one = [](int64_t lda, int64_t ldb) {
      sk_problem p{};
      p.op = SK_GEMM, p.dtype = SK_BF16, p.M = 300, p.N = 64, p.K = 64, p.lda = lda, p.ldb = ldb;
      p.A = (const void *)0x10000, p.B = (const void *)((uintptr_t)1 << 44), p.C = (void *)((uintptr_t)1 << 45);
      sk::HostPlan hp;
      std::string err;
      return sk::plan_host(&p, 1, nullptr, hp, err) == SK_OK && sk::narrow_plan(hp);
    };
    if (!one(0, 0) || one(1 << 22, 0) || !one((1 << 22) - 8, 0) || one(0, 1 << 23) || !one(0, (1 << 23) - 8))
      return fail("narrow_plan at its limits", -6);
    for (bool f : {false, true}) {
      const int64_t c = 256;
      if (!sk::narrow_pays(f, 9, c, c) || sk::narrow_pays(f, 9, c + 1, c) || sk::narrow_pays(f, 9, 2 * c, c) || !sk::narrow_pays(f, 9, 2 * c + 1, c) ||
          !sk::narrow_pays(f, 9, 691, c) || sk::narrow_pays(f, 9, 692, c) || sk::narrow_pays(f, 9, (f ? 8 : 15) * c - 1, c) ||
          !sk::narrow_pays(f, 9, (f ? 8 : 15) * c, c) || sk::narrow_pays(f, 13, 15 * c, c) != f || sk::narrow_pays(f, 13, c, c))
        return fail("narrow_pays", f);
    }
  }
  // lists the planner must reject
  {
    sk::HostPlan hp;
    std::string err;
    sk_problem p{};
    p.op = SK_GEMM;
    p.dtype = SK_BF16;
    p.M = 4;
    p.N = 64;
    p.K = 64;
    p.A = (const void *)0x1000;
    p.B = (const void *)0x2000;
    p.C = (void *)0x3000;
    sk_problem two[2] = {p, p};  // same output twice
    if (sk::plan_host(two, 2, nullptr, hp, err) != SK_ERR_OVERLAP) return fail("overlap not detected", -1);
    p.M = 0;
    if (sk::plan_host(&p, 1, nullptr, hp, err) != SK_ERR_INVALID_ARG) return fail("M = 0 accepted", -1);
    if (sk::plan_host(nullptr, 3, nullptr, hp, err) != SK_ERR_INVALID_ARG) return fail("null list accepted", -1);
  }
  // the launch ledger: which launches are admitted at once, which only after the plan's event has
  // completed, and what destroying the plan waits for
  {
    using L = sk::LaunchLedger;
    L l;
    const uintptr_t s1 = 0x100, s2 = 0x200;
    if (l.before_destroy() != L::NOTHING) return fail("a plan never launched waits for something", -2);
    if (l.before_launch(s1, false) != L::GO) return fail("first launch not admitted", -2);
    l.after_launch(s1, false, true);
    if (l.before_launch(s1, false) != L::GO) return fail("same stream must be admitted: the stream orders it", -2);
    if (l.before_launch(s2, false) != L::QUERY_EVENT) return fail("another stream must ask the event", -2);
    if (l.before_launch(0, false) != L::QUERY_EVENT) return fail("the default stream is another stream", -2);
    if (l.before_destroy() != L::EVENT) return fail("destroy must wait for the event", -2);
    l.after_launch(s2, false, true);  // admitted after the event completed: now the latest launch is on s2
    if (l.before_launch(s2, false) != L::GO || l.before_launch(s1, false) != L::QUERY_EVENT)
      return fail("the ledger did not move to the new stream", -2);
    if (l.before_destroy() != L::EVENT) return fail("one event covers launches admitted one after the other", -2);
    if (l.before_launch(s1, true) != L::GO) return fail("a captured launch cannot ask anything", -2);
    l.after_launch(s1, true, false);
    if (l.before_destroy() != L::DEVICE) return fail("graph replays need the device-wide wait", -2);
    if (l.before_launch(s1, false) != L::QUERY_EVENT) return fail("eager launches are still checked after a capture", -2);
    L m;
    m.after_launch(s1, false, false);  // the event could not be recorded
    if (m.before_destroy() != L::DEVICE) return fail("a launch without an event needs the device-wide wait", -2);
    if (m.before_launch(s2, false) != L::GO) return fail("nothing to ask without an event", -2);
    L d;                               // first launch on the default stream (handle 0)
    d.after_launch(0, false, true);
    if (d.before_launch(0, false) != L::GO || d.before_launch(s1, false) != L::QUERY_EVENT)
      return fail("default stream as the plan's stream", -2);
  }
  // the arrival queue's batch selection
  {
    const double inf = std::numeric_limits<double>::infinity();
    char buf[8];
    const void *c0 = buf, *c1 = buf + 1, *c2 = buf + 2, *c3 = buf + 3;
    // arrival order: deadlines 5, 1, inf, 1 (tie with index 1), 0.5 on the buffer of index 0
    std::vector<sk::QueuedOp> ops = {{5.0, 1000, c0}, {1.0, 1000, c1}, {inf, 1000, c2}, {1.0, 4000, c3}, {0.5, 1000, c0}};
    std::vector<const void *> none, busy = {c1};
    std::sort(busy.begin(), busy.end());
    auto same = [](const std::vector<size_t> &a, std::initializer_list<size_t> b) { return a == std::vector<size_t>(b); };
    // everything that is free, earliest deadline first, ties by arrival; the later operator of a shared buffer waits
    if (!same(sk::select_batch(ops, none, SK_QUEUE_COALESCE, 0.5, 1.0, 1000.0, 0.0), {4, 1, 3, 2}))
      return fail("coalesce order", -3);
    if (!same(sk::select_batch(ops, busy, SK_QUEUE_COALESCE, 0.5, 1.0, 1000.0, 0.0), {4, 3, 2}))
      return fail("an operator whose output is in flight must wait", -3);
    // 1000 bytes per ms: the cap of 2.5 ms closes the batch before the 4000-byte operator; the operators behind
    // it in deadline order wait as well
    if (!same(sk::select_batch(ops, none, SK_QUEUE_OOO, 2.5, 1.0, 1000.0, 0.0), {4, 1})) return fail("cap", -3);
    // ... a correction factor of 2 already before the second operator
    if (!same(sk::select_batch(ops, none, SK_QUEUE_OOO, 2.5, 2.0, 1000.0, 0.0), {4})) return fail("corrected cap", -3);
    // a first operator is always taken, however long
    if (!same(sk::select_batch(ops, none, SK_QUEUE_OOO, 0.001, 1.0, 1000.0, 0.0), {4})) return fail("first operator", -3);
    // the floor counts: three operators of 1 ms each are estimated at the floor of 10 ms
    if (!same(sk::select_batch(ops, none, SK_QUEUE_OOO, 10.0, 1.0, 1000.0, 10.0), {4, 1, 3, 2})) return fail("floor", -3);
    if (!same(sk::select_batch(ops, busy, SK_QUEUE_SEQUENTIAL, 0.5, 1.0, 1000.0, 0.0), {0})) return fail("arrival order", -3);
    if (!sk::select_batch({}, none, SK_QUEUE_OOO, 0.5, 1.0, 1000.0, 0.0).empty()) return fail("empty queue", -3);
    if (sk::estimate_launch_ms(5000, 1000.0, 0.02) != 5.0 || sk::estimate_launch_ms(10, 1000.0, 0.02) != 0.02)
      return fail("estimate", -3);
    sk_problem g{};
    g.op = SK_GEMM;
    g.dtype = SK_BF16;
    g.M = 3;
    g.N = 5;
    g.K = 7;
    if (sk::operand_bytes(g) != 2 * (3 * 7 + 5 * 7 + 3 * 5)) return fail("GEMM bytes", -3);
    sk_problem cv{};
    cv.op = SK_CONV2D_NHWC;
    cv.dtype = SK_F32;
    cv.Nb = 2; cv.H = 9; cv.Wd = 8; cv.Cin = 3; cv.Cout = 4; cv.R = 3; cv.S = 3; cv.pad_h = 1; cv.pad_w = 1; cv.stride = 2;
    // Ho = (9 + 2 - 3) / 2 + 1 = 5, Wo = (8 + 2 - 3) / 2 + 1 = 4
    if (sk::operand_bytes(cv) != 4 * (2 * 9 * 8 * 3 + 4 * 3 * 3 * 3 + 2 * 5 * 4 * 4)) return fail("convolution bytes", -3);
    cv.R = 20;
    if (sk::operand_bytes(cv) != 0) return fail("malformed operator", -3);
  }
  std::puts("planner_driver: ok");
  return 0;
}
