// Host planner: operators -> canonical GEMM view -> tile classes -> earliest-
// deadline-first operator order -> flat tile table.
//
// This is the paper's runtime packing step (Section 5.3: many small kernels are
// repacked into one large execution block) together with its latency-aware
// reordering (Section 5, item (a): tighter latency budgets first).  The paper
// gives no algorithm for either; the rule implemented here is a pure integer
// function of the operator list and sk_plan_params, so that it can be checked
// byte for byte against an independent reference planner.
//
// No HIP call is made in this file.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <limits>
#include <numeric>
#include <unordered_set>

#include "sk_internal.h"

namespace sk {

namespace {

struct Canon {
  int64_t Mg, Ng, Kg;
  int32_t Ho, Wo;
};

std::string at(int32_t i) { return "problem " + std::to_string(i) + ": "; }

// Canonical GEMM view (rows = output pixels, columns = output channels,
// reduction = filter taps x input channels for a convolution).
sk_status canonicalise(const sk_problem &p, int32_t i, Canon &c, std::string &err) {
  if (p.dtype != SK_F32 && p.dtype != SK_BF16 && p.dtype != SK_F16) {
    err = at(i) + "unknown dtype " + std::to_string(p.dtype);
    return SK_ERR_UNSUPPORTED;
  }
  if (!p.A || !p.B || !p.C) {
    err = at(i) + "null operand pointer";
    return SK_ERR_INVALID_ARG;
  }
  if (p.op == SK_GEMM) {
    if (p.M < 1 || p.N < 1 || p.K < 1) {
      err = at(i) + "GEMM dimensions must be >= 1";
      return SK_ERR_INVALID_ARG;
    }
    if (p.lda < 0 || p.ldb < 0 || p.ldc < 0 || (p.lda && p.lda < p.K) || (p.ldb && p.ldb < p.K) ||
        (p.ldc && p.ldc < p.N)) {
      err = at(i) + "row stride smaller than a row";
      return SK_ERR_INVALID_ARG;
    }
    c = Canon{p.M, p.N, p.K, 0, 0};
  } else if (p.op == SK_CONV2D_NHWC || p.op == SK_CONV2D_NCHW) {
    if (p.Nb < 1 || p.H < 1 || p.Wd < 1 || p.Cin < 1 || p.Cout < 1 || p.R < 1 || p.S < 1 || p.pad_h < 0 ||
        p.pad_w < 0) {
      err = at(i) + "convolution dimensions must be >= 1 and padding >= 0";
      return SK_ERR_INVALID_ARG;
    }
    if (p.stride < 0 || p.stride > 1 << 10) {
      err = at(i) + "stride must be 0 (meaning 1) or 1..1024";
      return SK_ERR_INVALID_ARG;
    }
    const int64_t st = p.stride ? p.stride : 1;
    const int64_t span_h = (int64_t)p.H + 2 * (int64_t)p.pad_h - p.R;
    const int64_t span_w = (int64_t)p.Wd + 2 * (int64_t)p.pad_w - p.S;
    const int64_t Ho = span_h < 0 ? 0 : span_h / st + 1;
    const int64_t Wo = span_w < 0 ? 0 : span_w / st + 1;
    if (Ho < 1 || Wo < 1) {
      err = at(i) + "filter larger than the padded image";
      return SK_ERR_INVALID_ARG;
    }
    if (Ho > 1 << 20 || Wo > 1 << 20) {
      err = at(i) + "image too large";
      return SK_ERR_UNSUPPORTED;
    }
    c = Canon{(int64_t)p.Nb * Ho * Wo, p.Cout, (int64_t)p.R * p.S * p.Cin, (int32_t)Ho, (int32_t)Wo};
  } else {
    err = at(i) + "unknown operator " + std::to_string(p.op);
    return SK_ERR_UNSUPPORTED;
  }
  const int64_t lim = std::numeric_limits<int32_t>::max() / 2;
  if (c.Mg > lim || c.Ng > lim || c.Kg > lim) {
    err = at(i) + "canonical dimension does not fit 31 bits";
    return SK_ERR_UNSUPPORTED;
  }
  return SK_OK;
}

double deadline_key(double d) {
  if (!(d > 0.0) || std::isinf(d)) return std::numeric_limits<double>::infinity();
  return d;
}

// Partial sums of one slice of an output rectangle, in 16-byte units: 4 waves x (2 * rm) accumulators x 64 lanes (LDS tiles: 256
// threads x 16 accumulator quads, 8 for the 64-column tile).
int64_t slice_f32x4(uint16_t cls) {
  return cls == CLS_TILE_128x128 ? 4096 : cls == CLS_TILE_128x64 ? 2048 : 4 * 2 * ((int64_t)1 << (cls / 3)) * 64;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// Operand bytes the tiles of an operator load ("stream bytes"): what the tile targets are measured in.
// A skinny operator reads its weights once.  An operator in the LDS-tile classes reads, per 128 x BN output
// tile, the 128 + BN operand rows of that tile over the whole reduction: its weight array alone would
// understate its share of a launch by the number of row blocks.
static int64_t stream_bytes(int64_t Mg, int64_t Ng, int64_t Kg, int64_t es, const sk_plan_params &prm) {
  if (Mg <= prm.skinny_max_m) return Ng * Kg * es;
  const int64_t bn = Ng <= 64 ? 64 : 128;
  return ((Mg + 127) / 128) * ((Ng + bn - 1) / bn) * (128 + bn) * Kg * es;
}

// Which accelerator die (XCD: 32 compute units behind one 4 MB L2) runs which LDS tile.  The tiles of an
// operator in the LDS-tile classes share operands: the tiles of one row block read the same 128 activation
// rows, those of one column block the same weight rows.  Handed out in table order they land on all eight
// dies, and every die fetches every panel from memory for itself.  So the output rectangles of such an
// operator are cut into `p` two-dimensional parts (p = 1, 2, 4 or 8: the fewest with at most xcd_part
// rectangles each; the pm x pn grid of parts that fetches the fewest operand rows in total), each part goes to
// one die (the dies with the fewest entries so far, lowest index first), and within a part the rectangles
// follow a Z-order curve in blocks of 8 x 8, so that the handful of tiles a die runs at any one time share panels as well.
// The reduction slices of a rectangle stay together.  The lists name tiles of the table; the table itself,
// and with it the order in which the launch takes LDS tiles up, does not change.
// xcd_part = -1: the planner decides.  The lists pay where the matrix cores, not memory, bound the launch and no
// skinny tile is in it (measured: plans of LDS tiles only gain 0 to 10 % when the sum over operators of
// flops / peak exceeds that of operand bytes / bandwidth, lose 2 to 5 % otherwise, and every plan that mixes in
// skinny tiles loses).  Peaks as the ratio of the datasheet figures (2500 TFLOP/s for 16-bit types, 157.3 for
// fp32, 8 TB/s), so that no device property enters: flops * 2 * (1573 | 25000) against bytes * 983125.
// Then a part is an eighth of all output rectangles of the plan: whole operators per die where there are
// many, an operator's eighths where there is one.
static int64_t resolve_xcd_part(const HostPlan &out, const std::vector<Canon> &canon) {
  if (out.params.xcd_part >= 0) return out.params.xcd_part;
  unsigned __int128 t_flops = 0, t_bytes = 0;
  int64_t rects = 0;
  for (size_t i = 0; i < out.problems.size(); ++i) {
    if (out.count[i] == 0) continue;
    const sk_tile &t0 = out.tiles[(size_t)out.first[i]];
    if (t0.cls != CLS_TILE_128x128 && t0.cls != CLS_TILE_128x64) return 0;  // a skinny operator
    const int64_t bn = t0.cls == CLS_TILE_128x64 ? 64 : 128;
    rects += ((canon[i].Mg + 127) / 128) * ((canon[i].Ng + bn - 1) / bn);
    const unsigned __int128 flops = (unsigned __int128)2 * (uint64_t)canon[i].Mg * (uint64_t)canon[i].Ng * (uint64_t)canon[i].Kg;
    t_flops += flops * 2u * (out.problems[i].dtype == SK_F32 ? 25000u : 1573u);
    t_bytes += (unsigned __int128)(uint64_t)operand_bytes(out.problems[i]) * 983125u;
  }
  if (rects == 0 || t_flops <= t_bytes) return 0;
  return (rects + 7) / 8;
}

static void build_xcd_lists(HostPlan &out, const std::vector<Canon> &canon) {
  out.xorder.clear();
  std::fill(std::begin(out.xoff), std::end(out.xoff), 0u);
  const int64_t part = resolve_xcd_part(out, canon);
  if (part <= 0) return;
  std::vector<uint32_t> lists[8];
  for (const int32_t i : out.order) {
    if (out.count[i] == 0) continue;
    const sk_tile &t0 = out.tiles[(size_t)out.first[i]];
    if (t0.cls != CLS_TILE_128x128 && t0.cls != CLS_TILE_128x64) continue;
    const int64_t bn = t0.cls == CLS_TILE_128x64 ? 64 : 128;
    const int64_t MB = (canon[i].Mg + 127) / 128, NB = (canon[i].Ng + bn - 1) / bn, S = t0.S;
    int64_t p = 1;
    while (p < 8 && MB * NB > p * part) p *= 2;
    // pn parts along the columns: every row block is then fetched by pn dies, every column block by pm
    int64_t pm = 1, pn = 1, best = -1;
    for (int64_t cn = 1; cn <= p; cn *= 2) {
      const int64_t cm = p / cn;
      if (cm > MB || cn > NB) continue;
      const int64_t rows = cn * MB * 128 + cm * NB * bn;
      if (best < 0 || rows < best) best = rows, pm = cm, pn = cn;
    }
    if (best < 0) {  // no such grid (three column blocks and one row block cut in four, say): cut the rows only
      pm = std::min<int64_t>(p, MB);
      pn = 1;
    }
    bool used[8] = {};
    for (int64_t a = 0; a < pm; ++a) {
      for (int64_t b = 0; b < pn; ++b) {
        int die = -1;
        for (int x = 0; x < 8; ++x)
          if (!used[x] && (die < 0 || lists[x].size() < lists[die].size())) die = x;
        used[die] = true;
        const int64_t m_lo = a * MB / pm, m_hi = (a + 1) * MB / pm, n_lo = b * NB / pn, n_hi = (b + 1) * NB / pn;
        // blocks of 8 x 8 rectangles row by row, a Z-order curve inside each block
        for (int64_t bm = m_lo; bm < m_hi; bm += 8) {
          for (int64_t bnn = n_lo; bnn < n_hi; bnn += 8) {
            for (int code = 0; code < 64; ++code) {
              // even bits of the code: column offset, odd bits: row offset
              const int64_t dn = (code & 1) | ((code >> 1) & 2) | ((code >> 2) & 4);
              const int64_t dm = ((code >> 1) & 1) | ((code >> 2) & 2) | ((code >> 3) & 4);
              if (bm + dm >= m_hi || bnn + dn >= n_hi) continue;
              const int64_t rect = (bm + dm) * NB + (bnn + dn);
              for (int64_t ks = 0; ks < S; ++ks) lists[die].push_back((uint32_t)(out.first[i] + rect * S + ks));
            }
          }
        }
      }
    }
  }
  for (int x = 0; x < 8; ++x) {
    out.xoff[x] = (uint32_t)out.xorder.size();
    out.xorder.insert(out.xorder.end(), lists[x].begin(), lists[x].end());
  }
  out.xoff[8] = (uint32_t)out.xorder.size();
}

// Whether the outputs of the plan's tiles go past the caches.  The launch itself gains by that (up to 10 % where it finds operands of its
// own in the caches, as on a relaunch), the launch that reads the outputs loses where they would have been there for it, and in a launch
// beyond the 256 MB last-level cache most of what it writes is gone when it ends.  Pairs and triples of layers that read each other's
// outputs in turn, us, in the caches / past them: sixteen 1024-cubed products (101 MB a launch) 88 / 102, four layers of 128 rows from 768 to 3072 and
// back 36.8 / 40.9, 16 bottlenecks of 14x14x1024 49.8 / 52.5, 3x3 56x56x64 x128 (112 MB) 88.0 / 92.4, 64 bottlenecks of 56x56x256
// (131 MB) 95.0 / 98.2, channel-major 3x3 28x28x128 x64 122.7 / 130.8; above the line 3x3 28x28x128 x256 (178 MB) 175.9 / 168.2, bottlenecks 56x56x256 x96 (196
// MB) 132.5 / 129.4, x256 329 / 307, 3x3 56x56x64 x512 269 / 263 (but x256, 224 MB of which half are outputs, 136 / 144).
static bool past_caches(const HostPlan &hp) {
  constexpr double LINE = 160.0 * 1024 * 1024;
  double bytes = 0;
  for (size_t i = 0; i < hp.dev.size(); ++i) {
    const DevProblem &d = hp.dev[i];
    const sk_problem &p = hp.problems[i];
    const double a = p.op == SK_GEMM ? (double)d.Mg * d.Kg : (double)p.Nb * p.H * p.Wd * p.Cin;
    bytes += elem_size(d.dtype) * (a + (double)d.Ng * d.Kg + (double)d.Mg * d.Ng);
  }
  return bytes > LINE;
}

static void mark_rows(HostPlan &hp);

sk_status plan_host(const sk_problem *problems, int32_t n, const sk_plan_params *params, HostPlan &out,
                    std::string &err) {
  if (n < 0 || (n > 0 && !problems)) {
    err = "problems is null or n < 0";
    return SK_ERR_INVALID_ARG;
  }
  sk_plan_params prm;
  if (params)
    prm = *params;
  else
    sk_plan_params_default(&prm);
  if (prm.skinny_max_m < 0 || prm.skinny_max_m > 64 || prm.tile_bytes_min < 1 ||
      prm.tile_bytes_max < prm.tile_bytes_min || prm.balance_div < 1 || prm.max_groups < 1 ||
      prm.max_groups > 256 || prm.grid_limit < 0 || prm.tail_div < 0 || prm.xcd_part < -1) {
    err = "sk_plan_params field out of range";
    return SK_ERR_INVALID_ARG;
  }
  out = HostPlan{};
  out.params = prm;
  out.problems.assign(problems, problems + n);
  out.dev.resize(n);
  out.first.assign(n, 0);
  out.count.assign(n, 0);

  // ---- canonical view, operand strides, vector-access flags ----
  std::vector<Canon> canon(n);
  int64_t total_w = 0;
  for (int32_t i = 0; i < n; ++i) {
    const sk_problem &p = out.problems[i];
    sk_status st = canonicalise(p, i, canon[i], err);
    if (st != SK_OK) return st;
    const Canon &c = canon[i];
    const int es = elem_size(p.dtype);
    const int ce = 16 / es;  // elements per 16-byte piece
    DevProblem d;
    std::memset(&d, 0, sizeof(d));
    d.A = p.A;
    d.B = p.B;
    d.C = p.C;
    d.Mg = (int32_t)c.Mg;
    d.Ng = (int32_t)c.Ng;
    d.Kg = (int32_t)c.Kg;
    d.dtype = p.dtype;
    if (p.op == SK_GEMM) {
      d.lda = p.lda ? p.lda : p.K;
      d.ldb = p.ldb ? p.ldb : p.K;
      d.ldc = p.ldc ? p.ldc : p.N;
      d.gather = 0;
    } else {
      d.ldb = c.Kg;
      d.ldc = p.Cout;
      d.H = p.H;
      d.W = p.Wd;
      d.Cin = p.Cin;
      d.Ho = c.Ho;
      d.Wo = c.Wo;
      d.R = p.R;
      d.S = p.S;
      d.pad_h = p.pad_h;
      d.pad_w = p.pad_w;
      d.stride = p.stride ? p.stride : 1;
      // a 1x1 filter without padding or stride reads the image as a plain [pixels, Cin] matrix
      d.gather = !(p.R == 1 && p.S == 1 && p.pad_h == 0 && p.pad_w == 0 && d.stride == 1);
      d.lda = p.Cin;
      const FastDiv f_hw = fast_div_of((uint32_t)(c.Ho * c.Wo)), f_wo = fast_div_of((uint32_t)c.Wo);
      const FastDiv f_cin = fast_div_of((uint32_t)p.Cin), f_s = fast_div_of((uint32_t)p.S);
      d.div_hw[0] = f_hw.mul, d.div_hw[1] = f_hw.shift;
      d.div_wo[0] = f_wo.mul, d.div_wo[1] = f_wo.shift;
      d.div_cin[0] = f_cin.mul, d.div_cin[1] = f_cin.shift;
      d.div_s[0] = f_s.mul, d.div_s[1] = f_s.shift;
      if (p.op == SK_CONV2D_NCHW) {
        d.nchw = 1;
        d.gather = 1;  // neither a patch row nor an output row is contiguous in this storage order
      }
      const __int128 row = (__int128)(c.Ho - 1) * d.stride + p.R - 1, col = (__int128)(c.Wo - 1) * d.stride + p.S - 1;
      const __int128 reach = (d.nchw ? ((__int128)(p.Cin - 1) * p.H + row) * p.Wd + col + 1 : (row * p.Wd + col + 1) * p.Cin) * es;
      d.reach = (uint32_t)std::min<__int128>(reach, (__int128)1 << 31);
    }
    int32_t flags = 0;
    if (d.nchw) {
      // read element by element: no 16-byte pieces of the image along the reduction or along an output row
      // (the weights, one contiguous row per output channel in either order, may still be read in pieces)
    } else if (d.gather) {
      if (aligned16(p.A) && p.Cin % ce == 0) flags |= FLAG_VEC_A;
    } else {
      if (aligned16(p.A) && d.lda % ce == 0 && c.Kg % ce == 0) flags |= FLAG_VEC_A;
    }
    if (aligned16(p.B) && d.ldb % ce == 0 && c.Kg % ce == 0) flags |= FLAG_VEC_B;
    if (!d.nchw && (reinterpret_cast<uintptr_t>(p.C) % (4 * es)) == 0 && d.ldc % 4 == 0) flags |= FLAG_VEC_C;
    if (planes_form(d, es) && offsets_below(d, 0, es, (int64_t)1 << 31)) flags |= FLAG_PLANES_FORM;
    if (rows_form(d, es).ok) flags |= FLAG_ROWS_FORM;
    d.flags = flags;
    out.dev[i] = d;
    total_w += stream_bytes(c.Mg, c.Ng, c.Kg, es, prm);
  }

  // ---- output ranges must be pairwise disjoint ----
  {
    struct Range {
      uintptr_t lo, hi;
      int32_t idx;
    };
    std::vector<Range> r(n);
    for (int32_t i = 0; i < n; ++i) {
      const DevProblem &d = out.dev[i];
      const uintptr_t lo = reinterpret_cast<uintptr_t>(d.C);
      const uint64_t elems = (uint64_t)(d.Mg - 1) * (uint64_t)d.ldc + (uint64_t)d.Ng;
      r[i] = Range{lo, lo + elems * (uint64_t)elem_size(d.dtype), i};
    }
    std::sort(r.begin(), r.end(), [](const Range &a, const Range &b) { return a.lo < b.lo; });
    for (int32_t i = 1; i < n; ++i) {
      if (r[i].lo < r[i - 1].hi) {
        err = "output ranges of problems " + std::to_string(r[i - 1].idx) + " and " + std::to_string(r[i].idx) +
              " overlap";
        return SK_ERR_OVERLAP;
      }
    }
  }

  // ---- target operand bytes per tile ----
  int64_t T = total_w / prm.balance_div;
  T = std::max<int64_t>(prm.tile_bytes_min, std::min<int64_t>(prm.tile_bytes_max, T));
  if (n == 0) T = prm.tile_bytes_min;
  out.target_tile_bytes = T;

  // ---- operator order: earliest deadline first, ties by index ----
  out.order.resize(n);
  std::iota(out.order.begin(), out.order.end(), 0);
  if (prm.edf) {
    std::stable_sort(out.order.begin(), out.order.end(), [&](int32_t a, int32_t b) {
      return deadline_key(out.problems[a].deadline_ms) < deadline_key(out.problems[b].deadline_ms);
    });
  }

  // ---- stream bytes from each position of the order to its end ----
  std::vector<int64_t> remaining(n + 1, 0);
  for (int32_t pos = n - 1; pos >= 0; --pos) {
    const int32_t i = out.order[pos];
    remaining[pos] = remaining[pos + 1] + stream_bytes(canon[i].Mg, canon[i].Ng, canon[i].Kg, elem_size(out.problems[i].dtype), prm);
  }

  // ---- flat table ----
  const int64_t T_all = T;
  uint32_t out_id = 0;
  for (int32_t pos = 0; pos < n; ++pos) {
    const int32_t i = out.order[pos];
    const Canon &c = canon[i];
    const int es = elem_size(out.problems[i].dtype);
    // towards the end of the table the target shrinks with what is left to do
    T = T_all;
    // towards the end of the table the target shrinks with the bytes that remain, but not below eight
    // times the lower clamp (tiles of a few dozen KB are all fixed cost, and a reduction cut to match
    // them ends in dozens of slices)
    if (prm.tail_div > 0)
      T = std::min<int64_t>(T_all, std::max<int64_t>(8 * prm.tile_bytes_min, remaining[pos] / prm.tail_div));
    uint16_t cls;
    int64_t BM, BN;
    int64_t S = 1, slice_len = c.Kg;  // reduction slices per output rectangle and their length
    if (c.Mg <= prm.skinny_max_m) {
      const int rm_code = c.Mg <= 16 ? 0 : (c.Mg <= 32 ? 1 : 2);  // 1, 2 or 4 blocks of 16 activation rows
      const int64_t gb = 32 * c.Kg * es;                          // bytes of one 32-row weight group
      int64_t G;
      if (4 * gb <= T) {
        G = std::min<int64_t>(prm.max_groups, 4 * std::max<int64_t>(1, T / (4 * gb)));
      } else {
        // four groups already exceed the target: cut the reduction into slices of whole chunks
        G = 4;
        const int64_t chunk = (16384 / (16 << rm_code)) / es;  // reduction elements per activation chunk
        const int64_t nchunks = (c.Kg + chunk - 1) / chunk;
        int64_t want = std::min<int64_t>(std::min<int64_t>(nchunks, (4 * gb + T - 1) / T), 255);
        const int64_t per = (nchunks + want - 1) / want;
        S = (nchunks + per - 1) / per;
        slice_len = per * chunk;
      }
      cls = (uint16_t)(3 * rm_code);
      BM = c.Mg;
      BN = 32 * G;
    } else {
      // 128 output columns per tile, or 64 for an operator that has no more than that
      cls = c.Ng <= 64 ? CLS_TILE_128x64 : CLS_TILE_128x128;
      BM = 128;
      BN = c.Ng <= 64 ? 64 : 128;
      // operand bytes of one tile over the whole reduction; far beyond the target: cut the reduction
      const int64_t tb = (BM + BN) * c.Kg * es;
      if (tb > 2 * T) {
        const int64_t chunk = 256;  // reduction elements: whole stages of every element type
        const int64_t nchunks = (c.Kg + chunk - 1) / chunk;
        // a slice hands over 64 KB of partial sums: never shorter than 1024 reduction elements
        int64_t want = std::min<int64_t>(std::min<int64_t>(nchunks, (tb + T - 1) / T), 255);
        want = std::min<int64_t>(want, std::max<int64_t>(1, c.Kg / 1024));
        const int64_t per = (nchunks + want - 1) / want;
        S = (nchunks + per - 1) / per;
        slice_len = per * chunk;
      }
    }
    out.first[i] = (int64_t)out.tiles.size();
    for (int64_t m0 = 0; m0 < c.Mg; m0 += BM) {
      for (int64_t n0 = 0; n0 < c.Ng; n0 += BN) {
        for (int64_t ks = 0; ks < S; ++ks) {
          sk_tile t;
          t.problem = (uint32_t)i;
          t.cls = cls;
          t.ks_idx = (uint8_t)ks;
          t.S = (uint8_t)S;
          t.m0 = (uint32_t)m0;
          t.n0 = (uint32_t)n0;
          t.m_len = (uint16_t)std::min<int64_t>(BM, c.Mg - m0);
          t.n_len = (uint16_t)std::min<int64_t>(BN, c.Ng - n0);
          t.k0 = (uint32_t)(ks * slice_len);
          t.k_len = (uint32_t)std::min<int64_t>(slice_len, c.Kg - ks * slice_len);
          t.out_tile_id = out_id;
          out.tiles.push_back(t);
        }
        if (S > 1) {
          out.ws_off.push_back((uint32_t)out.ws_f32x4);
          out.ws_f32x4 += S * slice_f32x4(cls);
        } else {
          out.ws_off.push_back(0u);
        }
        ++out_id;
        if (out.tiles.size() > (size_t)1 << 30 || out.ws_f32x4 > ((int64_t)1 << 31)) {
          err = "tile table or split-K workspace too large";
          return SK_ERR_UNSUPPORTED;
        }
      }
    }
    out.count[i] = (int64_t)out.tiles.size() - out.first[i];
    out.dev[i].tile_first = (int32_t)out.first[i];
    out.dev[i].tile_count = (int32_t)out.count[i];
  }
  build_xcd_lists(out, canon);
  if (past_caches(out))
    for (DevProblem &d : out.dev) d.flags |= FLAG_PAST_CACHES;
  mark_rows(out);
  return SK_OK;
}

// A launch that fills a whole MI355X: two workgroups on each of its 256 compute units.
constexpr int64_t CHIP_WORKGROUPS = 512;

// What a record costs, in nanoseconds: `time` by itself on a compute unit, and `work`, its share of a compute unit that two
// workgroups keep busy.  Measured on plans of one kind of record each, 1 to 1024 of them, over 3 to 27 stages (fp32 blocks that
// read rows: 1.2 times that time, which is what they take among other records).  They decide which records are cut
// (refine_tiles) and nothing else.
struct RecordCost {
  int64_t time, work;
};

// Whether the blocks for operands of any alignment run the record (the weight-streaming classes read GEMMs at any address too,
// and convolutions with whole pieces under a tap).
static bool runs_in_any_blocks(const DevProblem &d, const sk_tile &t) {
  const int32_t vec = FLAG_VEC_A | FLAG_VEC_B;
  if ((d.flags & vec) == vec) return false;
  const int64_t ce = 16 / elem_size(d.dtype);
  return !(t.cls < CLS_TILE_128x128 && !d.nchw && d.Kg >= ce && (!d.gather || d.Cin % ce == 0));
}

static bool in_one_image(const DevProblem &d, const sk_tile &t) {
  const uint32_t hw = (uint32_t)(d.Ho * d.Wo);
  return hw == (uint32_t)d.Mg || t.m0 / hw == (t.m0 + t.m_len - 1) / hw;
}
// Whether run_tile_rows runs the record: an LDS tile, or a run of them, of an operator that rows_form takes (only such are marked), not split, in one image.
// (Only in plans where such operators are marked, mark_rows.  In others they are planned as blocks of any alignment, and cut like those; in 16-bit types
// the parts also run as those, rows_tile.)
static bool runs_in_rows(const DevProblem &d, const sk_tile &t) {
  if (!(d.flags & FLAG_ROWS) || t.cls < CLS_TILE_128x128 || t.cls == CLS_WINDOW || t.S != 1 || !runs_in_any_blocks(d, t)) return false;
  return in_one_image(d, t) && ((int64_t)t.m_len * t.n_len + 255) / 256 * d.Kg > 64;
}
// Whether b, which follows a, takes what a takes: records of an operator are mostly alike.  (Which tiles of several images lie in one is asked of
// each.)
static bool alike(const DevProblem &d, const sk_tile &a, const sk_tile &b) {
  return a.problem == b.problem && a.m_len == b.m_len && a.n_len == b.n_len && a.k_len == b.k_len && a.S == b.S &&
         (!(d.flags & FLAG_ROWS) || d.Mg == d.Ho * d.Wo);
}
// ... and what that takes, in nanoseconds on a compute unit that two workgroups share: around the blocks of 128 pixels, a block.  (One figure for all types:
// alone in a launch 1176 blocks of the 7x7 stem in bf16 take 28.2 us, 1568 of a 3x3 one in fp32 31.5.)
constexpr int64_t ROWS_START = 6000, ROWS_BLOCK = 3000;

// A record of m_len x n_len outputs in blocks of any alignment, `stages` of 128 bytes of the reduction.
static RecordCost any_block_cost(const DevProblem &d, int64_t m_len, int64_t n_len, int64_t stages) {
  const bool m64 = m_len <= 64, n64 = n_len <= 64;
  const int64_t blocks = (m64 ? 1 : (m_len + 127) / 128) * (n64 ? 1 : (n_len + 127) / 128);
  // per stage, [channel-major][fp32][128 x 128, 128 x 64, 64 x 128, 64 x 64]
  static const RecordCost per_stage[2][2][4] = {{{{1850, 1120}, {1560, 900}, {1300, 790}, {1200, 730}},
                                                 {{3700, 2630}, {2500, 1600}, {2300, 1540}, {1550, 930}}},
                                                {{{2500, 1900}, {2450, 1500}, {2250, 1400}, {1800, 1150}},
                                                 {{3500, 3050}, {2560, 1800}, {2250, 1700}, {1600, 1240}}}};
  const int shape = (m64 ? 2 : 0) + (n64 ? 1 : 0);
  const RecordCost &s = per_stage[d.nchw ? 1 : 0][d.dtype == SK_F32 ? 1 : 0][shape];
  const int64_t start = shape == 0 ? 8000 : shape == 3 ? 5000 : 7000;  // set-up, first loads and outputs
  return RecordCost{blocks * (start + stages * s.time), blocks * (start / 2 + stages * s.work)};
}

static RecordCost record_cost(const DevProblem &d, const sk_tile &t) {
  const int64_t es = elem_size(d.dtype), kb = 128 / es, stages = ((int64_t)t.k_len + kb - 1) / kb;
  const bool f32 = d.dtype == SK_F32;
  if (runs_in_rows(d, t)) {
    const int64_t blocks = (t.m_len + 127) / 128;
    return RecordCost{ROWS_START + blocks * ROWS_BLOCK, ROWS_START / 2 + blocks * ROWS_BLOCK / 2};
  }
  if (runs_in_any_blocks(d, t)) return any_block_cost(d, t.m_len, t.n_len, stages);
  if (t.cls < CLS_TILE_128x128) {
    const int64_t steps = stages * ((t.n_len + 127) / 128);
    const bool rows64 = t.cls >= 6;
    return RecordCost{4000 + steps * (rows64 ? (f32 ? 1450 : 800) : 600), 2500 + steps * (rows64 ? (f32 ? 1200 : 720) : 620)};
  }
  if (t.cls == CLS_TILE_128x64) return RecordCost{4000 + stages * (f32 ? 1100 : 600), 2500 + stages * (f32 ? 820 : 650)};
  return RecordCost{5000 + stages * (f32 ? 2000 : 700), 2500 + stages * (f32 ? 1800 : 1000)};
}

// The work of all records; `rows`: of those that run_tile_rows runs.
static int64_t work_of(const HostPlan &hp, const std::vector<sk_tile> &records, int64_t *rows) {
  int64_t total = 0, of_rows = 0, work = 0;
  bool in_rows = false;
  const sk_tile *last = nullptr;
  for (const sk_tile &t : records) {
    const DevProblem &d = hp.dev[t.problem];
    if (!last || !alike(d, *last, t)) {
      work = record_cost(d, t).work;
      in_rows = runs_in_rows(d, t);
    }
    last = &t;
    total += work;
    if (in_rows) of_rows += work;
  }
  if (rows) *rows = of_rows;
  return total;
}

// A launch lasts at least as long as its longest record, and as long as the work of all records spread over the compute
// units.  Where a record without 16-byte pieces is what it would wait for, such records are cut into parts of at most 64 x 64
// outputs.  A part takes 0.4 (fp32) to 0.7 (16-bit types) of the time of a 128 x 128 block, but the parts together 1.4 to 2.6
// times its work, so nothing is cut where the launch waits for a record that cannot be cut, or fills the chip anyway.
// Measured, all records beyond an even share cut against none: stride-2 layers with the stem for two tenants 38.0 and 32.9 us, for
// four 55.9 and 49.4, channel-major ResNet layers for eight 151 and 145, in fp32 for two 218 and 164.
// Which records are cut where it pays:
//   * 16-bit types: those that take 0.6 of what the launch lasts with the longest cut.  In a plan whose records all start at
//     once the parts do too if those of the records that outlast the rest can: then as many others are cut,
//     the longest first, as there are workgroups left.  (60 odd bf16 operators 49 us with none cut, 44 with all beyond
//     an even share, 33 so.)
//   * fp32 among them: all beyond an even share of the stages over the workgroups.  Blocks that keep the matrix cores busy
//     slow down whoever shares their compute unit, so the shorter ones are worth cutting as well (96 operators in
//     three types 208 us with none cut, 134 so; the rule for 16-bit types takes 80 to 135 % of the time of this
//     one on plans of 20 to 96 odd fp32 operators).
// Slices of split reductions stay whole (their workspace is laid out by rectangle), and so do plans with per-die
// lists, which name the table's records.  The sums of an output do not change.
static bool refine_blocks(const HostPlan &hp, int64_t workgroups, std::vector<sk_tile> &work, std::vector<int64_t> &count) {
  if (workgroups < 1) return false;
  const int32_t vec = FLAG_VEC_A | FLAG_VEC_B;
  if (std::all_of(hp.dev.begin(), hp.dev.end(), [&](const DevProblem &d) { return (d.flags & vec) == vec; })) return false;
  auto parts_of = [](const sk_tile &t) { return ((t.m_len + 63) / 64) * ((t.n_len + 63) / 64); };
  auto stages_of = [&](const sk_tile &t) -> int64_t {  // 128 bytes of the reduction each; twice for fp32, over all 128 x 128 blocks
    const int64_t es = elem_size(hp.dev[t.problem].dtype), kb = 128 / es;
    return ((t.k_len + kb - 1) / kb) * ((t.m_len + 127) / 128) * ((t.n_len + 127) / 128) * (es == 4 ? 2 : 1);
  };
  // time of every record that can be cut, 0 for the others
  std::vector<int64_t> time(hp.tiles.size(), 0);
  int64_t longest = 0, whole = 0, part = 0, total = 0;  // cuttable; not cuttable; a part of the longest; work of all
  int64_t stages = 0;                                   // of all records in such blocks
  bool fp32 = false;                                    // one of those that can be cut is
  RecordCost c{0, 0};
  int64_t steps = 0;
  bool any = false, rows = false;
  for (size_t i = 0; i < hp.tiles.size(); ++i) {
    const sk_tile &t = hp.tiles[i];
    const DevProblem &d = hp.dev[t.problem];
    if (i == 0 || !alike(d, hp.tiles[i - 1], t)) {
      c = record_cost(d, t);
      any = runs_in_any_blocks(d, t);
      rows = runs_in_rows(d, t);
      steps = any ? stages_of(t) : 0;
    }
    total += c.work;
    stages += steps;
    // (up to 64 reduction elements a small rectangle may go the one-output-per-thread way, whose sums round differently: a
    // part must not where its record does not)
    if (t.S != 1 || (t.m_len <= 64 && t.n_len <= 64) || d.Kg <= 64 || !any || rows) {
      whole = std::max(whole, c.time);
      continue;
    }
    time[i] = c.time;
    fp32 = fp32 || d.dtype == SK_F32;
    if (c.time > longest) {
      longest = c.time;
      const int64_t kb = 128 / elem_size(d.dtype);
      part = any_block_cost(d, 64, 64, ((int64_t)t.k_len + kb - 1) / kb).time;
    }
  }
  const int64_t length = std::max(std::max(whole, part), 2 * total / workgroups);  // (two workgroups per compute unit)
  if (longest * 32 <= length * 33) return false;
  int64_t from = length * 6 / 10;  // 16-bit types: the time from which records are cut
  if (!fp32 && (int64_t)hp.tiles.size() <= workgroups) {
    std::vector<std::pair<int64_t, int64_t>> more;  // records that need not be cut, by how many records their parts are more
    int64_t all = (int64_t)hp.tiles.size(), least = all;
    for (size_t i = 0; i < hp.tiles.size(); ++i) {
      if (time[i] < from || time[i] == 0) continue;
      const int64_t n = parts_of(hp.tiles[i]) - 1;
      all += n;
      if (time[i] > length)
        least += n;
      else
        more.emplace_back(time[i], n);
    }
    if (all > workgroups && least <= workgroups) {
      std::sort(more.begin(), more.end(), std::greater<std::pair<int64_t, int64_t>>());
      for (const auto &m : more) {
        least += m.second;
        if (least > workgroups) {
          from = m.first + 1;
          break;
        }
      }
    }
  }
  work.clear();
  count.assign(hp.dev.size(), 0);
  for (size_t i = 0; i < hp.tiles.size(); ++i) {
    const sk_tile &t = hp.tiles[i];
    const bool c = time[i] > 0 && (fp32 ? stages_of(t) * workgroups > stages : time[i] >= from);
    const uint32_t bm = c ? 64u : t.m_len, bn = c ? 64u : t.n_len;
    for (uint32_t m = 0; m < t.m_len; m += bm)
      for (uint32_t n = 0; n < t.n_len; n += bn) {
        sk_tile u = t;
        u.m0 = t.m0 + m;
        u.n0 = t.n0 + n;
        u.m_len = (uint16_t)std::min<uint32_t>(bm, t.m_len - m);
        u.n_len = (uint16_t)std::min<uint32_t>(bn, t.n_len - n);
        work.push_back(u);
        ++count[t.problem];
      }
  }
  return true;
}

bool refine_tiles(const HostPlan &hp, int64_t workgroups, std::vector<sk_tile> &work, std::vector<int64_t> &count) {
  return hp.xorder.empty() && refine_blocks(hp, workgroups, work, count);
}

// Marks the operators that run_tile_rows serves where they are a fifth of the work of a plan of one element type.  (In the kernels for mixed types, which
// spill more scalars than any, it gains nothing: three plans of 70 to 95 operators in three types, a fifth to a quarter of their work such, took 4 to 7 %
// longer planned by its times.)
// (Nor in plans of less than two rounds of tiles, where runs leave too few records to even the launch's end out: 67 odd bf16 operators 35.9 -> 37.5 us, 30
// of them 29.4 -> 30.4, ten such plans 0.97 to 1.02; stride-2 layers for five, 885 tiles, would gain 3 %, for six, 1062 tiles, 10 %.)
static void mark_rows(HostPlan &hp) {
  if ((int64_t)hp.tiles.size() <= 2 * CHIP_WORKGROUPS) return;
  for (const DevProblem &d : hp.dev)
    if (d.dtype != hp.dev[0].dtype) return;
  for (DevProblem &d : hp.dev)
    if (d.flags & FLAG_ROWS_FORM) d.flags |= FLAG_ROWS, hp.rows = true;
  if (!hp.rows) return;
  int64_t rows = 0;
  const int64_t total = work_of(hp, hp.tiles, &rows);
  if (rows * 5 < total) {
    for (DevProblem &d : hp.dev) d.flags &= ~FLAG_ROWS;
    hp.rows = false;
  }
}

// What a record takes on a chip whose compute units hold two workgroups each, in nanoseconds: `start` around its steps (set-up, first
// loads, outputs, the next record), `step` per 128 bytes of the reduction, `hand` more if it hands partial sums over.  Means of clock
// stamps at the phase boundaries of the ResNet, BERT, stride-2 and odd-sized mixes.
struct RecordTime {
  int64_t start, step, hand;
};
// Runs of pixels (CLS_WINDOW): around their steps, and a step of 128 pixels.
constexpr int64_t WINDOW_START = 6000, WINDOW_STEP = 3000;
static RecordTime record_time(const DevProblem &d, const sk_tile &t, bool any) {
  const bool f32 = d.dtype == SK_F32;
  if (any && runs_in_rows(d, t)) return RecordTime{ROWS_START + (t.m_len + 127) / 128 * ROWS_BLOCK, 0, 0};
  if (any) {
    const int64_t one = any_block_cost(d, t.m_len, t.n_len, 1).time, step = any_block_cost(d, t.m_len, t.n_len, 2).time - one;
    return RecordTime{one - step, f32 ? step * 13 / 10 : step, 8000};
  }
  if (t.cls < CLS_TILE_128x128) return RecordTime{4500, f32 && t.cls >= 6 ? 2000 : 1100, 3000};
  if (t.cls == CLS_WINDOW) return RecordTime{WINDOW_START + (t.m_len + 127) / 128 * WINDOW_STEP, 0, 0};
  if (t.cls == CLS_TILE_128x64) return RecordTime{5000, f32 ? 1700 : 650, 4000};
  return RecordTime{6000, f32 ? 3400 : 950, 5000};
}

// The table is cut by bytes and ordered by deadline; how long its records take, and that the last of them end together, is
// settled here, for the device's list alone.  Stamped ends of the workgroups before: ResNet layers x16 41 to 78 us after the start,
// channel-major ones x8 23 to 135, 96 odd-sized operators 11 to 128, BERT layers x8 127 to 170.
//   * Operators of one deadline (all that have none) have no order among them that anyone asked for: those with the longest
//     records go first, so that the launch ends on short ones.  Whole operators move, so their tiles still meet in the L2s.
//   * A record longer than its share is cut: weight-streaming ones by columns (nothing but one more start per part; half a
//     workgroup's share of the whole launch: LSTM cells 64 230 -> 215 us, a quarter no better; not those of
//     operators with deadlines, which run where the table puts them and shrink towards its end: 52 mixed operators 215 -> 217), the others, if they outlast an
//     even share by a quarter (LDS tiles of 16-bit types: twice that share, a compute unit's that runs one of them at a time: six 45x45 convolutions of
//     256 channels 35.7 us whole, 43.7 in two slices), into equal slices of the reduction, as many as
//     slices that take an even share, and of 16 stages or more (blocks of any alignment eight), cover it: 36 stages 12/12/12, 40 stages 16/16/8, 17 stages
//     12/5.  All but the last have twelve stages (eight) at least, because a slice writes its
//     sums to memory and the last one reads all of them (in slices of 6 stages eleven 20x20 convolutions of 192 channels 24.7 -> 32.6 us, by this
//     rule 24.5).  Holding every slice to 16 (six) by making fewer is slower: nine 14x14 convolutions of 256 channels 19.9 -> 22.7,
//     three 18.3 -> 21.1, twenty 23.2 -> 24.4, 96 odd-sized operators 69 -> 83.  Weight-streaming records are not sliced any further: 16 low-batch layers 32 -> 39 us.
//   * Nothing is cut below 14 us: 10 and 18 measure the same.
// Before / after, us: channel-major ResNet layers x8 140 -> 96, odd-sized operators 134 -> 73, ResNet layers x16 80 -> 70, x3 34 -> 28,
// BERT layers x8 173 -> 156, stride-2 layers x3 43 -> 33; mixes whose operators all have deadlines of their own as before.
// Slices change the order of summation with the load of the launch, so plans without the tail rule, whose tiles may not depend on what
// else is in the plan, get none.  Plans with per-die lists get the same slices as without (the bits of a result do not depend on who
// runs a tile) and stay otherwise as they are.  Nor do they depend on the number of workgroups: `impose` names the slices of a launch that
// fills a whole MI355X (null: this is that launch, they are settled here).
// (`slices_only`: out.slicing is all that is wanted of the list.)
static bool balance_records(const HostPlan &hp, const std::vector<sk_tile> &records, int64_t workgroups, bool drop_lists,
                            const std::vector<Slicing> *impose, WorkList &out, bool slices_only = false) {
  constexpr int64_t SHORTEST = 14000;
  if (workgroups < 1 || records.empty()) return false;
  const bool lists = !hp.xorder.empty() && !drop_lists;
  const int32_t vec = FLAG_VEC_A | FLAG_VEC_B;
  // an output rectangle of the table: its records (reduction slices, or parts that refine_tiles has made), and how they are cut
  struct Rect {
    size_t first, count;
    int64_t time;             // of the longest of them
    int64_t width, S, slice;  // columns and reduction slices of a part, reduction elements per slice
  };
  struct Op {
    int32_t problem;
    size_t first, count;  // records
    int64_t longest;
    size_t rect, rects;  // of an operator with a record that may be cut
    bool sliced;         // slices imposed
  };
  std::vector<Rect> rects;
  std::vector<Op> ops;
  ops.reserve(hp.dev.size());
  auto any_of = [&](const sk_tile &t) { return runs_in_any_blocks(hp.dev[t.problem], t); };
  auto stages_of = [&](const sk_tile &t) -> int64_t {  // (shifts: this runs for every record)
    return hp.dev[t.problem].dtype == SK_F32 ? ((int64_t)t.k_len + 31) >> 5 : ((int64_t)t.k_len + 63) >> 6;
  };
  auto columns_of = [](const sk_tile &t, bool any) -> int64_t {  // blocks of 128 that a weight-streaming record walks one after the other
    return t.cls < CLS_TILE_128x128 && !any ? (t.n_len + 127) / 128 : 1;
  };
  auto time_of = [&](const sk_tile &t) {
    const bool any = any_of(t);
    const RecordTime rt = record_time(hp.dev[t.problem], t, any);
    return rt.start + stages_of(t) * columns_of(t, any) * rt.step + (t.S > 1 ? rt.hand : 0);
  };
  auto imposed = [&](const sk_tile &t) { return impose && t.out_tile_id < impose->size() ? (*impose)[t.out_tile_id] : Slicing{}; };
  auto alike = [](const sk_tile &a, const sk_tile &b) { return a.m_len == b.m_len && a.n_len == b.n_len && a.k_len == b.k_len && a.S == b.S; };
  int64_t total = 0;
  for (size_t i = 0; i < records.size();) {
    Op op{(int32_t)records[i].problem, i, 0, 0, 0, 0, false};
    int64_t time = 0;
    const sk_tile *timed = nullptr;  // (an operator's records are mostly alike)
    for (; i < records.size() && records[i].problem == (uint32_t)op.problem; ++i) {
      if (!timed || !alike(*timed, records[i])) {
        timed = &records[i];
        time = time_of(*timed);
        op.longest = std::max(op.longest, time);
      }
      total += time;
      op.sliced = op.sliced || imposed(records[i]).S > 0;
    }
    op.count = i - op.first;
    ops.push_back(op);
  }
  const int64_t share = total / workgroups;

  bool changed = false;
  std::vector<Slicing> slicing;
  auto slice_anew = [&](const sk_tile &t, const Rect &x) {
    if (slicing.size() <= t.out_tile_id) slicing.resize(t.out_tile_id + 1);
    slicing[t.out_tile_id] = Slicing{x.S, x.slice};
  };
  for (Op &op : ops) {
    if (op.longest * 10 <= std::max(SHORTEST, share / 2) * 11 && !op.sliced) continue;
    const bool dated = hp.params.edf && std::isfinite(deadline_key(hp.problems[op.problem].deadline_ms));
    op.rect = rects.size();
    const sk_tile *timed = nullptr;
    int64_t time = 0;
    for (size_t i = op.first; i < op.first + op.count; ++i) {
      const sk_tile &t = records[i];
      if (!timed || !alike(*timed, t)) {
        timed = &t;
        time = time_of(t);
      }
      if (i == op.first || t.out_tile_id != records[i - 1].out_tile_id) rects.push_back(Rect{i, 0, 0, t.n_len, t.S, t.k_len});
      Rect &x = rects.back();
      ++x.count;
      x.time = std::max(x.time, time);
      x.width = std::max<int64_t>(x.width, t.n_len);
    }
    op.rects = rects.size() - op.rect;
    op.longest = 0;
    const Rect *last = nullptr;  // the rectangle before, settled, and what its time was
    int64_t last_time = 0;
    for (size_t r = op.rect; r < op.rect + op.rects; ++r) {
      Rect &x = rects[r];
      const sk_tile &t = records[x.first];
      if (last && !impose && last_time == x.time && alike(records[last->first], t)) {  // settled alike
        x.time = last->time;
        x.width = std::min(x.width, last->width);
        x.S = last->S;
        x.slice = last->slice;
        if (x.S != t.S) slice_anew(t, x);
        last = &x;
        continue;
      }
      last = &x;
      last_time = x.time;
      const DevProblem &d = hp.dev[t.problem];
      const bool any = any_of(t), stream = !any && t.cls < CLS_TILE_128x128;
      const int64_t most = std::max<int64_t>(SHORTEST, stream ? share / 2 : any || d.dtype == SK_F32 ? share * 5 / 4 : share * 2);
      if (const Slicing given = imposed(t); given.S > 0) {
        const RecordTime rt = record_time(d, t, any);
        const int64_t kb = 128 / elem_size(d.dtype);
        x.S = given.S;
        x.slice = given.slice;
        x.width = std::min<int64_t>(x.width, 128);  // (a slice of a record without 16-byte pieces must be a single block)
        x.time = rt.start + (given.slice + kb - 1) / kb * rt.step + rt.hand;
        changed = true;
        op.longest = std::max(op.longest, x.time);
        continue;
      }
      // (up to 64 reduction elements an operator without 16-byte pieces may go the one-output-per-thread way, by the size of its record)
      if (x.time * 10 > most * 11 && ((d.flags & vec) == vec || d.Kg > 64)) {
        const RecordTime rt = record_time(d, t, any);
        if (stream) {
          const int64_t cols = columns_of(t, any);
          if (t.S == 1 && cols > 1 && !lists && !dated) {
            const int64_t parts = std::min(cols, (cols * stages_of(t) * rt.step + most - rt.start - 1) / (most - rt.start));
            const int64_t wide = (cols + parts - 1) / parts;
            x.width = wide * 128;
            x.time = rt.start + stages_of(t) * wide * rt.step;
            changed = changed || x.width < t.n_len;
          }
        } else if (!impose && rt.step > 0 && hp.params.tail_div > 0 && t.m_len <= 128 && t.n_len <= 128) {
          // (a step of no time: a run of pixels or of tiles, timed by its pixels; never sliced)
          constexpr int64_t GRAIN = 4;  // stages
          const int64_t kb = 128 / elem_size(d.dtype), k = t.S > 1 ? d.Kg : (int64_t)t.k_len, all = (k + kb - 1) / kb;
          const int64_t fits = (std::max<int64_t>((most - rt.start - rt.hand) / rt.step, any ? 8 : 16) + GRAIN - 1) / GRAIN * GRAIN;
          const int64_t want = std::min<int64_t>((all + fits - 1) / fits, 255);
          const int64_t per = ((all + want - 1) / want + GRAIN - 1) / GRAIN * GRAIN, n = (all + per - 1) / per;
          const int64_t time = rt.start + per * rt.step + rt.hand;
          if (n > t.S && time * 10 < x.time * 8) {
            x.S = n;
            x.slice = per * kb;
            x.time = time;
            changed = true;
            slice_anew(t, x);
          }
        }
      }
      op.longest = std::max(op.longest, x.time);
    }
  }
  if (slices_only) {
    out.slicing = std::move(slicing);
    return changed;
  }
  if (hp.params.edf && !lists) {
    auto before = [&](const Op &a, const Op &b) {
      const double da = deadline_key(hp.problems[a.problem].deadline_ms), db = deadline_key(hp.problems[b.problem].deadline_ms);
      return da != db ? da < db : a.longest > b.longest;
    };
    if (!std::is_sorted(ops.begin(), ops.end(), before)) {
      std::stable_sort(ops.begin(), ops.end(), before);
      changed = true;
    }
  }
  if (!changed) return false;

  out = WorkList{};
  out.work.reserve(records.size() + records.size() / 4);
  out.ws_off.reserve(records.size());
  out.count.assign(hp.dev.size(), 0);
  out.slicing = std::move(slicing);
  auto new_rect = [&](const sk_tile &t, int64_t S) {
    out.ws_off.push_back(S > 1 ? (uint32_t)out.ws_f32x4 : 0u);
    if (S > 1) out.ws_f32x4 += S * slice_f32x4(t.cls);
  };
  // records as they are
  auto copy = [&](const std::vector<sk_tile> &from, size_t first, size_t n) {
    const size_t at = out.work.size();
    out.work.insert(out.work.end(), from.begin() + (int64_t)first, from.begin() + (int64_t)(first + n));
    for (size_t i = 0; i < n; ++i) {
      const sk_tile &t = from[first + i];
      if (i == 0 || t.out_tile_id != from[first + i - 1].out_tile_id) new_rect(t, t.S);
      out.work[at + i].out_tile_id = (uint32_t)out.ws_off.size() - 1u;
    }
    if (n) out.count[from[first].problem] += (int64_t)n;
  };
  // columns of t, `width` at a time, in the slices of x
  auto emit = [&](const sk_tile &t, const Rect &x, int64_t width) {
    const int64_t k = t.S > 1 ? hp.dev[t.problem].Kg : (int64_t)t.k_len;
    for (int64_t n = 0; n < t.n_len; n += width) {
      new_rect(t, x.S);
      for (int64_t ks = 0; ks < x.S; ++ks) {
        sk_tile u = t;
        u.S = (uint8_t)x.S;
        u.ks_idx = (uint8_t)ks;
        u.k0 = (uint32_t)(ks * x.slice);
        u.k_len = (uint32_t)std::min<int64_t>(x.slice, k - ks * x.slice);
        u.n0 = t.n0 + (uint32_t)n;
        u.n_len = (uint16_t)std::min<int64_t>(width, t.n_len - n);
        u.out_tile_id = (uint32_t)out.ws_off.size() - 1u;
        out.work.push_back(u);
        ++out.count[t.problem];
      }
    }
  };
  if (!lists) {
    for (const Op &op : ops) {
      if (op.rects == 0) copy(records, op.first, op.count);
      for (size_t r = op.rect; r < op.rect + op.rects; ++r) {
        const Rect &x = rects[r];
        const sk_tile &t = records[x.first];
        if (x.S == t.S && x.width >= t.n_len)
          copy(records, x.first, x.count);
        else
          for (size_t i = x.first; i < x.first + x.count; i += records[i].S) emit(records[i], x, x.width);
      }
    }
  } else {
    std::vector<uint32_t> at(hp.tiles.size() + 1);  // where a table record's slices start in the list
    size_t i = 0;  // table record; the operators and their rectangles are in the table's order
    for (const Op &op : ops) {
      const size_t end = i + (size_t)hp.count[(size_t)op.problem];
      for (size_t r = op.rect; i < end; ++r) {
        const sk_tile &t = hp.tiles[i];
        const Rect *x = op.rects ? &rects[r] : nullptr;
        for (int64_t ks = 0; ks < t.S; ++ks) at[i + (size_t)ks] = (uint32_t)(out.work.size() + (x && x->S != t.S ? 0 : (size_t)ks));
        if (x && x->S != t.S)
          emit(t, *x, 128);  // (a slice of a record without 16-byte pieces must be a single block)
        else
          copy(hp.tiles, i, t.S);
        i += t.S;
      }
    }
    at[hp.tiles.size()] = (uint32_t)out.work.size();
    for (int die = 0; die < 8; ++die) {
      out.xoff[die] = (uint32_t)out.xorder.size();
      for (uint32_t e = hp.xoff[die]; e < hp.xoff[die + 1]; ++e) {
        const sk_tile &t = hp.tiles[hp.xorder[e]];
        if (t.ks_idx != 0) continue;
        const uint32_t from = at[hp.xorder[e]], to = at[hp.xorder[e] + t.S];
        for (uint32_t w = from; w < to; ++w) out.xorder.push_back(w);
      }
    }
    out.xoff[8] = (uint32_t)out.xorder.size();
  }
  return out.work.size() <= (size_t)1 << 30 && out.ws_f32x4 <= ((int64_t)1 << 31);
}

// Whether run_window serves the operator: a size-keeping 3x3 NHWC convolution of 64 channels of 16 bits into at most 64, of images
// whose rows its ring takes, and whose tiles are 128 x 64 LDS tiles.
bool window_operator(const HostPlan &hp, size_t i) {
  const DevProblem &d = hp.dev[i];
  const int32_t vec = FLAG_VEC_A | FLAG_VEC_B;
  if (d.dtype == SK_F32 || !d.gather || d.nchw || d.stride != 1 || d.R != 3 || d.S != 3 || d.pad_h != 1 || d.pad_w != 1 || d.Cin != 64 ||
      d.Ng > 64 || d.Ng % 8 != 0 || d.W > 63 || (d.flags & vec) != vec || !aligned16(d.C))
    return false;
  const sk_tile &t = hp.tiles[(size_t)hp.first[i]];
  return t.cls == CLS_TILE_128x64 && t.S == 1;
}

// The order of the operators means something.
static bool several_deadlines(const HostPlan &hp) {
  return hp.params.edf && std::any_of(hp.problems.begin(), hp.problems.end(), [&](const sk_problem &p) {
    return deadline_key(p.deadline_ms) != deadline_key(hp.problems[0].deadline_ms);
  });
}

// The table with such operators' tiles replaced by runs of pixels; false: none.
// Only where the tiles are more than the workgroups: with a tile for each at most, a run is a single block of 128 pixels, and its
// start (weights to registers, 36 loads a wave) is what it takes.  500 tiles of 56x56 images 18.8 us as tiles, 20.0 as runs; 525 tiles, a second
// round for some workgroups, 20.3 and 18.6, 1600 tiles 37.5 and 28.6, 12800 tiles 214 and 124.
// How long a run is: in a plan of nothing else, what takes the fewest steps over the rounds of runs; beside other operators, half
// a workgroup's share of the launch, as for weight streaming.
// In a plan of several deadlines a run is a fifth of a share at most, so that the first deadlines' operators are not done with the launch's
// middle, and where that is less than three steps (of a plan of nothing else: with a share of less than twelve) the tiles stay.  512 operators
// of 56x56 with deadlines of their own, us until the first tenth of them in that order are done, all of them in the mean, the
// last: as tiles 28.6, 122.9 and 223.8, in the longest runs 90.8, 102.1 and 132.8, in a fifth of a share 28.6, 86.3 and 142.7 (a third 34.8 in the first place, a sixth
// and an eighth 99 and 100 in the mean); 256: 23.9, 63.6 and 105.8, 50.4, 56.5 and 65.3, three steps 22.8, 57.7 and 90.9; 128: 16.1, 37.5 and 62.2, 34.2, 37.8 and 43.8.
bool window_records(const HostPlan &hp, int64_t workgroups, std::vector<sk_tile> &records, std::vector<int64_t> &count) {
  constexpr int64_t STEP = 128, START = 3, MOST = 500;  // pixels; steps that a start costs; steps of a run (its pixels fit 16 bits)
  constexpr int64_t DATED_LEAST = 3;
  if (workgroups < 1 || (int64_t)hp.tiles.size() <= workgroups) return false;
  std::vector<char> window(hp.dev.size(), 0);
  bool some = false, all = true;
  for (size_t i = 0; i < hp.dev.size(); ++i) {
    if (hp.dev[i].dtype != hp.dev[0].dtype || (hp.dev[i].flags & (FLAG_VEC_A | FLAG_VEC_B)) != (FLAG_VEC_A | FLAG_VEC_B)) return false;
    window[i] = window_operator(hp, i);
    some = some || window[i];
    all = all && window[i];
  }
  // (the per-die lists of other operators name tiles of the table; lists that the caller has asked for are kept: only the planner's own give
  // way)
  if (!some || (!hp.xorder.empty() && (!all || hp.params.xcd_part > 0))) return false;
  const bool dated = several_deadlines(hp);
  auto steps_of = [&](size_t i) { return (hp.dev[i].Mg + STEP - 1) / STEP; };
  int64_t per = MOST;
  if (all && dated) {
    int64_t steps = 0;
    for (size_t i = 0; i < hp.dev.size(); ++i) steps += steps_of(i);
    if (steps / workgroups < 4 * DATED_LEAST) return false;
    per = std::min(MOST, std::max(DATED_LEAST, steps / workgroups / 5));
  } else if (all) {
    int64_t best = 0, longest = 1;
    for (size_t i = 0; i < hp.dev.size(); ++i) longest = std::max<int64_t>(longest, steps_of(i));
    for (int64_t len = std::min(longest, MOST); len >= 1; len = len > 8 ? len * 7 / 8 : len - 1) {
      int64_t n = 0, most = 0;
      for (size_t i = 0; i < hp.dev.size(); ++i) {
        const int64_t parts = (steps_of(i) + len - 1) / len;
        n += parts;
        most = std::max(most, (steps_of(i) + parts - 1) / parts);
      }
      const int64_t time = (n + workgroups - 1) / workgroups * (most + START);
      if (best == 0 || time < best) best = time, per = len;
    }
  } else {
    int64_t total = 0;
    for (size_t i = 0; i < hp.dev.size(); ++i) {
      if (window[i]) {
        total += steps_of(i) * WINDOW_STEP;
        continue;
      }
      const sk_tile &t = hp.tiles[(size_t)hp.first[i]];  // (its first record is its largest)
      const RecordTime rt = record_time(hp.dev[i], t, false);
      const int64_t kb = 128 / elem_size(hp.dev[i].dtype), cols = t.cls < CLS_TILE_128x128 ? (t.n_len + 127) / 128 : 1;
      total += hp.count[i] * (rt.start + (t.k_len + kb - 1) / kb * cols * rt.step);
    }
    per = std::max<int64_t>(2, std::min(MOST, (total / workgroups / (dated ? 5 : 2) - WINDOW_START) / WINDOW_STEP));
    if (dated && per < DATED_LEAST) return false;
  }
  records.clear();
  records.reserve(hp.tiles.size());  // (there are fewer runs than tiles)
  count.assign(hp.dev.size(), 0);
  uint32_t id = 0x80000000u;  // (rectangles are numbered anew later; here they only have to differ)
  for (const int32_t o : hp.order) {
    const size_t i = (size_t)o;
    if (!window[i]) {
      records.insert(records.end(), hp.tiles.begin() + hp.first[i], hp.tiles.begin() + hp.first[i] + hp.count[i]);
      count[i] = hp.count[i];
      continue;
    }
    const int64_t parts = (steps_of(i) + per - 1) / per, rows = (steps_of(i) + parts - 1) / parts * STEP;
    for (int64_t m = 0; m < hp.dev[i].Mg; m += rows) {
      sk_tile t = hp.tiles[(size_t)hp.first[i]];
      t.cls = CLS_WINDOW;
      t.m0 = (uint32_t)m;
      t.m_len = (uint16_t)std::min<int64_t>(rows, hp.dev[i].Mg - m);
      t.out_tile_id = id++;
      records.push_back(t);
      ++count[i];
    }
  }
  return true;
}

// Tiles that run_tile_rows runs, side by side along the rows, as runs of a third of a workgroup's share of the launch: a run loads its weights
// once, and a block's rows while the one before is multiplied.  (Not where they are less than a fifth of the work, FLAG_ROWS: longer records
// cost the launch's end more than they save there.)  Down-sampling layers with the 7x7 stem, us, in single tiles / in runs of half, a third and a quarter of a
// share: for sixteen tenants 102.6 / 91.6, 85.4, 91.9, for eleven 70.1 / 65.3, 66.1, 63.8, for eight 54.0 / 53.8, 47.7, 51.1, for six 44.5 / 40.9, 39.9, 44.2;
// 96 odd-sized operators, of which they are a seventh, 70.5 / 75.7, 75.3, 70.1.
// In a plan of several deadlines of an eighth of a share, so that the first deadlines' operators are not done with the launch's middle: 64 stems with deadlines of
// their own, us until the first tenth of them in that order are done, all of them in the mean, the last: as tiles 25.5, 76.1 and 138.2, in runs of a
// third 43.6, 59.9 and 89.2, a fifth 28.2, 54.3 and 87.9, an eighth 24.4, 55.1 and 89.6; stride-2 layers for sixteen 61.5, 61.6 and 97, 65.4, 60.5 and 100,
// 64, 58.6 and 92, 62.6, 57.4 and 90; sixteen stems 16.4, 28.1 and 42.1, 20.8, 26.4 and 37.2, 16.6, 28.4 and 42.5, as a fifth (tiles).  False: nothing changed.
static bool rows_runs(const HostPlan &hp, int64_t workgroups, const std::vector<sk_tile> &records, std::vector<sk_tile> &joined,
                      std::vector<int64_t> &count) {
  constexpr int64_t MOST = 16, BLOCK = 4500;  // blocks; nanoseconds of one, with its part of what is around them
  if (workgroups < 1 || !hp.rows || !hp.xorder.empty()) return false;
  const int64_t blocks = std::min<int64_t>(MOST, work_of(hp, records, nullptr) * 2 / workgroups / (several_deadlines(hp) ? 8 : 3) / BLOCK);
  if (blocks < 2) return false;
  joined.clear();
  joined.reserve(records.size());
  count.assign(hp.dev.size(), 0);
  bool open = false, rows = false;  // whether run_tile_rows runs the last of `joined`, this record
  const sk_tile *last = nullptr;
  for (const sk_tile &t : records) {
    const DevProblem &d = hp.dev[t.problem];
    if (!last || !alike(d, *last, t)) rows = runs_in_rows(d, t);
    last = &t;
    if (open && rows) {
      sk_tile u = joined.back();
      if (u.problem == t.problem && u.n0 == t.n0 && u.m0 + u.m_len == t.m0 && u.m_len % 128 == 0 && u.m_len + t.m_len <= 128 * blocks) {
        u.m_len = (uint16_t)(u.m_len + t.m_len);
        if (in_one_image(d, u)) {
          joined.back() = u;
          continue;
        }
      }
    }
    open = rows;
    joined.push_back(t);
    ++count[t.problem];
  }
  return joined.size() != records.size();
}

// The list of tiles, and with `runs` of runs of pixels where they pay, for a launch of that many workgroups.
static bool list_records(const HostPlan &hp, int64_t workgroups, bool runs, bool tiles_only, const std::vector<Slicing> *impose, WorkList &out) {
  std::vector<sk_tile> cut;
  std::vector<int64_t> count;
  auto as_cut = [&]() {
    out = WorkList{};
    out.work = std::move(cut);
    out.count = std::move(count);
    out.ws_off = hp.ws_off;
    out.ws_f32x4 = hp.ws_f32x4;
  };
  if (runs && window_records(hp, workgroups, cut, count)) {
    // (balanced as if there were no lists: none are left)
    if (!balance_records(hp, cut, workgroups, true, impose, out)) {
      as_cut();
      for (sk_tile &t : out.work)
        if (t.cls == CLS_WINDOW) t.out_tile_id = 0;  // (never used: no slices)
    }
    out.window = true;
    return true;
  }
  if (tiles_only) return false;
  const bool refined = refine_blocks(hp, workgroups, cut, count);
  const std::vector<sk_tile> &records = refined ? cut : hp.tiles;
  std::vector<sk_tile> joined;
  std::vector<int64_t> joined_count;
  if (rows_runs(hp, workgroups, records, joined, joined_count)) {
    // (the slices are those of the tiles, with and without lists; order and cuts go by the runs)
    std::vector<Slicing> own;
    WorkList plain;
    if (!impose && balance_records(hp, records, workgroups, false, nullptr, plain, true)) own = std::move(plain.slicing);
    cut = std::move(joined);
    count = std::move(joined_count);
    if (balance_records(hp, cut, workgroups, false, impose ? impose : &own, out))
      out.slicing = std::move(own);
    else
      as_cut();
    return true;
  }
  if (balance_records(hp, records, workgroups, false, impose, out)) return true;
  if (!refined || !hp.xorder.empty()) return false;
  as_cut();
  return true;
}

// Slices, which change the sums' order, are those of a launch that fills the chip, whatever the grid of this one (its limit is the caller's,
// its compute units are the device's, and a host-only plan has no device yet): results depend on the operators and the
// table's parameters alone.  Order and cuts follow the grid.  Plans of short tiles alone get no slices.
static bool list_records(const HostPlan &hp, int64_t workgroups, bool runs, bool tiles_only, bool slices, WorkList &out) {
  const std::vector<Slicing> none;
  if (!slices || tiles_only) return list_records(hp, workgroups, runs, tiles_only, &none, out);
  if (workgroups == CHIP_WORKGROUPS) return list_records(hp, workgroups, runs, tiles_only, nullptr, out);
  WorkList chip;
  if (!list_records(hp, CHIP_WORKGROUPS, runs, tiles_only, nullptr, chip)) chip.slicing.clear();
  return list_records(hp, workgroups, runs, tiles_only, &chip.slicing, out);
}

bool device_list(const HostPlan &hp, int64_t workgroups, bool tiles_only, WorkList &out, bool slices) {
  return list_records(hp, workgroups, true, tiles_only, slices, out);
}

// Measured against the general kernel as it is now (3x3 64-channel convolutions in bf16, us, general / narrow): 25 tiles 11.4 / 10.6,
// 100 tiles 12.4 / 11.6, 300 to 500 tiles 1 to 4 % slower; 550 to 680 tiles, which start at once in threes but not in
// twos, 26 / 24; 750 tiles 27.3 / 28.4, 2800 tiles 59.4 / 63.3 (whole rounds of longer tiles); 4000 tiles 87.2 / 85.0, 12800 tiles 240
// / 223.  16-bit tiles of more than a dozen stages gain nothing (their ring of two stage images waits for
// every load): 1024 rows of 2048 121 us instead of 113.  fp32 tiles, bound by the matrix cores, gain up to 30 % at 640 tiles
// and 3 to 6 % from 3000 on, whatever their length.  (16-bit 3x3 convolutions of 64 channels with more tiles than workgroups run as
// runs of pixels by now: window_records.)
bool narrow_pays(bool fp32, int64_t stages, int64_t tiles, int64_t compute_units) {
  if (!fp32 && stages > 12) return false;
  if (tiles <= compute_units) return !fp32 || stages <= 12;
  return (tiles > 2 * compute_units && tiles * 10 <= 27 * compute_units) || tiles >= (fp32 ? 8 : 15) * compute_units;
}

bool narrow_plan(const HostPlan &hp) {
  if (hp.tiles.empty()) return false;
  for (const sk_tile &t : hp.tiles)
    if (t.cls != CLS_TILE_128x64) return false;
  for (const DevProblem &d : hp.dev) {
    const int64_t es = elem_size(d.dtype), limit = (int64_t)1 << 30;  // (bytes; a tile spans at most the operand)
    if ((d.flags & (FLAG_VEC_A | FLAG_VEC_B)) != (FLAG_VEC_A | FLAG_VEC_B) || d.nchw) return false;
    if ((int64_t)d.Ng * d.ldb * es >= limit) return false;
    if (!d.gather) {
      if (128 * d.lda * es >= limit) return false;
    } else {
      if (d.Cin % (128 / es) != 0 || d.R * d.S > 31) return false;
      const int64_t images = d.Mg / ((int64_t)d.Ho * d.Wo);
      if (!offsets_below(d, images - 1, es, limit)) return false;
    }
  }
  return true;
}

sk_status plan_host_each_alone(const HostPlan &whole, int64_t workgroups, HostPlan &out, std::string &err) {
  const int32_t n = (int32_t)whole.problems.size();
  out = HostPlan{};
  out.params = whole.params;
  out.problems = whole.problems;
  out.dev = whole.dev;
  out.order.resize(n);
  std::iota(out.order.begin(), out.order.end(), 0);
  out.first.assign(n, 0);
  out.count.assign(n, 0);
  out.target_tile_bytes = 0;
  sk_plan_params prm = whole.params;
  prm.host_only = 1;
  uint32_t rect_base = 0;
  for (int32_t i = 0; i < n; ++i) {
    HostPlan one;
    const sk_status st = plan_host(&whole.problems[i], 1, &prm, one, err);
    if (st != SK_OK) return st;
    std::vector<int64_t> counts;
    std::vector<sk_tile> cut;
    const std::vector<sk_tile> &records = refine_blocks(one, workgroups, cut, counts) ? cut : one.tiles;
    out.first[i] = (int64_t)out.tiles.size();
    out.count[i] = (int64_t)records.size();
    for (sk_tile t : records) {
      t.problem = (uint32_t)i;
      t.out_tile_id += rect_base;
      out.tiles.push_back(t);
    }
    for (uint32_t w : one.ws_off) out.ws_off.push_back(w + (uint32_t)out.ws_f32x4);
    rect_base += (uint32_t)one.ws_off.size();
    out.ws_f32x4 += one.ws_f32x4;
    out.dev[i].tile_first = (int32_t)out.first[i];
    out.dev[i].tile_count = (int32_t)out.count[i];
    if (out.tiles.size() > (size_t)1 << 30 || out.ws_f32x4 > ((int64_t)1 << 31)) {
      err = "tile table or split-K workspace too large";
      return SK_ERR_UNSUPPORTED;
    }
  }
  return SK_OK;
}

bool balance_each_alone(HostPlan &alone, int64_t workgroups) {
  HostPlan out = alone;
  out.tiles.clear();
  out.ws_off.clear();
  out.ws_f32x4 = 0;
  sk_plan_params prm = alone.params;
  prm.host_only = 1;
  std::string err;
  bool changed = false;
  for (size_t i = 0; i < alone.dev.size(); ++i) {
    HostPlan one;
    if (plan_host(&alone.problems[i], 1, &prm, one, err) != SK_OK) return false;
    one.xorder.clear();  // (its launch is a range of the tables: no lists)
    WorkList w;
    if (list_records(one, workgroups, false, false, true, w)) {
      changed = true;
    } else {
      w.work = one.tiles;
      w.ws_off = one.ws_off;
      w.ws_f32x4 = one.ws_f32x4;
    }
    out.first[i] = (int64_t)out.tiles.size();
    out.count[i] = (int64_t)w.work.size();
    const uint32_t base = (uint32_t)out.ws_off.size();
    for (sk_tile t : w.work) {
      t.problem = (uint32_t)i;
      t.out_tile_id += base;
      out.tiles.push_back(t);
    }
    for (const uint32_t w_off : w.ws_off) out.ws_off.push_back(w_off + (uint32_t)out.ws_f32x4);
    out.ws_f32x4 += w.ws_f32x4;
    out.dev[i].tile_first = (int32_t)out.first[i];
    out.dev[i].tile_count = (int32_t)out.count[i];
    if (out.ws_f32x4 > ((int64_t)1 << 31)) return false;
  }
  if (changed) alone = std::move(out);
  return changed;
}

// A launch on the stream of the previous launch is ordered behind it by the stream.  On another stream it
// may only go ahead when the previous launch has completed (the caller asks the event).  Inside a stream
// capture nothing can be asked: the launch is recorded, and the graph's replays are the caller's to order.
LaunchLedger::Ask LaunchLedger::before_launch(uintptr_t stream, bool capturing) const {
  if (capturing || !has_event || stream == last_stream) return GO;
  return QUERY_EVENT;
}

void LaunchLedger::after_launch(uintptr_t stream, bool capturing, bool event_recorded) {
  if (capturing || !event_recorded) {
    device_wide = true;  // replays of a graph, or a launch without an event behind it
    return;
  }
  // every earlier eager launch either shares this stream or had completed before this one was admitted:
  // the event behind this launch covers them all
  has_event = true;
  last_stream = stream;
}

LaunchLedger::Wait LaunchLedger::before_destroy() const {
  if (device_wide) return DEVICE;
  return has_event ? EVENT : NOTHING;
}

int64_t operand_bytes(const sk_problem &p) {
  const int64_t es = elem_size(p.dtype);
  if (p.op == SK_GEMM) {
    if (p.M < 1 || p.N < 1 || p.K < 1) return 0;
    return es * ((int64_t)p.M * p.K + (int64_t)p.N * p.K + (int64_t)p.M * p.N);
  }
  if (p.op != SK_CONV2D_NHWC && p.op != SK_CONV2D_NCHW) return 0;
  const int64_t st = p.stride > 0 ? p.stride : 1;
  const int64_t span_h = (int64_t)p.H + 2 * (int64_t)p.pad_h - p.R, span_w = (int64_t)p.Wd + 2 * (int64_t)p.pad_w - p.S;
  if (p.Nb < 1 || p.Cin < 1 || p.Cout < 1 || p.R < 1 || p.S < 1 || span_h < 0 || span_w < 0) return 0;
  const int64_t Ho = span_h / st + 1, Wo = span_w / st + 1;
  return es * ((int64_t)p.Nb * p.H * p.Wd * p.Cin + (int64_t)p.Cout * p.R * p.S * p.Cin + (int64_t)p.Nb * Ho * Wo * p.Cout);
}

double estimate_launch_ms(int64_t bytes, double bytes_per_ms, double floor_ms) {
  const double t = (double)bytes / bytes_per_ms;
  return t > floor_ms ? t : floor_ms;
}

std::vector<size_t> select_batch(const std::vector<QueuedOp> &ops, const std::vector<const void *> &busy, int policy,
                                 double cap_ms, double corr, double bytes_per_ms, double floor_ms) {
  std::vector<size_t> picked;
  if (ops.empty()) return picked;
  if (policy == SK_QUEUE_SEQUENTIAL) {
    // arrival order; one stream keeps launches into one buffer ordered, so a busy output does not hold it back
    picked.push_back(0);
    return picked;
  }
  std::vector<size_t> order(ops.size());
  std::iota(order.begin(), order.end(), (size_t)0);
  std::stable_sort(order.begin(), order.end(),
                   [&](size_t a, size_t b) { return ops[a].deadline_ms < ops[b].deadline_ms; });
  std::unordered_set<const void *> taken;  // outputs of this batch
  int64_t total = 0;
  for (size_t i : order) {
    const void *c = ops[i].C;
    if (std::binary_search(busy.begin(), busy.end(), c) || taken.count(c)) continue;
    if (policy == SK_QUEUE_OOO && !picked.empty() &&
        estimate_launch_ms(total + ops[i].bytes, bytes_per_ms, floor_ms) * corr > cap_ms)
      break;
    picked.push_back(i);
    taken.insert(c);
    total += ops[i].bytes;
  }
  return picked;
}

}  // namespace sk

extern "C" void sk_plan_params_default(sk_plan_params *p) {
  if (!p) return;
  std::memset(p, 0, sizeof(*p));
  p->edf = 1;
  p->stamps = 0;
  p->host_only = 0;
  p->skinny_max_m = 64;
  p->tile_bytes_max = 2048 * 1024;
  p->tile_bytes_min = 32 * 1024;
  p->balance_div = 512;
  p->max_groups = 256;
  p->grid_limit = 0;
  p->tail_div = 384;
  p->xcd_part = -1;
  p->reserved = 0;
}
