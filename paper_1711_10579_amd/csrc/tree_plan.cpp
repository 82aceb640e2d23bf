// Work plan of the sparse refactorisation (Sec. III-A) of one case: the lower
// levels a launch each, the upper ones as subtrees of the elimination tree
// dealt out to work-groups.

#include <algorithm>
#include <cstdint>
#include <queue>

#include "analysis.hpp"

namespace pfh {

namespace {

// lanes a wave gives a column of each class (the last two in several passes
// of the wave) and about the time of a pass (us)
constexpr int kClassLanes[kTreeClasses] = {8, 16, 32, 64, 128, 256};
constexpr double kPass[kTreeClasses] = {0.9, 0.9, 0.9, 0.9, 1.4, 2.4};
constexpr double kLevel = 0.8;       // a level's barrier and first reads (us)
constexpr double kTreeLaunch = 6.0;  // a stage's launch and the lists' way into LDS
constexpr double kLevelLaunch = 4.8;
constexpr double kChipWaves = 4096;  // waves a level launch keeps in flight, 4 us a round

int tree_class(int len, int G) {
  const int64_t lanes = (2LL * len + 2) * G;
  for (int c = 0; c < kTreeClasses; ++c)
    if (lanes <= kClassLanes[c]) return c;
  return kTreeClasses;  // the whole work-group
}

double class_waves(int c) { return c < 3 ? 0.125 * (1 << c) : 1.0; }

struct Binning {
  int la = 0, lb = 0, threads = 256, nbins = 0;
  double time = 0;
  std::vector<int> bin;  // of the stage's columns, in level order
};

}  // namespace

std::vector<int> factor_lanes(const Analysis& an, int lane_scale) {
  const int nl = (int)an.col_lev_ptr.size() - 1;
  std::vector<int> g(nl, 1);
  for (int l = 0; l < nl; ++l) {
    int64_t m = 0;
    for (int k = an.col_lev_ptr[l]; k < an.col_lev_ptr[l + 1]; ++k) {
      const int j = an.col_order[k], len = an.colptr[j + 1] - an.colptr[j];
      const int64_t t0 = j + 2LL * an.colptr[j];
      for (int t = 0; t <= 2 * len; ++t) m = std::max(m, an.uptr[t0 + t + 1] - an.uptr[t0 + t]);
      m = std::max<int64_t>(m, an.lrow_ptr[j + 1] - an.lrow_ptr[j]);
    }
    // one lane count for the level's update lists and its forward rows (run
    // by the same groups)
    g[l] = pick_lanes(m, lane_scale);
  }
  return g;
}

TreePlan plan_trees(const Analysis& an, const std::vector<int>& g, int max_bins, int first_level) {
  TreePlan tp;
  const int ns = an.ns, nl = (int)an.col_lev_ptr.size() - 1;
  tp.first_level = nl;
  tp.bin_off.push_back(0);
  tp.bin_ptr.push_back(0);
  if (ns == 0) return tp;
  std::vector<int> lev(ns), cls(ns), words(ns), root(ns), comp;
  std::vector<float> cost(ns), work(ns), slots, big;
  std::vector<double> level_launch(nl + 1, 0.0);  // time of the launches of levels below
  for (int l = 0; l < nl; ++l) {
    double waves = 0;
    for (int k = an.col_lev_ptr[l]; k < an.col_lev_ptr[l + 1]; ++k) {
      const int j = an.col_order[k], len = an.colptr[j + 1] - an.colptr[j];
      lev[j] = l;
      cls[j] = tree_class(len, g[l]);
      cost[j] = cls[j] < kTreeClasses ? class_waves(cls[j]) * kPass[cls[j]] : (2.0 * len + 2) * g[l] / 64.0;
      waves += cost[j];
      const int64_t t0 = j + 2LL * an.colptr[j];
      // column entry, target table, pairs of the update lists and the
      // forward row (level records are counted per bin)
      words[j] = 5 + 2 * len + 3 + 2 * (int)(an.uptr[t0 + 1 + 2 * len] - an.uptr[t0]) +
                 2 * (an.lrow_ptr[j + 1] - an.lrow_ptr[j]);
    }
    level_launch[l + 1] = level_launch[l] + kLevelLaunch + 4.0 * waves / kChipWaves;
  }
  // levels [la, lb) as one launch: the trees of the forest cut to them, dealt
  // to the least loaded bin, largest first; time infinite when a bin's lists
  // do not fit
  auto deal = [&](int la, int lb, int threads, int bins) {
    Binning b;
    b.la = la;
    b.lb = lb;
    b.threads = threads;
    const int k0 = an.col_lev_ptr[la], k1 = an.col_lev_ptr[lb];
    comp.clear();
    for (int k = k1 - 1; k >= k0; --k) {  // parents lie in higher levels
      const int j = an.col_order[k], p = an.parent[j];
      root[j] = p >= 0 && lev[p] < lb ? root[p] : j;
      if (root[j] == j) {
        comp.push_back(j);
        work[j] = 0;
      }
      work[root[j]] += cost[j];
    }
    std::sort(comp.begin(), comp.end(), [&](int x, int y) { return work[x] != work[y] ? work[x] > work[y] : x < y; });
    b.nbins = std::max(1, std::min<int>(bins, (int)comp.size()));
    std::priority_queue<std::pair<float, int>, std::vector<std::pair<float, int>>, std::greater<>> load;
    for (int i = 0; i < b.nbins; ++i) load.push({0.0f, i});
    std::vector<int> bin_of_root(comp.size());
    for (size_t i = 0; i < comp.size(); ++i) {
      auto t = load.top();
      load.pop();
      bin_of_root[i] = t.second;
      load.push({t.first + work[comp[i]], t.second});
    }
    for (size_t i = 0; i < comp.size(); ++i) work[comp[i]] = (float)bin_of_root[i];
    const int W = threads / 64, n = lb - la;
    slots.assign((size_t)b.nbins * n, 0.0f);
    big.assign((size_t)b.nbins * n, 0.0f);
    std::vector<int64_t> size(b.nbins, kTreeHead + kTreeRec * n + 8);
    b.bin.resize(k1 - k0);
    for (int k = k0; k < k1; ++k) {
      const int j = an.col_order[k], i = (int)work[root[j]];
      b.bin[k - k0] = i;
      size[i] += words[j];
      const size_t at = (size_t)i * n + (lev[j] - la);
      if (cls[j] < kTreeClasses)
        slots[at] += cost[j];
      else
        big[at] += 1.0f + cost[j] / W;
    }
    for (int i = 0; i < b.nbins; ++i) {
      double t = size[i] > kTreeWords ? 1e30 : 0;
      for (int l = 0; l < n; ++l) {
        const double s = slots[(size_t)i * n + l] / W, x = big[(size_t)i * n + l];
        if (s > 0 || x > 0) t += kLevel + x + (s > 0 ? std::max(0.9, s) : 0.0);
      }
      b.time = std::max(b.time, t);
    }
    b.time += kTreeLaunch;
    return b;
  };
  // 256 threads a work-group (two to a CU) or 512
  auto best = [&](int la, int lb) {
    Binning b = deal(la, lb, 512, std::max(1, max_bins / 2));
    if (b.nbins == std::max(1, max_bins / 2) && b.nbins < max_bins) {
      Binning a = deal(la, lb, 256, max_bins);
      if (a.time < b.time) return a;
    }
    return b;
  };
  // where the launches end and the trees begin: levels of very many columns
  // fill the chip by themselves and always take a launch
  int lo = 0;
  while (lo < nl && an.col_lev_ptr[lo + 1] - an.col_lev_ptr[lo] > kTreeColumns) ++lo;
  std::vector<Binning> st;
  double now = level_launch[nl];
  auto consider = [&](int c0) {
    if (c0 < 0 || c0 >= nl) return;
    Binning one = best(c0, nl);
    const double below = level_launch[c0];
    if (below + one.time < now) {
      now = below + one.time;
      st.clear();
      st.push_back(one);
    }
    // a tree that holds most of the work leaves the other work-groups idle:
    // its levels in two stages
    const int c1 = c0 + (nl - c0) / 2;
    if (c1 > c0 && one.time > 1.3 * (kTreeLaunch + (nl - c0) * (kLevel + 0.9))) {
      Binning a = best(c0, c1), b = best(c1, nl);
      if (below + a.time + b.time < now) {
        now = below + a.time + b.time;
        st.clear();
        st.push_back(std::move(a));
        st.push_back(std::move(b));
      }
    }
  };
  if (first_level >= nl) return tp;
  if (first_level >= 0) {
    now = 1e300;
    consider(first_level);
  } else {
    int last = -1;
    for (int f = 0; f <= 2; ++f) {
      const int c0 = lo + (nl - lo) * f / 3;
      if (c0 != last) consider(c0);
      last = c0;
    }
  }
  if (st.empty() || now >= 1e29) return tp;
  tp.first_level = st[0].la;
  {
    int64_t total = 0;
    for (const Binning& b : st) {
      for (int k = an.col_lev_ptr[b.la]; k < an.col_lev_ptr[b.lb]; ++k) total += words[an.col_order[k]];
      total += (int64_t)b.nbins * (kTreeHead + kTreeRec * (b.lb - b.la) + 8);
    }
    tp.prog.reserve(total);
  }
  for (const Binning& b : st) {
    tp.stages.push_back({(int)tp.bin_off.size() - 1, b.nbins, b.threads});
    const int k0 = an.col_lev_ptr[b.la];
    // the stage's columns by bin (stable: by level inside a bin)
    std::vector<int> start(b.nbins + 1, 0), cols(b.bin.size());
    for (int i : b.bin) start[i + 1]++;
    for (int i = 0; i < b.nbins; ++i) start[i + 1] += start[i];
    {
      std::vector<int> fill(start.begin(), start.end() - 1);
      for (size_t k = 0; k < b.bin.size(); ++k) cols[fill[b.bin[k]]++] = an.col_order[k0 + k];
    }
    for (int i = 0; i < b.nbins; ++i) {
      std::vector<int>& P = tp.prog;
      const size_t base = P.size();
      const int c0 = start[i], c1 = start[i + 1];
      // a level's columns by class, and the slots they take
      std::vector<std::pair<int, int>> recs;  // columns [first, end) of a record
      int nslots = 0;
      auto slots_of = [&](int k, int e, auto&& f) {  // f(first column, columns, log2 lanes); whole work-group: -1
        while (k < e) {
          const int c = cls[cols[k]], per = c < 3 ? 8 >> c : 1;
          int m = k;
          while (m < e && m - k < per && cls[cols[m]] == c) ++m;
          f(k, m - k, c == kTreeClasses ? -1 : std::min(c + 3, 6));
          k = m;
        }
      };
      for (int k = c0; k < c1;) {
        int e = k;
        while (e < c1 && lev[cols[e]] == lev[cols[k]]) ++e;
        std::stable_sort(cols.begin() + k, cols.begin() + e, [&](int x, int y) { return cls[x] < cls[y]; });
        recs.emplace_back(k, e);
        slots_of(k, e, [&](int, int, int) { ++nslots; });
        k = e;
      }
      // records | slots | columns | target tables and pairs, offsets from the
      // bin's first word
      const int nrec = (int)recs.size();
      int slot = kTreeHead + kTreeRec * nrec;
      const int col0 = (slot + nslots + 3) / 4 * 4;
      int tab = col0 + 4 * (c1 - c0);
      int size = tab;
      for (int k = c0; k < c1; ++k) size += words[cols[k]] - 5;
      P.resize(base + (size + 3) / 4 * 4, 0);
      P[base] = nrec;
      P[base + 1] = nslots;
      for (int r = 0; r < nrec; ++r) {
        int* rec = &P[base + kTreeHead + kTreeRec * r];
        rec[0] = slot;
        rec[2] = g[lev[cols[recs[r].first]]];
        slots_of(recs[r].first, recs[r].second, [&](int k, int n, int ll) {
          P[base + slot++] = (col0 + 4 * (k - c0)) | (ll < 0 ? 0 : ll) << 16 | n << 24;
          rec[ll < 0 ? 3 : 1]++;
        });
      }
      for (int k = c0; k < c1; ++k) {
        const int j = cols[k], len = an.colptr[j + 1] - an.colptr[j];
        const size_t at = base + col0 + 4 * (size_t)(k - c0);
        P[at] = j;
        P[at + 1] = an.colptr[j];
        P[at + 2] = len;
        P[at + 3] = tab;
        // targets: D, the U row, the forward row, the L column
        const int64_t t0 = j + 2LL * an.colptr[j];
        int* const table = &P[base + tab];
        tab += 2 * len + 3;
        int* w = &P[base] + tab;
        for (int t = 0; t < 2 * len + 2; ++t) {
          table[t] = (int)(w - &P[base]);
          if (t == len + 1) {
            for (int q = an.lrow_ptr[j]; q < an.lrow_ptr[j + 1]; ++q) {
              *w++ = an.lrow_blk[q];
              *w++ = an.lrow_col[q];
            }
          } else {
            const int64_t tg = t <= len ? t0 + t : t0 + t - 1;
            for (int64_t q = an.uptr[tg]; q < an.uptr[tg + 1]; ++q) {
              *w++ = an.upd_l[q];
              *w++ = an.upd_u[q];
            }
          }
        }
        tab = table[2 * len + 2] = (int)(w - &P[base]);
      }
      tp.bin_off.push_back((int)P.size());
      tp.bin_cols.insert(tp.bin_cols.end(), cols.begin() + c0, cols.begin() + c1);
      tp.bin_ptr.push_back((int)tp.bin_cols.size());
    }
  }
  return tp;
}

BwdTrees plan_bwd_trees(const Analysis& an, const TreePlan& tp, const std::vector<int>& lanes) {
  BwdTrees bt;
  const int ns = an.ns;
  bt.in.assign(ns, 0);
  if (tp.stages.empty()) return bt;
  std::vector<int> lev(ns), place(an.nu, -1), owner(an.nu, -1);
  for (int l = 0; l + 1 < (int)an.bwd_lev_ptr.size(); ++l)
    for (int k = an.bwd_lev_ptr[l]; k < an.bwd_lev_ptr[l + 1]; ++k) lev[an.bwd_rows[k]] = l;
  std::vector<int>& P = bt.prog;
  bt.off.push_back(0);
  int serial = 0;
  for (int s = (int)tp.stages.size() - 1; s >= 0; --s)
    for (int b = tp.stages[s].bin0; b < tp.stages[s].bin0 + tp.stages[s].nbins; ++b) {
      std::vector<int> rows(tp.bin_cols.begin() + tp.bin_ptr[b], tp.bin_cols.begin() + tp.bin_ptr[b + 1]);
      std::stable_sort(rows.begin(), rows.end(), [&](int x, int y) { return lev[x] < lev[y]; });
      const int nr = (int)rows.size();
      int nrec = 0, nent = 0;
      for (int k = 0; k < nr; ++k) {
        nrec += k == 0 || lev[rows[k]] != lev[rows[k - 1]];
        nent += an.colptr[rows[k] + 1] - an.colptr[rows[k]];
        bt.in[rows[k]] = 1;
        owner[rows[k]] = serial;
        place[rows[k]] = k;
      }
      const size_t base = P.size();
      const int row0 = 4 + 4 * nrec, ref0 = row0 + 4 * nr;
      P.resize(base + ref0 + 2 * (size_t)nent, 0);
      std::vector<int> out;
      int rec = 0, f = 0;
      for (int k = 0; k < nr; ++k) {
        const int i = rows[k], q0 = an.colptr[i], q1 = an.colptr[i + 1];
        if (k == 0 || lev[i] != lev[rows[k - 1]]) {
          int lg = 0;
          while (1 << lg < lanes[lev[i]]) ++lg;
          int* p = &P[base + 4 + 4 * rec++];
          p[0] = k;
          p[2] = lg;
        }
        P[base + 4 + 4 * (rec - 1) + 1]++;
        int* p = &P[base + row0 + 4 * (size_t)k];
        p[0] = i;
        p[1] = f;
        p[2] = q1 - q0;
        for (int q = q0; q < q1; ++q, ++f) {
          const int c = an.rowidx[q];
          if (owner[c] != serial) {  // read from elsewhere
            owner[c] = serial;
            place[c] = nr + (int)out.size();
            out.push_back(c);
          }
          P[base + ref0 + f] = place[c];
          P[base + ref0 + nent + f] = (int)(ns + an.nnzl + q);
        }
      }
      P[base] = nrec;
      P[base + 1] = nr;
      P[base + 2] = nent;
      P[base + 3] = (int)out.size();
      P.insert(P.end(), out.begin(), out.end());
      P.resize((P.size() + 3) / 4 * 4, 0);
      bt.off.push_back((int)P.size());
      ++serial;
      if (4 * (int64_t)(P.size() - base) + kBwdRowBytes * (int64_t)nr + 16 * (int64_t)out.size() > kBwdBytes) {
        // a bin of very many rows: every row by levels
        bt.off.clear();
        bt.prog.clear();
        bt.in.assign(ns, 0);
        return bt;
      }
    }
  return bt;
}

}  // namespace pfh
