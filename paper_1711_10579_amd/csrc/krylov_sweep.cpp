// ILU(0) preconditioner (Sec. III-B): the factor's targets by level, and the
// parts of its sweeps: runs of levels whose rows are written out in terms of
// the part's input, so that an application is one launch per part instead of
// one barrier or launch per level.

#include <algorithm>
#include <cstdint>

#include "analysis.hpp"

namespace pfh {

void factor_targets(const KAnalysis& ka, std::vector<int>* ptr, std::vector<int>* tgt) {
  const int nl = (int)ka.lev_ptr.size() - 1;
  std::vector<int> lev(ka.nu);
  for (int l = 0; l < nl; ++l)
    for (int k = ka.lev_ptr[l]; k < ka.lev_ptr[l + 1]; ++k) lev[ka.lev_rows[k]] = l;
  ptr->assign(nl + 1, 0);
  tgt->clear();
  std::vector<int> fill;
  for (int pass = 0; pass < 2; ++pass) {
    for (int r = 0; r < ka.nu; ++r)
      for (int t = ka.row_ptr[r]; t < ka.row_ptr[r + 1]; ++t) {
        const bool diag = t == ka.diag[r];
        if (!diag && ka.up_ptr[t] == ka.up_ptr[t + 1]) continue;
        const int l = lev[t < ka.diag[r] ? ka.col[t] : r];
        if (pass == 0)
          (*ptr)[l + 1]++;
        else
          (*tgt)[fill[l]++] = diag ? ~t : t;
      }
    if (pass == 0) {
      for (int l = 0; l < nl; ++l) (*ptr)[l + 1] += (*ptr)[l];
      tgt->resize(ptr->back());
      fill.assign(ptr->begin(), ptr->end() - 1);
    }
  }
}

bool build_sweep(const KAnalysis& ka, int cap, int64_t max_entries, KSweep* out) {
  KSweep& s = *out;
  s = KSweep();
  const int nu = ka.nu;
  s.part_ptr.push_back(0);
  s.op_ptr.push_back(0);
  s.rows.reserve(8 * (size_t)nu);
  s.step.reserve(2 * (size_t)nu);
  std::vector<int> pos_of(nu), part(nu), where(2 * (size_t)nu, -1);
  // one row's entries as first met, and its ops (entry, q, s)
  std::vector<int> keys, oe, oq, os, cnt, fill;
  struct Row {
    int r, key0, key1, op0, op1;
  };
  std::vector<Row> lrow;
  std::vector<int> lkeys, loe, loq, los, order;

  for (int upper = 0; upper < 2; ++upper) {
    const auto& ptr = upper ? ka.ulev_ptr : ka.lev_ptr;
    const auto& rows = upper ? ka.ulev_rows : ka.lev_rows;
    const int nl = (int)ptr.size() - 1;
    std::fill(part.begin(), part.end(), -1);
    int cur = -1, first = 0;  // current part and its first level
    for (int l = 0; l < nl; ++l) {
      // the level's rows inside the current part; when one grows past the
      // cap, again as the first level of a part of its own
      for (int pass = l == 0 ? 1 : 0; pass < 2; ++pass) {
        if (pass == 1) {
          if (cur >= 0) s.part_ptr.push_back((int)s.rows.size() / 4);
          ++cur;
          first = l;
        }
        lrow.clear();
        lkeys.clear();
        loe.clear();
        loq.clear();
        los.clear();
        bool fits = true;
        for (int k = ptr[l]; k < ptr[l + 1] && fits; ++k) {
          const int r = rows[k];
          const int key0 = (int)lkeys.size(), op0 = (int)loe.size();
          // key: 2 c for the part's input at row c, 2 c + 1 for an earlier row
          auto entry = [&](int key) {
            if (where[key] < key0) {
              where[key] = (int)lkeys.size();
              lkeys.push_back(key);
            }
            return where[key] - key0;
          };
          auto add = [&](int key, int q, int src) {
            loe.push_back(entry(key));
            loq.push_back(q);
            los.push_back(src);
          };
          if (upper) entry(2 * r);  // the row's own entry, without ops
          const int q0 = upper ? ka.diag[r] + 1 : ka.row_ptr[r], q1 = upper ? ka.row_ptr[r + 1] : ka.diag[r];
          for (int q = q0; q < q1; ++q) {
            const int c = ka.col[q];
            if (part[c] != cur) {
              add(2 * c + 1, q, -1);
              continue;
            }
            if (!upper) add(2 * c, q, -1);  // the identity on y_c's own input
            const int* rc = &s.rows[4 * (size_t)pos_of[c]];
            for (int e = rc[1]; e < rc[2]; ++e) add(s.col[e] < 0 ? 2 * ~s.col[e] : 2 * s.col[e] + 1, q, e);
          }
          const int key1 = (int)lkeys.size();
          for (int e = key0; e < key1; ++e) where[lkeys[e]] = -1;
          lrow.push_back({r, key0, key1, op0, (int)loe.size()});
          fits = pass == 1 || key1 - key0 <= cap;
        }
        if (fits) break;
      }
      // a wave holds several rows: rows of like length beside each other
      order.resize(lrow.size());
      for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
      std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return lrow[a].key1 - lrow[a].key0 > lrow[b].key1 - lrow[b].key0;
      });
      for (int i : order) {
        const Row& w = lrow[i];
        const int e0 = (int)s.col.size(), len = w.key1 - w.key0;
        part[w.r] = cur;
        pos_of[w.r] = (int)s.rows.size() / 4;
        s.rows.insert(s.rows.end(), {w.r, e0, e0 + len, 0});
        s.step.push_back(l - first);
        s.nsteps = std::max(s.nsteps, l - first + 1);
        cnt.assign(len + 1, 0);
        for (int o = w.op0; o < w.op1; ++o) cnt[loe[o] + 1]++;
        const int o0 = s.op_ptr.back();
        for (int e = 0; e < len; ++e) {
          const int key = lkeys[w.key0 + e];
          s.col.push_back(key & 1 ? key >> 1 : ~(key >> 1));
          cnt[e + 1] += cnt[e];
          s.op_ptr.push_back(o0 + cnt[e + 1]);
        }
        s.ops.resize(2 * (size_t)(o0 + (w.op1 - w.op0)));
        for (int o = w.op0; o < w.op1; ++o) {
          const size_t at = 2 * (size_t)(o0 + cnt[loe[o]]++);
          s.ops[at] = loq[o];
          s.ops[at + 1] = los[o];
        }
      }
      if (s.ne() > max_entries) return false;
    }
    if (cur >= 0) s.part_ptr.push_back((int)s.rows.size() / 4);
    (upper ? s.nup : s.nlp) = cur + 1;
  }
  return true;
}

bool plan_sweep(const KAnalysis& ka, bool wide, int64_t max_entries, KSweep* out) {
  // A part is one launch (2.3 us at a few hundred rows, 4.3 us at 48,000); a
  // level of the one-work-group sweep takes 1.3-1.8 us, a level launch 4.3
  // us.  Longer rows make fewer parts; 64 entries are two rounds of a row's
  // eight lanes, past that the added entries cost what the launches save
  // (48,000-bus grid: 12 parts at 64, 26 MB per application).
  // Up to 2,048 rows the level sweep's vector fits a quarter of a CU's LDS
  // and a batch overlaps its instances in one launch of 23-44 us (512 grids
  // of 100-600 buses: 25.0 ms by levels, 26.6 ms in parts; 256 of 150-3,000
  // with the line at 1,024 rows: 26.7 and 29.6 ms); above, the same solves
  // gain in parts alone and batched (3,000 buses 5.3 -> 3.8 ms, 16 grids of
  // 10,000 19.5 -> 13.8 ms).  A
  // factor of more updates than half its blocks (three-phase feeders:
  // triangles between the phases) gives entries of many terms, whose set-up
  // each Newton step outweighs the few applications such a solve takes
  // (300-bus feeder: 1.89 ms by levels, 2.02 ms in parts).
  if (ka.nu <= 2048 || 2 * ka.nup() > ka.nnz()) return false;
  const int levels = (int)(ka.lev_ptr.size() + ka.ulev_ptr.size()) - 2;
  for (int cap : {64, 32, 16}) {
    if (!build_sweep(ka, cap, max_entries, out)) continue;
    const int parts = out->nlp + out->nup;
    if (wide ? parts < levels : 3 * parts <= levels) return true;
  }
  *out = KSweep();
  return false;
}

}  // namespace pfh
