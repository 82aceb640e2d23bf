// ILU(0) preconditioner (Sec. III-B): the factor's targets by level, and the
// parts of its sweeps: runs of levels whose rows are written out in terms of
// the part's input, so that an application is one launch per part instead of
// one barrier or launch per level.

#include <algorithm>
#include <cstdint>

#include "analysis.hpp"
#include "parallel.hpp"

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

namespace {

// One triangle's sweep: positions, entries and ops counted from its own start.
struct Half {
  std::vector<int> part_ptr, step, rows, col, op_ptr, ops;
  int parts = 0, nsteps = 0;
};

// Makes one triangle's parts; false past max_entries.
bool build_half(const KAnalysis& ka, bool upper, int cap, int64_t max_entries, Half* out) {
  Half& s = *out;
  s = Half();
  const int nu = ka.nu;
  const auto& ptr = upper ? ka.ulev_ptr : ka.lev_ptr;
  const auto& rows = upper ? ka.ulev_rows : ka.lev_rows;
  const int nl = (int)ptr.size() - 1;
  s.part_ptr.push_back(0);
  s.op_ptr.push_back(0);
  s.rows.resize(4 * (size_t)nu);
  s.step.resize(nu);
  // (more than the triangles of meshes need: untouched pages cost nothing,
  // growing copies)
  s.col.reserve(24 * (size_t)nu);
  s.op_ptr.reserve(24 * (size_t)nu);
  s.ops.reserve(48 * (size_t)nu);
  std::vector<int> pos_of(nu), part(nu, -1), where(2 * (size_t)nu, -1);
  // the rows of a level as found: entries (keys) and ops (entry, q, s)
  struct Row {
    int r, key0, key1, op0, op1;
  };
  struct Op {
    int e, q, s;
  };
  std::vector<Row> lrow;
  std::vector<int> keys, order, cnt;
  std::vector<Op> ops;
  int cur = -1, first = 0, pos = 0;  // current part and its first level
  for (int l = 0; l < nl; ++l) {
    // the level's rows inside the current part; when one grows past the cap,
    // again as the first level of a part of its own
    size_t nkeys = 0, nops = 0;
    for (int pass = l == 0 ? 1 : 0; pass < 2; ++pass) {
      if (pass == 1) {
        if (cur >= 0) s.part_ptr.push_back(pos);
        ++cur;
        first = l;
      }
      lrow.clear();
      nkeys = nops = 0;
      bool fits = true;
      for (int k = ptr[l]; k < ptr[l + 1] && fits; ++k) {
        const int r = rows[k];
        const int q0 = upper ? ka.diag[r] + 1 : ka.row_ptr[r], q1 = upper ? ka.row_ptr[r + 1] : ka.diag[r];
        // room for the row: every entry of the rows it takes, one more each
        size_t most = 1;
        for (int q = q0; q < q1; ++q) {
          const int c = ka.col[q];
          most += part[c] != cur ? 1 : 1 + s.rows[4 * (size_t)pos_of[c] + 2] - s.rows[4 * (size_t)pos_of[c] + 1];
        }
        if (keys.size() < nkeys + most) keys.resize(2 * (nkeys + most));
        if (ops.size() < nops + most) ops.resize(2 * (nops + most));
        const int key0 = (int)nkeys, op0 = (int)nops;
        // key: 2 c for the part's input at row c, 2 c + 1 for an earlier row
        auto entry = [&](int key) {
          int& w = where[key];
          if (w < key0) {
            w = (int)nkeys;
            keys[nkeys++] = key;
          }
          return w - key0;
        };
        if (upper) entry(2 * r);  // the row's own entry, without ops
        for (int q = q0; q < q1; ++q) {
          const int c = ka.col[q];
          if (part[c] != cur) {
            ops[nops++] = {entry(2 * c + 1), q, -1};
            continue;
          }
          if (!upper) ops[nops++] = {entry(2 * c), q, -1};  // the identity on y_c's own input
          const int* rc = &s.rows[4 * (size_t)pos_of[c]];
          for (int e = rc[1]; e < rc[2]; ++e) ops[nops++] = {entry(s.col[e] < 0 ? 2 * ~s.col[e] : 2 * s.col[e] + 1), q, e};
        }
        for (size_t e = key0; e < nkeys; ++e) where[keys[e]] = -1;
        lrow.push_back({r, key0, (int)nkeys, op0, (int)nops});
        fits = pass == 1 || (int)nkeys - key0 <= cap;
      }
      if (fits) break;
    }
    // a wave holds several rows: rows of like length beside each other, the
    // longest first (counted into place)
    int most = 0;
    for (const Row& w : lrow) most = std::max(most, w.key1 - w.key0);
    cnt.assign(most + 2, 0);
    for (const Row& w : lrow) cnt[most - (w.key1 - w.key0) + 1]++;
    for (int i = 0; i <= most; ++i) cnt[i + 1] += cnt[i];
    order.resize(lrow.size());
    for (size_t i = 0; i < lrow.size(); ++i) order[cnt[most - (lrow[i].key1 - lrow[i].key0)]++] = (int)i;
    size_t e0 = s.col.size(), o0 = s.ops.size() / 2;
    s.col.resize(e0 + nkeys);
    s.op_ptr.resize(e0 + nkeys + 1);
    s.ops.resize(2 * (o0 + nops));
    s.nsteps = std::max(s.nsteps, l - first + 1);
    for (int i : order) {
      const Row& w = lrow[i];
      const int len = w.key1 - w.key0;
      part[w.r] = cur;
      pos_of[w.r] = pos;
      int* row = &s.rows[4 * (size_t)pos];
      row[0] = w.r;
      row[1] = (int)e0;
      row[2] = (int)e0 + len;
      row[3] = 0;
      s.step[pos++] = l - first;
      // ops by entry, each entry's in the order found: counted in op_ptr, which
      // ends up holding each entry's end
      int* end = &s.op_ptr[e0 + 1];
      for (int e = 0; e < len; ++e) {
        const int key = keys[w.key0 + e];
        s.col[e0 + e] = key & 1 ? key >> 1 : ~(key >> 1);
        end[e] = 0;
      }
      for (int o = w.op0; o < w.op1; ++o) end[ops[o].e]++;
      int at = (int)o0;
      for (int e = 0; e < len; ++e) {
        const int n = end[e];
        end[e] = at;
        at += n;
      }
      for (int o = w.op0; o < w.op1; ++o) {
        int* op = &s.ops[2 * (size_t)end[ops[o].e]++];
        op[0] = ops[o].q;
        op[1] = ops[o].s;
      }
      o0 = at;
      e0 += len;
    }
    if ((int64_t)e0 > max_entries) return false;
  }
  if (cur >= 0) s.part_ptr.push_back(pos);
  s.parts = cur + 1;
  return true;
}

}  // namespace

bool build_sweep(const KAnalysis& ka, int cap, int64_t max_entries, KSweep* out, int threads) {
  KSweep& s = *out;
  s = KSweep();
  // the triangles need nothing from each other
  Half half[2];
  bool ok[2];
  parallel_for(2, threads, [&](int i) { ok[1 - i] = build_half(ka, i == 0, cap, max_entries, &half[1 - i]); });
  Half &low = half[0], &up = half[1];
  const int64_t ne = (int64_t)low.col.size(), nops = (int64_t)low.ops.size() / 2;
  if (!ok[0] || !ok[1] || ne + (int64_t)up.col.size() > max_entries) return false;
  s.nlp = low.parts;
  s.nup = up.parts;
  s.nsteps = std::max(low.nsteps, up.nsteps);
  s.part_ptr = std::move(low.part_ptr);
  s.step = std::move(low.step);
  s.rows = std::move(low.rows);
  s.col = std::move(low.col);
  s.op_ptr = std::move(low.op_ptr);
  s.ops = std::move(low.ops);
  for (size_t p = 1; p < up.part_ptr.size(); ++p) s.part_ptr.push_back(ka.nu + up.part_ptr[p]);
  s.step.insert(s.step.end(), up.step.begin(), up.step.end());
  for (size_t k = 0; k < up.rows.size(); k += 4) {
    up.rows[k + 1] += (int)ne;
    up.rows[k + 2] += (int)ne;
  }
  s.rows.insert(s.rows.end(), up.rows.begin(), up.rows.end());
  s.col.insert(s.col.end(), up.col.begin(), up.col.end());
  s.op_ptr.reserve(s.op_ptr.size() + up.op_ptr.size());
  for (size_t e = 1; e < up.op_ptr.size(); ++e) s.op_ptr.push_back((int)nops + up.op_ptr[e]);
  for (size_t o = 1; o < up.ops.size(); o += 2)
    if (up.ops[o] >= 0) up.ops[o] += (int)ne;
  s.ops.insert(s.ops.end(), up.ops.begin(), up.ops.end());
  return true;
}

bool plan_sweep(const KAnalysis& ka, bool wide, int64_t max_entries, KSweep* out, int threads) {
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
  // Where no update falls outside the pattern the factor is exact (a radial
  // grid; a mesh without triangles drops fill instead): an inner solve takes
  // one iteration, so its few applications carry neither long plans nor, where
  // the level sweeps run in one work-group, any.  Radial grids of 2,100, 3,000 and
  // 6,000 buses: 1.56, 0.92 and 4.1 ms a GMRES solve by levels, 1.80, 0.95 and 4.0
  // in parts, their first solve 2.0, 1.3 and 4.5 for 2.8, 2.2 and 6.0; of 20,000 (a
  // launch per level otherwise) 1.68 and 1.61 ms with rows of 8 and of 16 entries,
  // the first 3.9 and 9.3, by levels 3.0 and 4.8.
  int64_t updates = 0;  // of the entries in and outside the pattern
  for (int r = 0; r < ka.nu; ++r)
    for (int q = ka.row_ptr[r]; q < ka.diag[r]; ++q) updates += ka.row_ptr[ka.col[q] + 1] - ka.diag[ka.col[q]] - 1;
  const bool exact = ka.nup() == updates;
  if (exact && !wide) return false;
  const int levels = (int)(ka.lev_ptr.size() + ka.ulev_ptr.size()) - 2;
  for (int cap : {64, 32, 16, 8}) {
    if (exact != (cap == 8)) continue;
    if (!build_sweep(ka, cap, max_entries, out, threads)) continue;
    const int parts = out->nlp + out->nup;
    if (wide ? parts < levels : 3 * parts <= levels) return true;
  }
  *out = KSweep();
  return false;
}

}  // namespace pfh
