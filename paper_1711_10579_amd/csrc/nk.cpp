// Newton-Krylov inner solve (Sec. III-B) on the host side: the case's Krylov
// storage, the batch's launch lists, and the Newton step that drives the
// batched GMRES kernels (krylov.hip).
//
// The number of Arnoldi steps an instance needs is decided on the device.
// After every step the host reads the instances' Krylov states: it ends the
// cycle of the instances that asked for it (solution update, restart or
// result) and launches the next step for the others, until none iterates.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstring>

#include "internal.hpp"
#include "kernels.hpp"
#include "parallel.hpp"

namespace pfi {

namespace {

template <typename T>
size_t carve_bytes(int64_t count) {
  return ((size_t)std::max<int64_t>(count, 0) * sizeof(T) + 255) & ~(size_t)255;
}

template <typename T>
T* carve(char*& p, int64_t count) {
  T* r = (T*)p;
  p += carve_bytes<T>(count);
  return r;
}

}  // namespace

void free_krylov(Case* c) {
  if (c->kbase && c->kown) {
    c->ctx->dfree(c->kbase);
    c->bytes -= c->kbytes;
  }
  c->kbase = nullptr;
  c->kbytes = 0;
  c->kown = false;
  c->km = 0;
}

void detach_krylov(Case* c) {
  if (c->kbase && !c->kown) {
    c->kbase = nullptr;
    c->kbytes = 0;
    c->km = 0;
  }
}

namespace {

int krylov_m(int m) { return std::max(m, 30); }

}  // namespace

bool krylov_wide(const pfh::KAnalysis& ka) {
  for (size_t l = 0; l + 1 < ka.lev_ptr.size(); ++l)
    if (ka.lev_ptr[l + 1] - ka.lev_ptr[l] > 4096) return true;
  for (size_t l = 0; l + 1 < ka.ulev_ptr.size(); ++l)
    if (ka.ulev_ptr[l + 1] - ka.ulev_ptr[l] > 4096) return true;
  return false;
}

size_t krylov_bytes(const Case* c, int m) {
  if (!c->ka) return 0;
  const pfh::KAnalysis& ka = *c->ka;
  const int km = krylov_m(m);
  const int nu = ka.nu;
  const int64_t knnz = ka.nnz(), nup = ka.nup();
  const int nb = ka.nblocks();
  const int kchunks = (nu + pfd::KCH - 1) / pfd::KCH;
  const int64_t n2 = 2LL * nu;
  const int64_t nh = (int64_t)(km + 1) * km + 2LL * km + (km + 1) + km;
  const int nl = (int)ka.lev_ptr.size() - 1, nul = (int)ka.ulev_ptr.size() - 1;
  size_t total = carve_bytes<int>(nu) + carve_bytes<int>(nu + 1) + carve_bytes<int>(knnz) + carve_bytes<int>(nu) +
                 carve_bytes<int>(c->nnz) + carve_bytes<int>(knnz + 1) + 2 * carve_bytes<int>(nup) +
                 carve_bytes<int>(nb + 1) + 2 * carve_bytes<int>(nu) + carve_bytes<int64_t>(nb + 1);
  total += carve_bytes<int>(nl + 1) + carve_bytes<int>(nul + 1) + 2 * carve_bytes<int4>(nu) + carve_bytes<int>(nb);
  total += 2 * carve_bytes<double>(4 * knnz) + carve_bytes<double>(4LL * nu) + carve_bytes<double>(ka.bj_off.back()) +
           carve_bytes<double>((km + 1) * n2) + 3 * carve_bytes<double>(n2);
  total += carve_bytes<double>(nh) + carve_bytes<double>(3LL * std::max(kchunks, 1) * (km + 1)) +
           carve_bytes<pfd::KState>(1);
  return total;
}

bool attach_krylov(Case* c, int m, char* base, bool own, hipStream_t s) {
  if (c->kbase && c->kown && !own) free_krylov(c);  // too small for this request: replaced by the lent storage
  const pfh::KAnalysis& ka = *c->ka;
  const int km = krylov_m(m);
  const int nu = ka.nu;
  const int64_t knnz = ka.nnz(), nup = ka.nup();
  const int nb = ka.nblocks();
  const int kchunks = (nu + pfd::KCH - 1) / pfd::KCH;
  const int64_t n2 = 2LL * nu;
  const int64_t nh = (int64_t)(km + 1) * km + 2LL * km + (km + 1) + km;
  const int nl = (int)ka.lev_ptr.size() - 1, nul = (int)ka.ulev_ptr.size() - 1;
  const size_t total = krylov_bytes(c, m);
  char* p = base;
  pfd::Inst& h = c->hinst;
  int* kp_of_r = carve<int>(p, nu);
  int* krow_ptr = carve<int>(p, nu + 1);
  int* kcol = carve<int>(p, knnz);
  int* kdiag = carve<int>(p, nu);
  int* kmap = carve<int>(p, c->nnz);
  int* kup_ptr = carve<int>(p, knnz + 1);
  int* kup_q = carve<int>(p, nup);
  int* kup_s = carve<int>(p, nup);
  int* bj_ptr = carve<int>(p, nb + 1);
  int* bj_rows = carve<int>(p, nu);
  int* bj_loc = carve<int>(p, nu);
  int64_t* bj_off = carve<int64_t>(p, nb + 1);
  int* kl_ptr = carve<int>(p, nl + 1);
  int* ku_ptr = carve<int>(p, nul + 1);
  int4* kl_info = carve<int4>(p, nu);
  int4* ku_info = carve<int4>(p, nu);
  h.bjbad = carve<int>(p, nb);
  h.jval = carve<double>(p, 4 * knnz);
  h.pval = carve<double>(p, 4 * knnz);
  h.pdinv = carve<double>(p, 4LL * nu);
  h.bjinv = carve<double>(p, ka.bj_off.back());
  h.kv = carve<double>(p, (km + 1) * n2);
  h.kw = carve<double>(p, n2);
  h.kz = carve<double>(p, n2);
  h.kx = carve<double>(p, n2);
  h.kh = carve<double>(p, nh);
  h.kpart = carve<double>(p, 3LL * std::max(kchunks, 1) * (km + 1));
  h.ks = carve<pfd::KState>(p, 1);
  if ((size_t)(p - base) != total) {
    set_error("pf_solve: internal Krylov layout error");
    return false;
  }
  h.km = km;
  h.kchunks = kchunks;
  h.knb = nb;
  h.kp_of_r = kp_of_r;
  h.krow_ptr = krow_ptr;
  h.kcol = kcol;
  h.kdiag = kdiag;
  h.kmap = kmap;
  h.kup_ptr = kup_ptr;
  h.kup_q = kup_q;
  h.kup_s = kup_s;
  h.bj_ptr = bj_ptr;
  h.bj_rows = bj_rows;
  h.bj_loc = bj_loc;
  h.bj_off = bj_off;
  h.knl = nl;
  h.knul = nul;
  h.kwide = krylov_wide(ka) ? 1 : 0;
  h.kl_ptr = kl_ptr;
  h.kl_info = kl_info;
  h.ku_ptr = ku_ptr;
  h.ku_info = ku_info;

  // the sources stay alive with the case (the copies are asynchronous)
  if (c->k_linfo.empty() && nu > 0) {
    c->k_linfo.resize(nu);
    c->k_uinfo.resize(nu);
    for (int k = 0; k < nu; ++k) {
      const int r = ka.lev_rows[k];
      c->k_linfo[k] = make_int4(r, ka.row_ptr[r], ka.diag[r], 0);
      const int u = ka.ulev_rows[k];
      c->k_uinfo[k] = make_int4(u, ka.diag[u] + 1, ka.row_ptr[u + 1], 0);
    }
  }
  bool ok = true;
  auto up = [&](void* dst, const void* src, size_t bytes) {
    if (bytes) ok &= hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s) == hipSuccess;
  };
  up(kp_of_r, ka.p_of_r.data(), sizeof(int) * nu);
  up(krow_ptr, ka.row_ptr.data(), sizeof(int) * (nu + 1));
  up(kcol, ka.col.data(), sizeof(int) * knnz);
  up(kdiag, ka.diag.data(), sizeof(int) * nu);
  up(kmap, c->kmap_host.data(), sizeof(int) * c->nnz);
  up(kup_ptr, ka.up_ptr.data(), sizeof(int) * (knnz + 1));
  up(kup_q, ka.up_q.data(), sizeof(int) * nup);
  up(kup_s, ka.up_s.data(), sizeof(int) * nup);
  up(bj_ptr, ka.bj_ptr.data(), sizeof(int) * (nb + 1));
  up(bj_rows, ka.bj_rows.data(), sizeof(int) * nu);
  up(bj_loc, ka.bj_loc.data(), sizeof(int) * nu);
  up(bj_off, ka.bj_off.data(), sizeof(int64_t) * (nb + 1));
  up(kl_ptr, ka.lev_ptr.data(), sizeof(int) * (nl + 1));
  up(ku_ptr, ka.ulev_ptr.data(), sizeof(int) * (nul + 1));
  up(kl_info, c->k_linfo.data(), sizeof(int4) * nu);
  up(ku_info, c->k_uinfo.data(), sizeof(int4) * nu);
  static_assert(sizeof(pfd::KState) % 4 == 0, "KState is cleared as 32-bit words");
  pfd::launch_zero_words(s, h.ks, (int64_t)(sizeof(pfd::KState) / 4));
  pfd::launch_set_inst(s, c->d_inst, h);
  if (!ok || hipGetLastError() != hipSuccess) {
    set_error("pf_solve: upload of the Krylov storage failed");
    return false;
  }
  c->kbase = base;
  c->kbytes = total;
  c->kown = own;
  c->km = km;
  if (own) c->bytes += total;
  return true;
}

bool ensure_krylov(Case* c, int m) {
  if (c->kbase && c->km >= m) return true;
  if (!c->ka) {
    set_error("pf_solve: the case has no Krylov analysis");
    return false;
  }
  Ctx* ctx = c->ctx;
  if (hipStreamSynchronize(ctx->stream) != hipSuccess) {
    set_error("pf_solve: device failure before the Krylov set-up");
    return false;
  }
  if (c->kbase && !c->kown) {
    set_error("pf_solve: lent Krylov storage is too small");
    return false;
  }
  free_krylov(c);
  const size_t total = krylov_bytes(c, m);
  char* base = (char*)ctx->dalloc(total);
  if (!base) {
    set_error("pf_solve: device allocation of the Krylov storage failed");
    return false;
  }
  if (!attach_krylov(c, m, base, true, ctx->stream) || hipStreamSynchronize(ctx->stream) != hipSuccess) {
    ctx->dfree(base);
    c->kbase = nullptr;
    c->kbytes = 0;
    c->km = 0;
    set_error("pf_solve: set-up of the Krylov storage failed");
    return false;
  }
  return true;
}

namespace {

// Work-groups without a chunk past which a batch's chunks go by a list (one more
// load at the start of a work-group).  With four lanes a row such a work-group
// is 16 waves to start: 512 grids of 100-5,000 buses (7,626 of 10,240 without)
// with block-Jacobi GMRES 71.5 -> 65.5 ms and BiCGStab 45.1 -> 40.1, with ILU(0)
// 31.5 -> 29.6 and 29.5 -> 28.8; 16 of 500-10,000 (400 of 608) 14.7 -> 14.4 and
// 6.5 -> 6.3; 32 of 150-3,000 (208 of 352, by the grid) the same either way.
constexpr int64_t kEmptyChunks = 256;

}  // namespace

bool Batch::build_krylov() {
  std::vector<int2> work;
  kchunks = {};
  kchunks.nslots = nslots;
  k_blocks_big = 0;
  for (Case* c : cases) {
    if (!c->ka) return false;
    const int nc = (c->ka->nu + pfd::KCH - 1) / pfd::KCH;
    kchunks.most = std::max(kchunks.most, nc);
    kchunks.count += nc;
    kchunks.rows += c->ka->nu;
  }
  {
    // the groups above the small size first (a work-group each), then the
    // small ones (a wave each for their inverse, four to a wave when
    // applied), in fours of one instance, padded with entries of group -1
    const int64_t off = (int64_t)work.size();
    const int small = pfd::bj_small_nodes();
    for (int pass = 0; pass < 2; ++pass) {
      for (int s = 0; s < nslots; ++s) {
        const pfh::KAnalysis& ka = *cases[s]->ka;
        for (int b = 0; b < ka.nblocks(); ++b)
          if ((ka.bj_ptr[b + 1] - ka.bj_ptr[b] > small) == (pass == 0)) work.push_back(make_int2(s, b));
        if (pass == 1)
          while (((int64_t)work.size() - off - k_blocks_big) % 4 != 0) work.push_back(make_int2(s, -1));
      }
      if (pass == 0) k_blocks_big = (int)((int64_t)work.size() - off);
    }
    k_blocks = {off, (int)((int64_t)work.size() - off)};
  }
  // the chunks by a list where a grid of the most chunks for every instance would
  // hold many work-groups without one
  const int64_t chunks_off = (int64_t)work.size();
  const bool list = (int64_t)kchunks.most * nslots - kchunks.count > kEmptyChunks;
  for (int s = 0; list && s < nslots; ++s)
    for (int k = 0; k * pfd::KCH < cases[s]->ka->nu; ++k) work.push_back(make_int2(s, k));
  const size_t bw = (sizeof(int2) * std::max<size_t>(work.size(), 1) + 255) & ~(size_t)255;
  if (kmem) ctx->dfree(kmem);
  kmem = (char*)ctx->dalloc(bw);
  kbytes = kmem ? bw : 0;
  if (!kmem) return false;
  d_kwork = (int2*)kmem;
  if (list) kchunks.list = d_kwork + chunks_off;
  hipStream_t st = stream;
  bool ok = true;
  if (!work.empty())
    ok &= hipMemcpyAsync(d_kwork, work.data(), sizeof(int2) * work.size(), hipMemcpyHostToDevice, st) == hipSuccess;
  ok &= hipStreamSynchronize(st) == hipSuccess;
  kbuilt = ok;
  return ok;
}

namespace {

// The index lists of the cases' sweep plans on the device, with one
// synchronisation for all; a case that gets no memory sweeps by levels.
// False on a device failure: nothing of these plans stays, since the kernels
// index with the lists.
bool upload_sweeps(const std::vector<Case*>& cases, hipStream_t s) {
  struct Up {
    Case* c;
    char* base;
    size_t bytes;
    pfd::Inst h;
  };
  std::vector<Up> ups;
  bool ok = true;
  for (Case* c : cases) {
    if (c->sw_state != Case::SW_HOST) continue;
    const int64_t nu = c->ka->nu, ne = c->sw.ne(), nops = c->sw.nops();
    Up u;
    u.c = c;
    u.bytes = carve_bytes<int4>(2 * nu) + carve_bytes<int>(ne) + carve_bytes<int>(ne + 1) + carve_bytes<int2>(nops);
    u.base = (char*)c->ctx->dalloc(u.bytes);
    if (!u.base) {
      (void)hipGetLastError();  // else the next launch would be held to have failed
      c->sw = pfh::KSweep();
      c->sw_state = Case::SW_NONE;
      continue;
    }
    u.h = c->hinst;
    char* p = u.base;
    auto put = [&](const std::vector<int>& src) {
      int* d = carve<int>(p, (int64_t)src.size());
      if (!src.empty())
        ok &= hipMemcpyAsync(d, src.data(), sizeof(int) * src.size(), hipMemcpyHostToDevice, s) == hipSuccess;
      return (const int*)d;
    };
    u.h.sw_rows = (const int4*)put(c->sw.rows);
    u.h.sw_col = put(c->sw.col);
    u.h.sw_op_ptr = put(c->sw.op_ptr);
    u.h.sw_ops = (const int2*)put(c->sw.ops);
    if (ok) pfd::launch_set_inst(s, c->d_inst, u.h);
    ups.push_back(u);
  }
  if (ups.empty()) return true;
  ok &= hipGetLastError() == hipSuccess && hipStreamSynchronize(s) == hipSuccess;
  if (!ok)
    for (const Up& u : ups) pfd::launch_set_inst(s, u.c->d_inst, u.c->hinst);
  if (!ok) (void)hipStreamSynchronize(s);
  if (!ok) (void)hipGetLastError();
  for (const Up& u : ups) {
    Case* c = u.c;
    if (!ok) {
      c->ctx->dfree(u.base);
      continue;
    }
    c->hinst = u.h;
    c->swbase = u.base;
    c->swbytes = u.bytes;
    // the launch lists need the plan's rows and steps only
    c->sw.col = c->sw.op_ptr = c->sw.ops = std::vector<int>();
    c->sw_state = Case::SW_PLAN;
  }
  return ok;
}

}  // namespace

bool Batch::plan_ilu() {
  int64_t rows = 0;
  for (Case* c : cases) {
    if (!c->ka) return false;
    rows += c->ka->nu;
  }
  ilu_host.assign(nslots, IluHost());
  // a thread pays for itself from some thousands of rows (10,000 buses: 1.7 ms
  // for the plan of a case, 0.3 ms for its targets)
  const int threads = (int)std::min<int64_t>(8, 1 + rows / 2048);
  try {
    pfh::parallel_for(2 * nslots, threads, [&](int i) {
      Case* c = cases[i / 2];
      const pfh::KAnalysis& ka = *c->ka;
      IluHost& h = ilu_host[i / 2];
      if (i % 2) {
        pfh::factor_targets(ka, &h.ptr, &h.tgt);
        return;
      }
      // the entry values take the place of the block-Jacobi inverses
      if (c->sw_state == Case::SW_NEW)
        c->sw_state = pfh::plan_sweep(ka, krylov_wide(ka), ka.bj_off.back() / 4, &c->sw, nslots == 1 ? 2 : 1)
                          ? Case::SW_HOST
                          : Case::SW_NONE;
      if (c->sw_state == Case::SW_NONE) return;
      // the positions by their step
      const auto& step = c->sw.step;
      h.step_ptr.assign(c->sw.nsteps + 1, 0);
      for (int t : step) h.step_ptr[t + 1]++;
      for (int t = 0; t < c->sw.nsteps; ++t) h.step_ptr[t + 1] += h.step_ptr[t];
      std::vector<int> fill(h.step_ptr.begin(), h.step_ptr.end() - 1);
      h.step_pos.resize(step.size());
      for (int k = 0; k < (int)step.size(); ++k) h.step_pos[fill[step[k]]++] = k;
    });
  } catch (const std::exception&) {
    ilu_host.clear();
    return false;
  }
  return true;
}

namespace {

// Levels of up to this many targets run behind barriers of one work-group (a
// pass of 512 targets takes about 1.2 us, a launch of its own 4.5 us).
constexpr int kNarrowTargets = 1536;
// A batch of many instances has the chip full in any case, and a launch of its
// own for the wide levels of some holds up the others (512 grids of 100-5,000
// buses: 219 and 130 us, with every level behind barriers 204; 64 of 1,000-5,000
// 17.5 -> 16.8 ms a GMRES solve; 32 of 150-3,000 the same either way).
constexpr int kManyInstances = 64;

}  // namespace

bool Batch::build_ilu() {
  if (ilu_host.empty() && !plan_ilu()) return false;
  const std::vector<IluHost> host = std::move(ilu_host);
  ilu_host.clear();
  if (!upload_sweeps(cases, stream)) return false;
  std::vector<int2> work;
  for (auto* v : {&f_seg, &s_low, &s_up, &s_step, &s_lev, &s_ulev}) v->clear();
  s_narrow = false;
  s_min_nu = s_max_nu = 0;
  // factor targets and levels of every instance, its launches' descriptors
  std::vector<int> tgt, lev;
  {
    size_t nt = 0, nl = 0, nw = 0;
    for (int s = 0; s < nslots; ++s) {
      nt += host[s].tgt.size();
      nl += host[s].ptr.size();
      // rows of the steps and parts, each padded for an instance
      if (cases[s]->sw_state == Case::SW_PLAN)
        nw += 2 * cases[s]->sw.step.size() + 32 * (cases[s]->sw.part_ptr.size() + cases[s]->sw.nsteps);
    }
    tgt.reserve(nt);
    lev.reserve(nl);
    work.reserve(nw);
  }
  std::vector<std::vector<int4>> seg;
  int nlp = 0, nup = 0, nst = 0;
  size_t max_l = 0, max_u = 0;
  // each instance takes its own path, whatever the batch holds
  std::vector<char> by_level(nslots, 0);
  const int narrow = nslots < kManyInstances ? kNarrowTargets : INT_MAX;
  for (int s = 0; s < nslots; ++s) {
    Case* c = cases[s];
    const pfh::KAnalysis& ka = *c->ka;
    const std::vector<int>&ptr = host[s].ptr, &one = host[s].tgt;
    const int t0 = (int)tgt.size(), l0 = (int)lev.size(), nl = (int)ptr.size() - 1;
    tgt.insert(tgt.end(), one.begin(), one.end());
    for (int p : ptr) lev.push_back(t0 + p);
    size_t k = 0;
    for (int l = 0; l < nl; ++k) {
      if (seg.size() <= k) seg.emplace_back();
      int e = l;
      while (e < nl && ptr[e + 1] - ptr[e] <= narrow) ++e;
      if (e > l) {
        seg[k].push_back(make_int4(s, l0 + l, l0 + e, 1));
        l = e;
      } else {
        const int per = pfd::ilu_factor_threads();
        for (int i = ptr[l]; i < ptr[l + 1]; i += per)
          seg[k].push_back(make_int4(s, t0 + i, t0 + std::min(i + per, ptr[l + 1]), 0));
        ++l;
      }
    }
    if (c->sw_state == Case::SW_PLAN) {
      nlp = std::max(nlp, c->sw.nlp);
      nup = std::max(nup, c->sw.nup);
      nst = std::max(nst, c->sw.nsteps);
    } else if (krylov_wide(ka)) {
      by_level[s] = 1;
      max_l = std::max(max_l, ka.lev_ptr.size() - 1);
      max_u = std::max(max_u, ka.ulev_ptr.size() - 1);
    } else {
      s_min_nu = s_narrow ? std::min(s_min_nu, ka.nu) : ka.nu;
      s_max_nu = std::max(s_max_nu, ka.nu);
      s_narrow = true;
    }
  }
  const size_t per = (size_t)pfd::sweep_rows_per_group();
  auto list = [&](std::vector<std::pair<int64_t, int>>* out, auto&& positions) {
    const size_t off = work.size();
    for (int s = 0; s < nslots; ++s) {
      if (cases[s]->sw_state != Case::SW_PLAN) continue;
      positions(s, cases[s]->sw);
      while ((work.size() - off) % per != 0) work.push_back(make_int2(s, -1));
    }
    out->emplace_back((int64_t)off, (int)(work.size() - off));
  };
  auto parts = [&](int np, bool upper, std::vector<std::pair<int64_t, int>>* out) {
    for (int p = 0; p < np; ++p) {
      if (nslots == 1) {  // positions of the only instance, no list
        const int* pp = &cases[0]->sw.part_ptr[upper ? nlp + p : p];
        out->emplace_back(pp[0], pp[1] - pp[0]);
        continue;
      }
      list(out, [&](int s, const pfh::KSweep& sw) {
        if (p >= (upper ? sw.nup : sw.nlp)) return;
        const int* pp = &sw.part_ptr[upper ? sw.nlp + p : p];
        for (int k = pp[0]; k < pp[1]; ++k) work.push_back(make_int2(s, k));
      });
    }
  };
  parts(nlp, false, &s_low);
  parts(nup, true, &s_up);
  for (int t = 0; t < nst; ++t)
    list(&s_step, [&](int s, const pfh::KSweep& sw) {
      if (t >= sw.nsteps) return;
      for (int k = host[s].step_ptr[t]; k < host[s].step_ptr[t + 1]; ++k)
        work.push_back(make_int2(s, host[s].step_pos[k]));
    });
  auto levels = [&](bool upper, size_t nl, std::vector<std::pair<int64_t, int>>* out) {
    for (size_t l = 0; l < nl; ++l) {
      const int64_t off = (int64_t)work.size();
      for (int s = 0; s < nslots; ++s) {
        if (!by_level[s]) continue;
        const pfh::KAnalysis& ka = *cases[s]->ka;
        const auto& lp = upper ? ka.ulev_ptr : ka.lev_ptr;
        const auto& rows = upper ? ka.ulev_rows : ka.lev_rows;
        if (l + 1 >= lp.size()) continue;
        for (int k = lp[l]; k < lp[l + 1]; ++k) work.push_back(make_int2(s, rows[k]));
      }
      out->emplace_back(off, (int)((int64_t)work.size() - off));
    }
  };
  levels(false, max_l, &s_lev);
  levels(true, max_u, &s_ulev);
  std::vector<int4> desc;
  for (const auto& v : seg) {
    f_seg.emplace_back((int64_t)desc.size(), (int)v.size());
    desc.insert(desc.end(), v.begin(), v.end());
  }
  // the lists packed on the host as on the device: one copy
  const size_t total = carve_bytes<int2>((int64_t)work.size()) + carve_bytes<int4>((int64_t)desc.size()) +
                       carve_bytes<int>((int64_t)tgt.size()) + carve_bytes<int>((int64_t)lev.size());
  if (smem) ctx->dfree(smem);
  smem = (char*)ctx->dalloc(std::max<size_t>(total, 256));
  sbytes = smem ? std::max<size_t>(total, 256) : 0;
  if (!smem) return false;
  std::vector<char> pack(total);
  char* p = smem;
  auto put = [&](const auto& src) {
    typedef typename std::decay_t<decltype(src)>::value_type V;
    if (!src.empty()) std::memcpy(pack.data() + (p - smem), src.data(), sizeof(V) * src.size());
    return carve<V>(p, (int64_t)src.size());
  };
  d_swork = put(work);
  d_fdesc = put(desc);
  d_ftgt = put(tgt);
  d_flev = put(lev);
  bool ok = true;
  if (total) ok &= hipMemcpyAsync(smem, pack.data(), total, hipMemcpyHostToDevice, stream) == hipSuccess;
  ok &= hipStreamSynchronize(stream) == hipSuccess;
  sbuilt = ok;
  return ok;
}

template <typename T>
void precond_setup(Batch* b, bool ilu) {
  hipStream_t s = b->stream;
  const auto* I = b->d_insts;
  if (ilu) {
    for (const auto& l : b->f_seg)
      pfd::launch_ilu_factor<T>(s, I, b->d_fdesc + l.first, l.second, b->d_ftgt, b->d_flev);
    pfd::launch_ilu_scale<T>(s, I, b->kchunks);
    for (const auto& l : b->s_step) pfd::launch_sweep_values<T>(s, I, b->d_swork + l.first, l.second);
  } else {
    pfd::launch_bj_inv<T>(s, I, b->d_kwork + b->k_blocks.first, b->k_blocks_big,
                          b->k_blocks.second - b->k_blocks_big);
  }
}

template <typename T>
void precond_apply(Batch* b, bool ilu, int mode) {
  hipStream_t s = b->stream;
  const auto* I = b->d_insts;
  const int ns = b->nslots;
  if (ilu) {
    auto part = [&](const std::pair<int64_t, int>& l, int upper) {
      if (ns == 1)
        pfd::launch_sweep_part<T>(s, I, nullptr, (int)l.first, l.second, upper, mode);
      else
        pfd::launch_sweep_part<T>(s, I, b->d_swork + l.first, 0, l.second, upper, mode);
    };
    // the instances without a plan, by levels, the narrow ones beside the others'
    // first part
    size_t first = 0;
    if (b->s_narrow) {
      const bool beside = ns > 1 && !b->s_low.empty();
      pfd::launch_ilu_apply_wg<T>(s, I, ns, mode, b->s_min_nu, b->s_max_nu,
                                  beside ? b->d_swork + b->s_low[0].first : nullptr, beside ? b->s_low[0].second : 0);
      first = beside;
    }
    for (size_t k = first; k < b->s_low.size(); ++k) part(b->s_low[k], 0);
    for (const auto& l : b->s_up) part(l, 1);
    for (const auto& l : b->s_lev) pfd::launch_ilu_fwd<T>(s, I, b->d_swork + l.first, l.second, mode);
    for (const auto& l : b->s_ulev) pfd::launch_ilu_bwd<T>(s, I, b->d_swork + l.first, l.second, mode);
  } else {
    pfd::launch_bj_apply<T>(s, I, b->d_kwork + b->k_blocks.first, b->k_blocks_big, b->k_blocks.second, mode);
  }
}

template void precond_setup<double>(Batch*, bool);
template void precond_setup<float>(Batch*, bool);
template void precond_apply<double>(Batch*, bool, int);
template void precond_apply<float>(Batch*, bool, int);

namespace {

template <typename T>
pf_status nk_step_t(Batch* b, const pf_options* opt) {
  Ctx* ctx = b->ctx;
  hipStream_t s = b->stream;
  const auto* I = b->d_insts;
  for (Case* c : b->cases)
    if (!ensure_krylov(c, opt->gmres_m)) return PF_E_NOMEM;
  if (!b->kbuilt && !b->build_krylov()) {
    set_error("pf_solve: Krylov batch set-up failed");
    return PF_E_NOMEM;
  }
  pfd::KOpts ko;
  ko.eta_max = opt->eta_max;
  ko.eta_floor = opt->precision == PF_PREC_MIXED ? 1e-6 : 1e-12;
  ko.m = opt->gmres_m;
  ko.max_restarts = opt->gmres_max_restarts;
  const bool ilu = opt->precond == PF_PRECOND_ILU0;
  const int ns = b->nslots;
  const pfd::KChunks& kc = b->kchunks;
  {
    Prof p(ctx, PF_K_JFILL, 0.0, 0.0);
    pfd::launch_kfill<T>(s, I, ns, b->max_nnz, ilu ? 1 : 0);
  }
  {
    Prof p(ctx, PF_K_PRECOND_SETUP, 0.0, 0.0);
    precond_setup<T>(b, ilu);
  }
  const bool bcg = opt->solver == PF_SOLVER_BICGSTAB;
  {
    Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
    if (bcg) {
      pfd::launch_bcg_begin<T>(s, I, kc, ko);
      pfd::launch_bcg_dir<T>(s, I, kc);  // p = r = r0 = F
    } else
      pfd::launch_kbegin<T>(s, I, kc, ko);
    pfd::launch_kfinish<T>(s, I, kc);
  }
  auto apply = [&](int mode) {
    Prof p(ctx, PF_K_PRECOND_APPLY, 0.0, 0.0);
    precond_apply<T>(b, ilu, mode);
  };
  // Iterations (BiCGStab) or Arnoldi steps (GMRES) queued per read of the
  // instances' Krylov states: first as many as the inner solve at this
  // Newton step took in the batch's last solve, then the rest of that count
  // up to 8 at a time, or 2 at a time once it is passed.  An instance that
  // finishes within a run skips the rest of it.
  std::vector<int> st(ns), tot(ns);
  int queued = 0;
  const size_t step_k = (size_t)b->nk_step_index++;
  const int guess = step_k < b->k_inner.size() ? b->k_inner[step_k]
                    : b->k_inner.empty()       ? 8
                                               : b->k_inner.back();
  auto run_length = [&](int done) {
    if (queued == 0) return std::max(1, std::min(guess, 64));
    return guess > done ? std::min(guess - done, 8) : 2;
  };
  auto remember = [&](int most) {
    if (queued == 0) return;
    if (b->k_inner.size() <= step_k) b->k_inner.resize(step_k + 1, 8);
    b->k_inner[step_k] = std::max(1, most);
  };
  const int64_t guard_max = (int64_t)(opt->gmres_max_restarts + 1) * (opt->gmres_m + 2) + 4;
  for (int64_t guard = 0;; ++guard) {
    if (guard > guard_max) {
      set_error("pf_solve: the Krylov inner solve did not settle");
      return PF_E_DEVICE;
    }
    // the gather writes straight into pinned host memory
    pfd::launch_kgather(s, I, ns, b->h_kstate);
    if (hipStreamSynchronize(s) != hipSuccess) {
      set_error("pf_solve: device failure in the Krylov inner solve");
      return PF_E_DEVICE;
    }
    std::memcpy(st.data(), b->h_kstate, sizeof(int) * ns);
    std::memcpy(tot.data(), b->h_kstate + ns, sizeof(int) * ns);
    int most = 0;
    for (int i = 0; i < ns; ++i) most = std::max(most, tot[i]);
    if (bcg) {
      bool any = false;
      for (int v : st) any |= v == pfd::KS_BP || v == pfd::KS_BS || v == pfd::KS_BH;
      if (!any) {
        remember(most);
        break;
      }
      // a run of BiCGStab iterations between two reads of the states (each
      // kernel acts only on the instances in the state it serves)
      const int run = run_length(most);
      queued += run;
      for (int i = 0; i < run; ++i) {
        // the iteration's index in the inner solve: every instance still
        // iterating has done exactly that many
        const int it = queued - run + i;
        apply(2);
        {
          Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
          pfd::launch_bcg_half<T>(s, I, kc, it);
        }
        apply(3);
        Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
        pfd::launch_bcg_end<T>(s, I, kc, ko, it);
      }
      Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
      pfd::launch_kfinish<T>(s, I, kc);
      continue;
    }
    bool iter = false, cyc = false;
    for (int v : st) {
      iter |= v == pfd::KS_ITER;
      cyc |= v == pfd::KS_CYCLE;
    }
    if (!iter && !cyc) {
      remember(most);
      break;
    }
    // a run of Arnoldi steps, then the end of every cycle they complete,
    // between two reads of the states: each kernel acts only on the
    // instances in the state it serves, so an instance whose cycle ends
    // within the run skips its remaining steps
    // (a run ends with the current cycle: steps past it would be skipped)
    const int left = ko.m - most % std::max(ko.m, 1);
    const int run = iter ? std::max(1, std::min(run_length(most), left)) : 0;
    queued += std::max(run, 1);
    for (int i = 0; i < run; ++i) {
      apply(0);
      Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
      pfd::launch_karnoldi<T>(s, I, kc, ko);
    }
    {
      Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
      pfd::launch_kycomb<T>(s, I, kc);
    }
    apply(1);
    Prof p(ctx, PF_K_KRYLOV, 0.0, 0.0);
    pfd::launch_kcycle_end<T>(s, I, kc, ko);
    pfd::launch_kfinish<T>(s, I, kc);
  }
  {
    Prof p(ctx, PF_K_UPDATE, 0.0, 0.0);
    pfd::launch_update<T>(s, I, ns, b->max_nu);
  }
  return launch_status("pf_solve");
}

}  // namespace

pf_status nk_step(Batch* b, const pf_options* opt) {
  return opt->precision == PF_PREC_MIXED ? nk_step_t<float>(b, opt) : nk_step_t<double>(b, opt);
}

}  // namespace pfi
