// Launchers of the device kernels (kernels.hip, dense.hip, krylov.hip).  All
// take the batch's device table of instance descriptors.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "device.hpp"

namespace pfd {

// descriptor upload (by value, stream-ordered) and a zero fill of 32-bit words
void launch_set_inst(hipStream_t, Inst* dst, const Inst& src);
void launch_zero_words(hipStream_t, void* p, int64_t words);

// Newton driver
void launch_init(hipStream_t, const Inst* const* insts, int nslots, int max_n, int flat);
void launch_start(hipStream_t, const Inst* const* insts, int nslots);
void launch_decide(hipStream_t, const Inst* const* insts, int nslots, DevOpts o);
void launch_gather_red(hipStream_t, const Inst* const* insts, int nslots, Red* out);
// voltages of n >= 1 nodes to pinned host memory, by blocks of kVoltBlock
// nodes that each set their flag to seq once stored
constexpr int kVoltBlock = 1024;
void launch_read_volt(hipStream_t, const double* v, int n, double* re, double* im, unsigned long long* flag,
                      unsigned long long seq);
// rows of more than kHeavyRow Ybus entries run one work-group each (max_heavy:
// the most such rows of an instance in the batch)
constexpr int kHeavyRow = 64;
void launch_mismatch(hipStream_t, const Inst* const* insts, int nslots, int max_n, int max_heavy);
template <typename T>
void launch_update(hipStream_t, const Inst* const* insts, int nslots, int max_nu);

// Jacobian fill: RHS copy, zero the factor storage (chunk items, see
// zero_chunk_values), scatter J
template <typename T>
void launch_fill(hipStream_t, const Inst* const* insts, int nslots, int max_nu2, const int2* zero_work, int nzero,
                 int max_nnz);
int zero_chunk_values();

// sparse part (G lanes per list).  Factor columns: (slot, position in the
// instance's level order) items, or positions of the only instance (work
// null), by class of lanes per column; wide: all in class 4, 1024 threads a
// column
template <typename T>
void launch_factor_cols(hipStream_t, const Inst* const* insts, const int2* work, const FacLevel& v, int wide);
// one stage of the upper levels' subtrees: `nbins` programs at
// words[bin_off[b]], each of at most kTreeLds words, `threads` (256 or 512)
// threads each
constexpr int kTreeLds = 16000;
template <typename T>
void launch_factor_trees(hipStream_t, const Inst* const* insts, const int* bin_off, const int* words, int nbins,
                         int threads);
template <typename T>
void launch_fwd_rows(hipStream_t, const Inst* const* insts, const int2* work, int nwork, int G);
template <typename T>
void launch_tail_schur(hipStream_t, const Inst* const* insts, const int2* work, int nwork, int G);

// dense trailing block
template <typename T>
void launch_dense_step(hipStream_t, const Inst* const* insts, const int2* work, int nwork, int nflag, int npanel,
                       int k0);
// backward solve of the whole factorisation in one launch: nd dense items
// (slot, w) (single: (slot, 0), one work-group per instance), then nrw
// work-groups of sparse rows, each described by work[nd + k] = (offset of its
// first row item in work, rows | G << 16), row items (slot, row); between the
// two, for the only instance, nbins programs at words[bin_off[b]] of at most
// kBwdLds bytes with their values
constexpr int kBwdLds = 72 * 1024;
template <typename T>
void launch_bwd_solve(hipStream_t, const Inst* const* insts, const int2* work, int nd, int nrw, int single,
                      int nbins, const int* bin_off, const int* words);

// The chunks of a batch's Krylov vectors: a list of all `count` {slot, chunk}, or
// (null) the `most` of an instance for every one of nslots; their rows.
struct KChunks {
  const int2* list;
  int count, most, nslots;
  int64_t rows;
};

// Newton-Krylov inner solve (krylov.hip); preconditioner mode 0 = Arnoldi
// step, 1 = end of a GMRES cycle, 2 and 3 = the halves of a BiCGStab
// iteration
template <typename T>
void launch_kfill(hipStream_t, const Inst* const* insts, int nslots, int max_nnz, int ilu);
// ILU(0) factor: work-group descriptors {slot, a, b, kind} (kind 0: targets
// tgt[a, b) of one level, ilu_factor_threads at a time; 1: levels a .. b - 1
// of the pointers lev into tgt), then the scaling of the lower blocks
int ilu_factor_threads();
template <typename T>
void launch_ilu_factor(hipStream_t, const Inst* const* insts, const int4* desc, int ngroups, const int* tgt,
                       const int* lev);
template <typename T>
void launch_ilu_scale(hipStream_t, const Inst* const* insts, const KChunks& c);
template <typename T>
void launch_bj_inv(hipStream_t, const Inst* const* insts, const int2* work, int nbig, int nsmall);
int bj_small_nodes();  // groups of at most this many nodes are inverted one per wave
template <typename T>
void launch_ilu_fwd(hipStream_t, const Inst* const* insts, const int2* work, int nwork, int mode);
template <typename T>
void launch_ilu_bwd(hipStream_t, const Inst* const* insts, const int2* work, int nwork, int mode);
// (work, nrows: rows of a forward part that run beside them, a list; 0: none)
template <typename T>
void launch_ilu_apply_wg(hipStream_t, const Inst* const* insts, int nslots, int mode, int min_nu, int max_nu,
                         const int2* work, int nrows);
template <typename T>
void launch_bj_apply(hipStream_t, const Inst* const* insts, const int2* work, int nbig, int nwork, int mode);
// ILU(0) sweeps in parts: rows of one launch are positions p0.. of the only
// instance (work null), or a list of (slot, position) padded with position -1
// to whole work-groups (sweep_rows_per_group rows) of one instance each
int sweep_rows_per_group();
template <typename T>
void launch_sweep_values(hipStream_t, const Inst* const* insts, const int2* work, int nrows);
template <typename T>
void launch_sweep_part(hipStream_t, const Inst* const* insts, const int2* work, int p0, int nrows, int upper, int mode);
template <typename T>
void launch_karnoldi(hipStream_t, const Inst* const* insts, const KChunks& c, KOpts o);
template <typename T>
void launch_kbegin(hipStream_t, const Inst* const* insts, const KChunks& c, KOpts o);
template <typename T>
void launch_kycomb(hipStream_t, const Inst* const* insts, const KChunks& c);
template <typename T>
void launch_kcycle_end(hipStream_t, const Inst* const* insts, const KChunks& c, KOpts o);
template <typename T>
void launch_kfinish(hipStream_t, const Inst* const* insts, const KChunks& c);
// BiCGStab: start and the first direction, then per iteration it [apply
// mode 2], v = J p^ and s, [apply mode 3], the first half's test with
// t = J s^, the update of x and r, and the test with the next direction
template <typename T>
void launch_bcg_begin(hipStream_t, const Inst* const* insts, const KChunks& c, KOpts o);
template <typename T>
void launch_bcg_dir(hipStream_t, const Inst* const* insts, const KChunks& c);
template <typename T>
void launch_bcg_half(hipStream_t, const Inst* const* insts, const KChunks& c, int it);
template <typename T>
void launch_bcg_end(hipStream_t, const Inst* const* insts, const KChunks& c, KOpts o,
                    int it);
void launch_kgather(hipStream_t, const Inst* const* insts, int nslots, int* out);
int krylov_max_restart();

}  // namespace pfd
