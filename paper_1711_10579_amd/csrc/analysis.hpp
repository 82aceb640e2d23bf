// Host-side symbolic analysis of the Newton Jacobian (runs once per topology).
//
// The Jacobian of both formulations is a sparse matrix of 2x2 blocks over a
// node graph: buses for the single-phase polar form (unknowns angle and |V|,
// eq. 10) and phase-nodes for the three-phase current-injection form
// (unknowns Re V and Im V, eq. 19-22).  Its block pattern is the pattern of
// Ybus restricted to the nodes with unknowns, so the analysis works on that
// graph: fill-reducing ordering (Sec. III-A), symbolic block LU with a dense
// trailing block, column levels for the refactorisation and row levels for
// the two triangular solves, and the map from Ybus entries to LU storage.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace pfh {

struct Ordering {
  std::vector<int> perm;  // position -> node
  int n_sparse = 0;       // leading positions eliminated as sparse columns
};

Ordering min_degree_order(int n, const std::vector<std::vector<int>>& adj,
                          double dense_switch, int min_dense);

// Block ids of the sparse factor storage:
//   D_j          : id j                         (j < ns)
//   L(r_p, j)    : id ns + colptr[j] + p        (r_p = rowidx[colptr[j]+p] > j)
//   U(j, r_p)    : id ns + nnzl + colptr[j] + p
// Each block holds 4 values, row-major [a00 a01 a10 a11].
// The dense trailing block (positions ns..nu-1) is a column-major scalar
// matrix of order 2*nt with leading dimension ldt.
struct Analysis {
  int nu = 0, ns = 0, nt = 0;
  std::vector<int> node_of_pos;  // [nu]
  std::vector<int> pos_of_node;  // [n_nodes], -1 for fixed nodes
  std::vector<int> colptr;       // [ns+1]
  std::vector<int> rowidx;       // [nnzl]
  std::vector<int> parent;       // elimination tree over sparse columns (-1: root or tail)
  int64_t nnzl = 0;
  int ldt = 0;

  // refactorisation: columns grouped by level
  std::vector<int> col_lev_ptr;  // [nlev+1]
  std::vector<int> col_order;    // [ns]
  // per column target list: D, U(j, r_0..), L(r_0.., j) -> target id
  // tbase[j] = j + 2*colptr[j]; target t's updates are upd[uptr[t]..uptr[t+1])
  std::vector<int64_t> uptr;     // [ntargets+1]
  std::vector<int> upd_l, upd_u; // source block ids
  // Schur complement into the dense tail: tail block (a,b) -> list of
  // (L block, U block) pairs; only blocks with a non-empty list are listed
  std::vector<int> tail_tgt;     // a*nt + b
  std::vector<int64_t> tail_uptr;
  std::vector<int> tail_l, tail_u;

  // forward solve (L y = b) over sparse rows, by level: row i gathers
  // L(i,k) y_k for the listed (block id, k) pairs
  std::vector<int> fwd_lev_ptr, fwd_rows;
  std::vector<int> lrow_ptr, lrow_blk, lrow_col;  // [nu+1], by row position
  // backward solve (U x = y) over sparse rows, by level (tail first)
  std::vector<int> bwd_lev_ptr, bwd_rows;

  // statistics
  double flops_sparse = 0, flops_tail_schur = 0, flops_dense = 0;
  std::string summary() const;
};

// Lanes (a power of two) for lists of up to m entries.
inline int pick_lanes(int64_t m, int lane_scale) {
  int g = 1;
  while (g < 64 && 4LL * g < m) g *= 2;
  return g * lane_scale < 64 ? g * lane_scale : 64;
}
// Lanes per update list and forward row of each level.
std::vector<int> factor_lanes(const Analysis& an, int lane_scale);

// The sparse refactorisation of a case solved alone: levels below
// first_level take a launch each; the others run in one launch or two
// (stages, cutting the levels).  The subtrees of the elimination tree inside a
// stage need nothing from each other, so they are dealt out to bins, and a
// bin is a work-group that walks its levels with a barrier between them, its
// columns' lists in LDS.  Only who forms a column and when depends on this,
// not how (the lanes are the level's).
// A bin's program, in words from its start: number of records, number of
// slots; kTreeRec words per level with columns {first slot, slots, lanes per
// list, columns of the whole work-group}; a word per slot of a wave {first
// column entry, log2 of its lanes per column << 16, columns << 24} and, after
// a level's slots, per column of the whole work-group; per column {column,
// first block, blocks, target table}; per table the offsets of its 2 len + 2
// lists and the end; lists of pairs, (L, U) block ids or, the forward row
// (target len + 1), (L block, column).
constexpr int kTreeClasses = 6;     // columns of up to 8, 16, 32, 64, 128, 256 lanes; above: the whole work-group
constexpr int kTreeRec = 4, kTreeHead = 4;
constexpr int kTreeWords = 16000;   // a program's most words (of 64 KB of LDS)
constexpr int kTreeColumns = 20000; // levels of more columns always take a launch
struct TreePlan {
  struct Stage {
    int bin0, nbins, threads;
  };
  int first_level = 0;
  std::vector<Stage> stages;
  std::vector<int> bin_off;  // [bins + 1] first word of a bin's program (a multiple of 4)
  std::vector<int> prog;
  std::vector<int> bin_ptr, bin_cols;  // [bins + 1] the bins' columns
};
// max_bins work-groups of 256 threads, or half as many of 512; first_level
// -1: where the estimated time is least (possibly no level in trees).
TreePlan plan_trees(const Analysis& an, const std::vector<int>& lanes, int max_bins, int first_level = -1);

// The backward solve of the same subtrees, for a case solved alone: a
// work-group walks its bin's rows by backward level, the rows' values, the
// entries of the solution it reads from elsewhere and its own in LDS; the
// upper stage's bins first (the lower ones read their entries).  A bin's
// program, in words from its start: records, rows, list entries, entries
// read from elsewhere; four words per level with rows {first row, rows, log2
// of the lanes per row, 0}; four per row {row, first list entry, entries, 0};
// per list entry the place of its column's values (own rows first, then the
// ones from elsewhere); per list entry its U block; the columns read from
// elsewhere.
constexpr int kBwdBytes = 72 * 1024;  // LDS of a bin (two work-groups to a CU)
constexpr int kBwdRowBytes = 48;      // of a row's inverse and solution, FP64 (a block: 32, an entry read: 16)
struct BwdTrees {
  std::vector<int> off, prog;  // [bins + 1]; empty: no bins, every row by levels
  std::vector<char> in;        // [ns] the row is in a bin
};
BwdTrees plan_bwd_trees(const Analysis& an, const TreePlan& tp, const std::vector<int>& lanes);

struct GraphInput {
  int n_nodes = 0;
  std::vector<char> unknown;          // [n_nodes]
  std::vector<std::vector<int>> adj;  // node graph over all nodes
};

Analysis analyze(const GraphInput& g, double dense_switch, int min_dense, int tail_align);

// Destination of every Ybus entry (i, j) in the factor storage: the block id
// of D/L/U, or -2 - (a*nt + b) for block (a, b) of the dense tail, or -1 when
// i or j has no unknowns.  yrow[q] is the row of entry q.
void build_jmap(const Analysis& an, int n, const int* row_ptr, const int* col, std::vector<int>* yrow,
                std::vector<int>* jmap);

}  // namespace pfh

namespace pfh {

// Host analysis of the Newton-Krylov inner solve (Sec. III-B), once per
// topology.  The Krylov vectors hold the two unknowns of every node with
// unknowns, nodes in reverse Cuthill-McKee order of the node graph (row r).
// The Jacobian is kept as 2x2 blocks on that graph's pattern (block CSR,
// sorted columns); ILU(0) works on the same pattern.
struct KAnalysis {
  int nu = 0;
  std::vector<int> p_of_r, r_of_p;       // Krylov row <-> factor position of the node
  std::vector<int> row_ptr, col, diag;   // block CSR pattern in Krylov order
  // ILU(0) by targets: block t = (r, j) receives A(r, j) -= L(r, k) U(k, j)
  // for the listed pairs (q = position of (r, k), s = position of (k, j)),
  // k < min(r, j) ascending
  std::vector<int> up_ptr;               // [nnz+1]
  std::vector<int> up_q, up_s;
  // rows by level: a row's lower neighbours are in earlier levels (factor
  // and forward solve); its upper neighbours are in earlier levels of the
  // backward order
  std::vector<int> lev_ptr, lev_rows, ulev_ptr, ulev_rows;
  // block-Jacobi blocks: connected groups of at most bj_cap nodes grown
  // breadth-first from seeds in Krylov order; rows of each block in that
  // growth order, dense (2s)x(2s) inverse at bj_off[b]
  std::vector<int> bj_ptr, bj_rows, bj_loc;
  std::vector<int64_t> bj_off;
  int bj_max = 0;
  int64_t nnz() const { return (int64_t)col.size(); }
  int64_t nup() const { return (int64_t)up_q.size(); }
  int nblocks() const { return (int)bj_ptr.size() - 1; }
};

// The ILU(0) sweeps z = U^{-1} L^{-1} w with runs of levels merged into
// parts (a partitioned inverse): inside a part every row is written out in
// terms of the part's input and of rows of earlier parts, so the rows of a
// part need nothing from each other and one launch runs them all.
//   lower part: y_r = w_r + sum_e V(e) x(e)   (x = w inside the part, y before it)
//   upper part: z_r = sum_e V(e) x(e)         (x = y inside the part, z before it;
//                                              the row's own entry first)
// The entry values follow from the factor by levels inside each part, parts
// side by side ("steps"):
//   lower: V(e) = -sum over ops (q, s) of L(q) V(s)
//   upper: V(e) = -D_r^{-1} sum over ops (q, s) of U(q) V(s); no ops: D_r^{-1}
// with V(-1) the identity, q a block of the factor pattern and s an entry of
// a row of the same part.
struct KSweep {
  int nlp = 0, nup = 0;             // lower and upper parts
  std::vector<int> part_ptr;        // [nlp + nup + 1] positions
  std::vector<int> step;            // [2 nu] level of a position inside its part
  int nsteps = 0;
  std::vector<int> rows;            // [4 x 2 nu] per position {row, first entry, end, 0}; lower rows first
  std::vector<int> col;             // [ne] ~c: input at row c; c: row c of an earlier part
  std::vector<int> op_ptr;          // [ne + 1]
  std::vector<int> ops;             // [2 x nops] pairs (q, s)
  int64_t ne() const { return (int64_t)col.size(); }
  int64_t nops() const { return (int64_t)ops.size() / 2; }
};

// The reverse Cuthill-McKee order of an undirected graph (adjacency lists,
// no self loops): breadth-first from a pseudo-peripheral start in every
// connected component, neighbours taken by increasing degree, the whole
// sequence reversed.  Returns order[r] = vertex.
std::vector<int> rcm_order(const std::vector<std::vector<int>>& adj);

KAnalysis analyze_krylov(const Analysis& an, int n, const int* row_ptr, const int* col, int bj_cap);

// The factor's targets by level (a block (r, j) with updates is due in the
// level of row min(r, j), row r's diagonal block, listed as ~t, in its own):
// ptr [levels + 1] into tgt.  The blocks left of the diagonal hold A - sum
// L U, unscaled, until the factor's last pass multiplies them by D^{-1}.
void factor_targets(const KAnalysis& ka, std::vector<int>* ptr, std::vector<int>* tgt);

// Merge the sweep levels into parts whose rows have at most `cap` entries
// each (the rows of a level on its own may have more), the two triangles on
// up to `threads` threads; false, and the plan unusable, past max_entries.
bool build_sweep(const KAnalysis& ka, int cap, int64_t max_entries, KSweep* out, int threads = 1);
// The plan the solver uses, chosen from the case alone; `wide`: without a
// plan the sweeps take one launch per level.  False when no plan of at most
// max_entries entries beats the level sweeps.
bool plan_sweep(const KAnalysis& ka, bool wide, int64_t max_entries, KSweep* out, int threads = 1);

// Ybus entry -> block position in the Krylov pattern, -1 when the row or the
// column node has no unknowns.
void build_kmap(const Analysis& an, const KAnalysis& ka, int n, const int* row_ptr, const int* col,
                std::vector<int>* kmap);

}  // namespace pfh
