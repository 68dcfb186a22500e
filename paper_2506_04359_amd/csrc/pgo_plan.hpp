// Pose-graph optimisation (paper Sec. 2.3, Eq. 15): host plan of the sparse
// block Cholesky and the workspace carve.  Plain C++ (no HIP), so that it can
// be built and sanitised on the host alone.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace ba {

// Host plan of one pose graph over its free poses.  Columns of the block
// factor L are numbered in elimination order, grouped by level of the
// elimination tree (every column after its children); a column's blocks are
// its diagonal block followed by its off-diagonal blocks in increasing row.
struct PgoPlan {
  int n_poses = 0, n_edges = 0, n_free = 0, n_levels = 0;
  std::vector<int32_t> col_of_pose;   // n_poses: column of a free pose, -1 when fixed
  std::vector<int32_t> pose_of_col;   // n_free
  std::vector<int32_t> lev_ptr;       // n_levels + 1: columns of each level
  std::vector<int32_t> blk_ptr;       // n_free + 1: blocks of each column
  std::vector<int32_t> blk_row;       // n_blocks: row (column index) of each block
  std::vector<int32_t> upd_ptr;       // n_blocks + 1: updates L_rk L_ck^T into block (r, c)
  std::vector<int32_t> upd_a, upd_b;  //   block ids of L_rk and L_ck
  std::vector<int32_t> fwd_ptr;       // n_free + 1: forward updates y_c -= L_ck y_k
  std::vector<int32_t> fwd_blk, fwd_col;
  std::vector<int32_t> asm_ptr;       // n_blocks + 1: edge terms gathered into each block
  std::vector<int32_t> asm_edge;      //   edge * 2 + (1 when subtracted)
  std::vector<int32_t> rhs_ptr;       // n_free + 1: edge terms gathered into each RHS
  std::vector<int32_t> rhs_edge;      //   edge * 2 + (1 when subtracted)
  std::vector<int32_t> edge_i, edge_j;
  // the update and forward lists cut into chunks of kPgoChunk entries, each
  // summed by its own thread: chunks of block b are [chunk_ptr[b],
  // chunk_ptr[b+1]), chunk_blk the block of a chunk; the same for the forward
  // lists of the columns
  std::vector<int32_t> blk_col;       // n_blocks: column of each block
  std::vector<int32_t> chunk_ptr, chunk_blk, fchunk_ptr, fchunk_col;
  // per chunk its kPgoChunk block pairs (L_rk ids, then L_ck ids) and per
  // forward chunk its (block, column) pairs, -1 past the list's end: a
  // chunk's thread reads its whole list at once
  std::vector<int32_t> chunk_ab, fchunk_bc;
  // The factorisation's schedule.  A tier is a set of groups that do not depend on
  // each other: subtrees of the elimination tree (without the earlier tiers'
  // columns), each a workgroup's; the last tier is one group, the rest.  A group is a
  // run of steps, a step a set of columns of one level, small enough for the
  // workgroup's LDS.  tier_ptr: groups of each tier; grp_ptr: steps of each group.
  std::vector<int32_t> tier_ptr, grp_ptr;
  // Per step 8 ints: first chunk record and count, first forward record and count,
  // first block record and count, first column record and count.  A column too large
  // for a step has one of its own, with chunk count -1.
  std::vector<int32_t> steps;
  // Per column {column, first block, blocks, its first block in the step, first and
  // end forward chunk in the step, 0, 0}; per block {block, first and end chunk in
  // the step, row, -1 for the diagonal}; chunk_ab and fchunk_bc in step order.
  std::vector<int32_t> step_col, step_blk, step_ab, step_bc;
  int n_tiers() const { return (int)tier_ptr.size() - 1; }
  int n_blocks() const { return (int)blk_row.size(); }
};

constexpr int kPgoChunk = 4;
// Largest step: update chunks, forward chunks, blocks and columns (the LDS of k_pgo_tree).
constexpr int kStepChunks = 80, kStepFwd = 64, kStepBlks = 42, kStepCols = 42;

// Builds the plan; returns an error message (empty on success).
std::string build_pgo_plan(int32_t n_poses, int32_t n_edges, const int32_t* edge_i,
                           const int32_t* edge_j, const uint8_t* pose_fixed, PgoPlan& P);

// Workspace carved by the solve (FP64 unless noted).
struct PgoWork {
  double* edge[2];    // n_edges * 28: w B^T B (21, upper), w B^T r (6), w |r|^2
  double* cand;       // n_poses * 12 candidate poses
  double* L;          // n_blocks * 36 factor blocks (row-major)
  double* y;          // n_free * 6 right-hand side / forward solution
  double* x;          // n_free * 6 step
  double* part;       // n_chunks * 36 + n_fchunks * 6 partial sums of the update chunks
  double* state;      // 8: F, lambda, F0, ...
  int32_t* istate;    // 8: current edge buffer, candidate valid, accepted, chol failures, pivot failed, last accepted
};

size_t pgo_workspace_bytes(const PgoPlan& P);
PgoWork pgo_carve(const PgoPlan& P, void* ws);

}  // namespace ba
