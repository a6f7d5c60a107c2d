// Sparse tangent by colouring (the paper's Alg. 2): declarations shared by
// sparse.cpp and kernels_sparse.hip.
#pragma once

#include <vector>

#include "efem_internal.h"

namespace efem {

// The assembly by node rows: every (element, local node) pair is a visit of
// that node, and a node's row of 3x3 blocks is the sum over its visits.  A wave
// takes the rows [wstart[w], wstart[w + 1]) (nodes in block order, at most
// kRowNodes, at most kRowBlocks blocks in all) and keeps them in LDS.
constexpr int kRowBlocks = 256;   // at most 18 KB of LDS per wave
constexpr int kRowNodes = 8;      // eight lanes share a node's visits
struct RowVisits {
    int32_t n_waves = 0, max_blocks = 0;
    const int32_t *wstart = nullptr;  // [n_waves + 1]
    const int32_t *node = nullptr;    // [n_nodes] row -> node
    const int32_t *vptr = nullptr;    // [n_nodes + 1] row -> its visits
    const uint32_t *visit = nullptr;  // internal element << 3 | local node
    const uint8_t *pos = nullptr;     // [visits][4 or 8] block of the row that each of the element's nodes is
    const int32_t *conn = nullptr;    // [n_elems][nen] nodes in the internal element order
    const int64_t *bptr = nullptr;
    const int32_t *bcol = nullptr;
};

// Per-context state: the CSR pattern of K (node 1-ring in 3x3 blocks) and a
// distance-2 colouring of the DOFs.  The values come from the visits above; a
// mesh with a ring of more than 255 nodes (a visit's block positions are one
// byte each) takes the entries by colour instead, grouped by the colour of
// their column, the product of K with a colour's indicator vector giving every
// entry of that colour at once.
struct SparseState {
    int64_t n_rows = 0, nnz = 0;
    int32_t n_colours = 0, max_row = 0;
    double setup_seconds = 0.0;
    int64_t *row_ptr = nullptr;     // device [n_rows+1]
    int32_t *col = nullptr;         // device [nnz]
    // the same pattern by 3x3 blocks: node row i holds the blocks (i, j) of
    // the nodes j of its 1-ring, bcol[bptr[i] .. bptr[i+1]) (sorted); the
    // values of node row i start at 9 bptr[i]
    int64_t n_blocks = 0;
    int64_t *bptr = nullptr;        // device [n_nodes+1]
    int32_t *bcol = nullptr;        // device [n_blocks]
    int32_t *dof_colour = nullptr;  // device [n_rows]
    RowVisits rows;                 // n_waves = 0: assembly by colours
    std::vector<int64_t> cstart;    // host [n_colours+1]: ranges into ent / ent_row
    int64_t *ent = nullptr;         // device [nnz]: entry index, grouped by column colour
    int32_t *ent_row = nullptr;     // device [nnz]: row of that entry
    double *seed = nullptr, *y = nullptr;   // device [n_rows] scratch
    std::vector<void *> owned;
};

// values of K at the FP64 linearization record xrec, by node rows (kernels.hip)
hipError_t launch_assemble_rows(const Ctx &c, const RowVisits &rv, const double *xrec, double *values);
hipError_t launch_seed(hipStream_t s, int64_t n, const int32_t *dof_colour, int32_t colour, double *seed);
hipError_t launch_extract(hipStream_t s, int64_t count, const int64_t *ent, const int32_t *ent_row,
                          const double *y, double *values);
hipError_t launch_block_spmv(hipStream_t s, int64_t n_nodes, const int64_t *bptr, const int32_t *bcol,
                             const double *val, const double *x, double *y);

}  // namespace efem
