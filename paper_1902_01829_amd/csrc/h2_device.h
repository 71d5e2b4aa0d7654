// Device-side data layout and kernel launchers of libh2mv (gfx950).
//
// Block layout ("16-byte column groups").  An R x C block of elements of size
// e bytes is stored as ceil(C / W) column groups of W = 16 / e columns; group
// g holds R items of 16 bytes, item r being the W entries (r, gW .. gW+W-1).
// Element (r, c) sits at ((c / W) * R + r) * W + c % W; columns past C are
// zero.  A wavefront streaming the block has lane r read item r of each group:
// consecutive lanes read consecutive 16-byte items, every load of a
// wavefront is one contiguous run of R * 16 bytes, and each lane accumulates
// the dot product of its own row -- no cross-lane reduction when R > 32.
// When R <= 32, 64 / R lane groups take interleaved column groups and are
// summed at the end.
#pragma once

#include <cstdint>
#include <hip/hip_runtime.h>

namespace h2 {

// One output segment of a block-row product: out[0..R) = init[0..R) + sum over
// the row's blocks of A_b * in_b.
struct RowDesc {
    int64_t out;    // element offset of the output segment
    int64_t init;   // element offset of the segment added to the result, or -1
    int32_t b0, b1; // blocks [b0, b1) of the block list
    int32_t R;      // rows of the segment (<= 64)
    int32_t sel;    // ROW_IN_X: input is the point vector; ROW_OUT_P: output is the point vector.
                    // Above the low 8 bits: in batches the member; in single-vector streaming lists the
                    // row's number of steps, the sum over its blocks of ceil(C / (G W)), G = 64 / R lane
                    // groups of W columns per item (0: not known)
};
enum { ROW_IN_X = 1, ROW_OUT_P = 2 };

struct BlkDesc {
    int64_t a;      // element offset of the block in the data array (16-byte aligned)
    int64_t in;     // element offset of the input segment
    int32_t C;      // columns of the block (<= 64)
    int32_t sidx;   // index of the block's scale (BF16 storage)
};

// Block to be generated by the fill kernel.
struct FillDesc {
    int64_t a;      // element offset of the block
    int32_t s, t;   // row / column node (tree node ids)
    int32_t sidx;   // scale index (BF16)
    int32_t kind;   // FILL_COUPLING or FILL_DENSE
};
enum { FILL_COUPLING = 0, FILL_DENSE = 1 };

// Geometry shared by the fill kernels.
struct Geometry {
    const double *pts;      // n x dim, tree order
    const double *lo, *hi;  // nnodes x dim boxes
    const int64_t *begin, *end;
    const double *cheb;     // cheb_p 1-D nodes
    int dim, cheb_p, rank;
    double corr_len;
};

// Storage element kinds.
enum ElemKind { ELEM_F64 = 0, ELEM_F32 = 1, ELEM_BF16 = 2 };
inline int elem_bytes(int kind) { return kind == ELEM_F64 ? 8 : kind == ELEM_F32 ? 4 : 2; }
inline int64_t block_elems(int R, int C, int kind) {
    const int W = 16 / elem_bytes(kind);
    return int64_t(R) * ((C + W - 1) / W) * W;
}

// Fills leaf bases (U as m_j x k, V^T as k x m_j) and transfers (E as k x k,
// F^T as k x k) in the basis element kind.  leaves: tree node of each leaf;
// offsets per leaf / per node (-1 for the root).
hipError_t launch_fill_bases(const Geometry &g, int basis_kind, void *basis,
                             const int64_t *leaf_node, const int64_t *off_U, const int64_t *off_VT,
                             int64_t nleaves, const int64_t *off_E, const int64_t *off_FT,
                             int64_t nnodes, hipStream_t st);

// Fills coupling / dense blocks in the block element kind (scales for BF16).
// Transposed copies of blocks in 16-byte column groups: dst (C x R) = src (R x C)^T,
// raw element copies (any element kind; BF16 scales are per block and unchanged).
struct TransDesc {
    int64_t src, dst;   // element offsets
    int32_t R, C;       // source block size
};
hipError_t launch_transpose_blocks(int kind, const void *src, void *dst, const TransDesc *desc, int64_t n,
                                   hipStream_t st);
hipError_t launch_fill_blocks(const Geometry &g, int block_kind, void *blocks, float *scales,
                              const FillDesc *desc, int64_t nblocks, hipStream_t st);

// Streaming launch over one work list.  kind: element kind of data; vec_f64:
// vector workspace (in0, out0) is double (else float); out1 is double with
// out1_f64 (a cut list writes FP64 partial sums), else of the workspace type.
struct RowLaunch {
    const RowDesc *rows;
    int64_t nrows;
    const BlkDesc *blks;
    const void *data;
    const float *scales;
    const void *in0;        // tree vectors
    const double *in1;      // point vector x
    void *out0;
    void *out1;
    int lds_bytes = 0;      // LDS requested beyond the kernel's own (caps workgroups per compute unit)
};
// Phases of the product (the tile launches have a kernel name each).
enum { PHASE_UP = 0, PHASE_STREAM = 1, PHASE_DOWN = 2, PHASE_LEAF = 3 };
hipError_t launch_stream(const RowLaunch &L, int kind, bool vec_f64, bool out1_f64, hipStream_t st);

// Levels `level` .. `level` + `depth` of a tree sweep in one launch, a
// workgroup of 2^(depth + split) wavefronts per node of `level`.
constexpr int SWEEP_MAX_DEPTH = 4;   // largest depth + split (1024 threads)
struct SumRange {
    int32_t c0, c1;   // chunks [c0, c1) of a cut stream list
};
struct SweepLaunch {
    const void *basis;
    const int64_t *off_leaf;         // V_j^T (up) or U_j (down; NULL: no basis) per leaf, element offsets
    const int64_t *off_tr;           // F_c^T (up) or E_c (down) per node
    const int64_t *leaf_begin, *leaf_end;
    const double *x;                 // up, leaf
    double *y;                       // down, leaf
    void *tree;                      // x^ (up) or y^ (down)
    const void *near;                // down, leaf: y_near
    const double *partials;          // down: chunk sums of a cut stream list, else NULL
    const SumRange *tree_sums, *near_sums;   // per node, per leaf
    int stride;                      // elements per node in tree
    int level, depth, split;
    bool leaf;                       // level + depth is the leaf level: leaf projection / leaf expansion too
    bool root_done;                  // down: the y^ of the nodes of `level` is complete
    int rank[SWEEP_MAX_DEPTH + 1];   // ranks of the levels
};
hipError_t launch_sweep(const SweepLaunch &L, bool up, bool vec_f64, hipStream_t st);

// Row sums of a list stored by halves: a segment's partial slots (64 values
// each), added in order to its output segment.
struct ReduceDesc {
    int64_t out;      // element offset of the output segment
    int32_t c0, c1;   // its slots
    int32_t R;        // rows of the segment
    int32_t point;    // 1: the near-field point vector (out1), 0: the tree vector (out0)
};
// partials: of the vectors' type.
hipError_t launch_reduce_chunks(const ReduceDesc *desc, int64_t n, const void *partials, void *out0, void *out1,
                                bool vec_f64, hipStream_t st);
// Stream phase of a matrix stored by halves (blocks with j >= i): rows write
// their direct sums to out0/out1 (the input segment of a row has its output
// segment's offset); slot[b] >= 0 names the 64-double partial slot that
// receives block b's transposed product S_b^T x_i, -1 for a diagonal block;
// partials are FP64 with FP64 vectors (vec_f64), FP32 otherwise.
// Stored by halves: a run of consecutive block rows [r0, r1) of the stream
// list taken by one wavefront, whose transposed products of one column
// segment are added in LDS; its merged slots are gslot[s0 .. s1).  Per block,
// slot >= 0 is the LDS slot of its column (< HALF_LDS_SLOTS), -1 a diagonal
// block, <= -2 a partial slot -(slot + 2) of its own.
struct HalfGroup {
    int32_t r0, r1;
    int32_t s0, s1;
};
constexpr int HALF_GROUP_ROWS = 4;
constexpr int HALF_LDS_SLOTS = 32;
// Workgroups of four wavefronts of the stream launch one compute unit holds.
hipError_t stream_half_workgroups_per_cu(int kind, bool vec_f64, int *n);
hipError_t launch_stream_half(const RowLaunch &L, const HalfGroup *groups, int64_t ngroups, const int32_t *slot,
                              const int32_t *gslot, void *partials, int kind, bool vec_f64, hipStream_t st);

// Plain streaming read of bytes (a multiple of 16) at buf by grid workgroups;
// one 8-byte value per workgroup to sink (the measured HBM read ceiling).
hipError_t launch_read_probe(const void *buf, int64_t bytes, int grid, void *sink, hipStream_t st);

// ---- many right-hand sides on MFMA (h2_mm.hip)
// Tiles of MM_TILE right-hand sides, FP32, [rhs][row] with the row count
// rounded up to 16 (zero-padded).  Tree tiles: node v at v * round16(k) *
// MM_TILE.  Point tiles: leaf j at j * slot.  Offsets in RowDesc / BlkDesc of
// the tile lists are tile offsets (elements); in the leaf phase RowDesc.out is
// the first row of the leaf in Y.
constexpr int MM_TILE = 32;
// Wavefront work items of a tile list: item = (row << 1) | half (the 32-row
// half of the row's output; rows of <= 32 rows have one item), -1 = none.
// The host lays them out in dispatch order: workgroup wg (4 items) runs on
// XCD wg % MM_XCDS, and each XCD's workgroups walk one contiguous range of the
// list holding about 1/MM_XCDS of its work.  Length: a multiple of 4 * MM_XCDS.
constexpr int MM_XCDS = 8;
// Pair items of a tile list (launch shapes that share tiles): two per
// workgroup, the two halves of a row of more than 32 rows, or two
// independent items of rows of at most 32 rows (-1 = none); laid out like
// the wavefront items (workgroup wg on XCD wg % MM_XCDS, contiguous ranges).
// Length: a multiple of 2 * MM_XCDS.
struct MmLaunch {
    const RowDesc *rows;
    const int32_t *items;
    int64_t nitems;
    const int32_t *pitems;
    int64_t npitems;
    const BlkDesc *blks;
    const void *data;        // FP32 or BF16 blocks
    const float *scales;
    const float *in_tree, *in_pts, *init;
    float *out_tree, *out_pts;
    double *Y;               // leaf phase: caller's column-major result
    int64_t ldy;
    int ncols;               // leaf phase: valid right-hand sides in this tile
};
// Launch configuration chosen by the autotuner: the block loop's prefetch
// depth (pipelined: 0 none, 1 the next block, 2 or 3 a ring of that many
// blocks refilled chunk by chunk; 4 or 5 a ring of 1 or 2 blocks with the two
// halves of a row sharing each input tile through LDS, 32-wide tiles only;
// 6 or 7 a ring of 6 or 8 column chunks, 16-wide tiles only), the number of workgroups of a grid-strided
// (persistent) launch (0 = one workgroup per 4 items; a multiple of MM_XCDS
// keeps every workgroup on its XCD's range),
// and the MFMA tile width: 16 (16x16 MFMAs, 16 right-hand sides per pass) or
// 32 (32x32 MFMAs); passes of more than 16 right-hand sides always use 32.
constexpr int MM_MAX_PIPE = 7;      // largest pipelined value
constexpr int MM_FIRST_PAIR = 4;    // 4 and 5 need 32-wide tiles
constexpr int MM_FIRST_CRING = 6;   // 6 and 7 (chunk rings) need 16-wide tiles
// whether a pipelined value runs with a tile width
inline bool mm_pipe_fits(int pipelined, int nt) {
    return pipelined < MM_FIRST_PAIR || (pipelined < MM_FIRST_CRING ? nt == 32 : nt == 16);
}
struct MmConfig {
    int pipelined;
    int64_t grid;
    int nt = 0;
};
// Right-hand sides per tile of a pass: the launches of one pass agree on it.
inline int mm_tile_width(const MmConfig &cfg, int ncols) { return cfg.nt == 32 || ncols > 16 ? 32 : 16; }
hipError_t launch_mm(const MmLaunch &L, int kind, int phase, const MmConfig &cfg, hipStream_t st);

// ---- many right-hand sides, FP64 matrices (h2_mm64.h)
// The same tile lists; tiles hold FP64 values, [row][rhs] with NR = 16 (at
// most 16 right-hand sides in the pass) or 32 per row, rows padded to 16.
struct Mm64Launch {
    const RowDesc *rows;
    const int32_t *items;
    int64_t nitems;
    const BlkDesc *blks;
    const double *data;
    const double *in_tree, *in_pts, *init;
    double *out_tree, *out_pts;
    double *Y;               // leaf phase: caller's column-major result
    int64_t ldy;
    int ncols;               // right-hand sides of the pass
    bool half;               // streaming list of a matrix stored by halves: every block of a row
                             // listed, BlkDesc.sidx = 1 where the stored block is its transpose
};
hipError_t launch_mm64(const Mm64Launch &L, int phase, hipStream_t st);
// Packs ncols right-hand sides of X (column-major, ldx) into FP64 point tiles.
hipError_t launch_pack64(const double *X, int64_t ldx, int ncols, const int64_t *leaf_begin, const int64_t *leaf_end,
                         int64_t nleaves, int64_t slot, double *tiles, hipStream_t st);

// ---- batches of H^2 matrices (many right-hand sides, one launch per level slot)
// Block offsets (BlkDesc.a) are absolute addresses; tile offsets index pool;
// the leaf phase writes member m's result at Ytab[m] with leading dimension
// ldytab[m] (m = RowDesc.sel >> 8).
struct MmBatchLaunch {
    const RowDesc *rows;
    const int32_t *items;
    int64_t nitems;
    const int32_t *pitems;
    int64_t npitems;
    const BlkDesc *blks;
    const float *scales;
    float *pool;
    double *const *Ytab;
    const int64_t *ldytab;
    int ncols;
};
hipError_t launch_mm_batch(const MmBatchLaunch &L, int kind, int phase, const MmConfig &cfg, hipStream_t st);
struct PackEntry {
    int64_t dst;   // pool offset of the leaf's point tile
    int64_t row;   // first row of the leaf in its member's X
    int32_t m;     // leaf size
    int32_t member;
};
hipError_t launch_batch_pack(const PackEntry *entries, int64_t count, double const *const *Xtab,
                             const int64_t *ldxtab, int nrhs, int tile_width, float *pool, int64_t grid, hipStream_t st);
// Packs right-hand sides j0 .. j0+MM_TILE-1 of X (column-major, ldx) into point tiles (16: j0+15).
hipError_t launch_pack(const double *X, int64_t ldx, int j0, int nrhs, const int64_t *leaf_begin,
                       const int64_t *leaf_end, int64_t nleaves, int64_t slot, float *tiles, int tile_width,
                       hipStream_t st);

// ---- basis orthogonalization and projection (FP64, symmetric)
// Doubles allocated after every T array handed to launch_project: the
// projection reads each node's T as a 64 x 64 frame (leading dimension kmax)
// and ignores what lies outside the node's k x k block.
constexpr int64_t PROJ_T_PAD = 64 * 64;
struct ProjDesc {
    int64_t off;        // element offset of the coupling block (input region)
    int64_t out;        // element offset of the projected block (output region)
    int64_t row, col;   // its row and column tree nodes
    int32_t k;          // its rank, >= 1 (the clamped loads of project_kernel rely on it)
    int32_t kout;       // rank of the projected block, 1 <= kout <= k
};
struct OrthLaunch {
    double *basis, *blocks, *T;   // T: nnodes x kmax x kmax scratch (column-major per node)
    double *T_col = nullptr;      // the column tree's, when it is not the row tree (V != U)
    const int64_t *off_U, *off_VT, *off_E, *off_FT;
    const int64_t *leaf_begin, *leaf_end;
    const ProjDesc *proj;
    int64_t nleaves, first_leaf, nproj;
    const int *level_rank;        // host, q + 1 values
    int q, lmin, kmax;
};
hipError_t launch_orthogonalize(const OrthLaunch &L, hipStream_t st);
// Every listed block: out(kout x kout) = T_row(0:kout, 0:k) in(k x k) T_col(0:kout, 0:k)^T,
// T and T_col kmax x kmax per node (column-major); in and out may be the same region.
// triangular: T and T_col are upper triangular (their zero K steps are skipped).
hipError_t launch_project(const double *in, double *out, const ProjDesc *desc, int64_t n, const double *T,
                          const double *T_col, int kmax, hipStream_t st, bool triangular);

// ---- algebraic compression (FP64, symmetric, orthonormal bases)
constexpr int COMP_XLD = 128;                    // leading dimension of a node's left singular vectors
constexpr int COMP_XSLOT = COMP_XLD * 64;        // doubles per node in CompLaunch::X
constexpr int COMP_USLOT = 64 * 64;              // doubles per leaf in CompLaunch::Unew (leading dimension 64)
struct CompLaunch {
    const double *basis, *blocks;        // orthonormal bases and coupling blocks (current layout)
    const int64_t *off_U, *off_E;        // per leaf / per node: the tree's leaf bases and transfers
    const int64_t *leaf_begin, *leaf_end;
    const ProjDesc *blk;                 // coupling blocks in BSR order, all levels (off, row, col, k used)
    const int64_t *row_start;            // per node: first entry of its block row in blk (nnodes + 1 values)
    const int64_t *col_blk;              // element offsets of the blocks S_ji of every block column, by column
    const int64_t *col_start;            // per node: first entry of its block column in col_blk (nnodes + 1)
    int use_rows;                        // 1: the basis generation stacks the block rows (transposed)
    int columns;                         // 1: the basis generation stacks the block columns
    int b_t, x_t;                        // 1: the tree's leaf bases / transfers are stored transposed
                                         //    (off_U, off_E then point at V_j^T, F_c^T: the column tree)
    double *R, *T, *Enew;                // per node, kmax x kmax, column-major
    double *X;                           // per node of the level being truncated: COMP_XSLOT doubles
    double *sigma;                       // per node of that level: 64 singular values, descending
    int32_t *count;                      // per node of that level: singular values kept
    double *Unew;                        // per leaf: COMP_USLOT doubles
    int64_t first_leaf, nleaves;
    int kmax;
};
// Tree R of the basis generation, nodes of `level` (k = its rank, kp = its
// parent level's; parent_term: the parent's R enters the stack).
hipError_t launch_basis_generation(const CompLaunch &L, int level, int k, int kp, bool parent_term, hipStream_t st);
// Leaves (rank k): singular values and left singular vectors of U_j R_j^T, kept counts for eps.
hipError_t launch_truncate_leaves(const CompLaunch &L, int k, double eps, hipStream_t st);
// Leaves: new bases (k~ columns) into Unew, T_j = first k~ left singular vectors, transposed.
hipError_t launch_truncate_leaves_apply(const CompLaunch &L, int k, int kt, hipStream_t st);
// Parents of the nodes of level l (children of rank kc truncated to kt, parents of rank kp):
// singular values and left singular vectors of Z_p R_p^T, kept counts for eps.
hipError_t launch_truncate_level(const CompLaunch &L, int l, int kc, int kt, int kp, double eps, hipStream_t st);
// Parents of level l: new transfers of their children into Enew, T_p = Q^T Z_p (ktp rows).
hipError_t launch_truncate_level_apply(const CompLaunch &L, int l, int kc, int kt, int kp, int ktp, hipStream_t st);
// Sets *flag to 1 if some pair (a, b) of k x k FP64 blocks has b != a^T.
struct MirrorDesc {
    int64_t a, b;   // element offsets
    int32_t k, pad;
};
hipError_t launch_symmetry_check(const double *blocks, const MirrorDesc *desc, int64_t n, int32_t *flag,
                                 hipStream_t st);
// Copies of column-major FP64 matrices into FP64 blocks in 16-byte column groups.
struct PlaceDesc {
    int64_t src, dst;     // element offsets
    int32_t R, C;         // destination block size
    int32_t ld;           // source leading dimension
    int32_t transpose;    // 1: the destination is the transpose of a C x R source
};
hipError_t launch_place(const double *src, double *dst, const PlaceDesc *desc, int64_t n, hipStream_t st);

}  // namespace h2
