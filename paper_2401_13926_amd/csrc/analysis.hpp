// Host-side analysis for the KKT refactorization solver: ordering, pivoted LU of the first
// system, and every schedule / layout the GPU kernels consume.  Pure C++, no HIP calls.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace kkt {

enum { ORDER_MD = 0, ORDER_ND = 1 };

// Refactorization hand-out: columns of at most kLaneLen entries run one per lane of a
// wavefront (64 x kLaneLen entries fill its LDS stage of 1,024); longer columns of a wide
// level are handed out kLaneChunk at a time.
constexpr int kLaneLen = 16;
constexpr int kLaneChunk = 8;

struct AnalysisOptions {
    int ordering = ORDER_MD;     // exact minimum degree, or BFS nested dissection
    const int32_t *fixed_order = nullptr;  // when set: this column order (n entries) is used
    int64_t nd_leaf = 64;
    double pivot_tau = 1e-10;
    int tile_threads = 256;      // threads of a triangular-solve block
    int tile_rows = 2048;        // rows of a tile at most
    int64_t tile_lds = 32768;    // LDS bytes of a staged tile at most (tile_lds_bytes)
    // LDS that tiles keep free for dense blocks (0: no dense segments), per triangle.  The top
    // of L's DAG is many levels of few long rows, where fusing pays; measured on the 60k
    // sequence, fusing in U (shorter rows, wider levels) cost more than it saved.
    int64_t dense_reserve_l = 16384;
    int64_t dense_reserve_u = 0;
    int narrow_columns = 1024;   // refactorization levels with at most this many columns are
                                 // handed out one column at a time
    int64_t ref_lds = 0;         // LDS bytes of a refactorization tile (0: no tiles)
    int64_t sol_lds = 20480;     // LDS bytes a solve tile is formed for (with refactorization tiles)
    int64_t sol_dense_lds = 32768;  // LDS bytes of a solve tile with its dense range at most
    int64_t list_max = INT32_MAX;   // entries of a list of the refactorization tiles at most
};

// Flags in TriSchedule::seg_lg: the segment's rows fit one wavefront; the segment is a
// *dense* one (several consecutive levels, at most kDenseRows rows, whose references to each
// other are kept as a dense strictly lower triangle in solve order and resolved by a
// wavefront-level column sweep; the packed entries of its rows hold only the references to
// earlier segments and tiles).
constexpr int32_t kSegWave = 0x40;
constexpr int32_t kSegDense = 0x80;
constexpr int kDenseRows = 64;
// A solve window whose first level has at most this many rows keeps part of its tile budget
// for dense blocks (the narrow top of the DAG); wider windows use the whole budget.
constexpr int kDenseWindowRows = 2048;

// Schedule of one triangular solve.  A tile is a contiguous run of rows solved by one block;
// it is cut into segments, each a set of mutually independent rows covered by one pass of the
// block (2^lg lanes per row), with a block barrier between segments.  Tiles are handed out in
// order; every reference of a row is to an earlier tile or an earlier segment of its own tile.
//
// Entries are stored "packed": the rows of the solve order one after the other, each row's
// entries in ascending column order.  A staged tile (tile_lds = 1) is copied into LDS when its
// block takes it: its entries, its rows' right-hand-side data, and the solution values of the
// rows it references in earlier tiles ("externals"); its references are then LDS slots
// (0..rows-1: the tile's own rows, rows + k: external k).  An unstaged tile (one row too long
// to stage) reads its entries from global memory and its references are source rows.
struct TriSchedule {
    std::vector<int32_t> rows;      // solve order
    std::vector<int32_t> tile_seg;  // first segment of each tile (tiles + 1)
    std::vector<int32_t> seg_row;   // start of each segment in rows (segments + 1)
    std::vector<int32_t> seg_lg;    // log2 of the lanes per row of each segment, | kSegWave when
                                    // the segment fits one wavefront (solved by wavefront 0)
    std::vector<int64_t> row_ent;   // first packed entry of each position of rows (n + 1)
    std::vector<int32_t> ent_ref;   // per packed entry: LDS slot (staged tile) or source row
    std::vector<int32_t> tile_ext;  // first external of each tile (tiles + 1)
    std::vector<int32_t> ext_src;   // source row of each external
    std::vector<uint8_t> tile_lds;  // 1: staged in LDS, 0: entries read from global memory
    std::vector<int64_t> csr2ent;   // CSR entry (row-wise layout of the triangle) -> index in the
                                    // triangle's values: [packed entries | dense blocks]
    std::vector<int64_t> tile_dense;  // first dense-block value of each tile (tiles + 1), index in
                                      // the triangle's values
    std::vector<int32_t> seg_dofs;  // dense segment: offset of its block within the tile's dense
                                    // values (column-major strictly lower triangle), else -1
    int64_t packed = 0;             // number of packed entries
    int64_t values() const { return tile_dense.empty() ? packed : tile_dense.back(); }
    int64_t levels = 0;             // depth of the dependency DAG
    int64_t windows = 0;            // groups of levels whose tiles are mutually independent
    int64_t tiles() const { return (int64_t)tile_seg.size() - 1; }
    int64_t segments() const { return (int64_t)seg_row.size() - 1; }
};

// LDS bytes a staged tile needs with FP64 values (the kernel's layout: solution slots, rhs,
// diagonal, entry values, dense-block values; row ids, column-permutation ids, row offsets;
// 16-bit references).
inline int64_t tile_lds_bytes(int64_t rows, int64_t ext, int64_t ent, int64_t dense = 0) {
    return 8 * (rows + ext) + 36 * rows + 10 * ent + 8 * dense + 32;
}
inline int64_t dense_block_values(int64_t m) { return m * (m - 1) / 2; }

// Schedule of the refactorization by tiles, for factors whose L and U patterns are each other's
// transposes (diagonal pivots on a symmetric pattern).  Node m is pivot step m with the entries
// it finishes: its diagonal, column m of L and row m of U.  Every update of an entry (i, j)
// with min(i, j) = m comes from a step k that has both i and j in its column, hence from a
// descendant of m in the elimination tree.  A tile is a set of whole subtrees of what earlier
// layers of tiles left over; it keeps all its entries in LDS, so that an update reads its two
// factors there: own entries, or externals (entries of earlier tiles' nodes, staged with the
// tile).  Tiles are handed out in layer order, so a tile only waits for earlier ones.
//
// Inside a tile, nodes are solved by level (segment) with a barrier in between.  Segment g
// first runs its items (an item applies consecutive updates of one entry, in ascending k, whose
// factors are all final by then), then guards its nodes' pivots and divides their L entries.
// Entry slots are ordered by segment: the nodes' L entries, their diagonals, their U entries.
constexpr int kRefDesc = 20;  // int32 per tile descriptor
struct RefTiles {
    // per tile: 0 first segment, 1 segments, 2 first entry, 3 entries, 4 first item, 5 items, 6 first
    // further update, 7 further updates, 8 first pivot reference, 9 pivot references, 10 first
    // export, 11 exports, 12 first external, 13 externals, 14 nodes, 15 first column-maximum
    // extra, 16 extras
    std::vector<int32_t> desc;
    // per segment, two words of cumulative counts within the tile: items | first slot << 16, nodes |
    // pivot references << 16 (each at the segment's end, the slot at its start)
    std::vector<uint32_t> seg;
    std::vector<int32_t> src;     // per entry slot: its value's entry in the copy of K, or -1 (fill)
    std::vector<uint16_t> col;    // per entry slot: tile-local node of its column, 0xFFFF if none
    // (slots in the next three are byte offsets, 8 x the slot: a tile has fewer than 8,192)
    // per item (and one past a tile's last) two words: slot | start of its further updates << 16;
    // its first update
    std::vector<uint32_t> item;
    std::vector<uint32_t> upd;    // per update after an item's first: slots of its L | U factor << 16
    std::vector<uint16_t> lq;     // pivot references, per L entry and diagonal in slot order: pivot slot
    std::vector<uint16_t> exp;    // per export: slot (entries whose other index is in a later tile)
    std::vector<int32_t> ext;     // per external: the export it is
    std::vector<uint32_t> cmx_node;  // column-maximum extras: entries of K in a node's column whose
    std::vector<int32_t> cmx_src;    // U entry belongs to an earlier tile (node; entry of K's copy)
    std::vector<int32_t> out_pos;   // per entry, by ascending position in the solve layout: that
    std::vector<uint16_t> out_slot;  // position and the entry's slot
    int64_t lds = 0;              // LDS bytes of the largest tile
    int64_t layers = 0;
    int64_t tiles() const { return (int64_t)desc.size() / kRefDesc; }
};
// LDS bytes of a refactorization tile: entry and external slots and pivot thresholds (8 bytes each
// for either precision); items, further updates; pivot references.
inline int64_t ref_lds_bytes(int64_t entries, int64_t ext, int64_t nodes, int64_t further, int64_t items, int64_t nq) {
    return 8 * (entries + ext + nodes) + 8 * (items + 1) + 4 * further + 2 * nq + 16;
}

// Schedule of both triangular solves by tiles, built together with RefTiles (the same factors
// qualify).  A tile is again a set of whole subtrees of what earlier layers left over, but
// formed for the solves' own footprint.  The L sweep takes the tiles in order, the U sweep in
// reverse; one launch runs both, each tile twice.
//
// Rows of a tile are ordered by segment (level inside the tile, of the sweep's own direction);
// the solution of tile t's row r (L order) is position base + r of the exchange vector of the L
// sweep, and likewise for U.  A segment's rows are cut into chunks of one wavefront pass: 2^lg
// lanes per row, every lane with the same even number of (value, reference) places, so a
// lane's places are at a fixed distance from each other and the chunk needs no row offsets;
// places without an entry hold the value 0 and refer to a zero slot.
//
// The narrow end of a tile (the last levels of the L sweep, the first of the U sweep) may form a
// dense range: at most 64 rows, several levels, whose references to each other go to a packed
// strictly lower triangle in LDS (column-major, in sweep order, zero where there is no entry) and
// are resolved by one wavefront's column sweep; the rows' other entries are places of chunks
// before it, which leave the right-hand side minus those terms.
constexpr int kSolDesc = 24;  // int32 per tile descriptor
constexpr int kSolSweep = 10;  // int32 of it per sweep
constexpr int kSolWaves = 4;   // wavefronts of a solve block (a segment's chunks go round robin)
struct SolveTiles {
    // per tile: 0 first position, 1 rows; for L at 2 and for U at 12: first chunk, chunks, first
    // place, places, first external, externals; dense range: first row, rows, entries (after the
    // tile's places, an even number), chunks before it
    std::vector<int32_t> desc;
    // per chunk two words: first row | rows << 13 | lg << 20 | places per lane / 2 << 23 (8 bits) |
    // barrier before the chunk << 31; first place (within the tile) | short << 28 | no division by the
    // pivot yet (dense range) << 29 | wavefront << 30.  short: the only chunk of its segment, after
    // another such one (no barrier, wavefront 0), with four places per lane
    std::vector<uint32_t> chunk_l, chunk_u;
    // per place: 8 x the slot it refers to (rows, externals, zero); per dense entry: its place in
    // the triangle
    std::vector<uint16_t> ref_l, ref_u;
    std::vector<int32_t> ext_l, ext_u;   // per external: exchange position; a tile's first is the
                                         // one expected to be written last
    std::vector<int32_t> node_l, node_u;  // pivot step of every position (L order, U order)
    std::vector<int32_t> pos_u;           // per U position: the L position of the same step
    int64_t lds = 0;                      // LDS bytes of the largest tile
    int64_t layers = 0;
    int64_t tiles() const { return (int64_t)desc.size() / kSolDesc; }
};
// LDS bytes of a solve tile: row, external and zero slots, U's reciprocal diagonals, places, the
// triangle of a dense range of m rows (and a place for the padding entry).
inline int64_t sol_lds_bytes(int64_t rows, int64_t ext, int64_t places, int64_t m) {
    return 8 * (rows + ext + 2) + 8 * (rows + 1) + 10 * places + (m > 0 ? 8 * (m * (m - 1) / 2 + 1) : 0) + 32;
}

// Everything derived from the pattern and the first system's values.
//
// Index spaces: "original" rows/columns are those of K; "steps" are pivot steps of the
// factorization P K Q = L U (row k of P K Q is original row prow[k], column k is q[k]).
struct Analysis {
    int64_t n = 0, nnz = 0;
    std::vector<int64_t> rowptr;  // K pattern (copy), CSR
    std::vector<int32_t> colidx;

    std::vector<int32_t> q, prow, pinv;
    int64_t offdiag_pivots = 0;

    // Factors in "exchange" layout (matches kkt_get_factor_pattern):
    //   L: strictly lower, per column original rows ascending; U: per column steps ascending,
    //   diagonal last.  Values of system 1 from the pivoted factorization.
    std::vector<int64_t> lp, up;
    std::vector<int32_t> li, ui;
    std::vector<double> lx, ux;

    // Combined factor F = L + U in step space, column-compressed, rows ascending:
    // column j = U part (rows < j), diagonal (row j), L part (rows > j).
    std::vector<int64_t> fp;      // n+1
    std::vector<int32_t> fi;      // f
    std::vector<int32_t> fdiag;   // per column: offset of the diagonal inside the column
    std::vector<int64_t> fsrc;    // per F entry: index into K's CSR values, or -1 (fill)
    std::vector<double> fx;       // system-1 values in F layout (host reference)

    // Update positions: for column j, for each U-part row k ascending, for each L-part
    // entry of column k in order: offset (inside column j) of that row.
    std::vector<int64_t> relptr;  // n+1
    std::vector<int32_t> relpos;  // sum of updates
    // The same updates as a flat list (the refactorization's paths when it exists): the F
    // index of the L entry each update applies, and the position in column j of its source's
    // U entry.  Empty when the factor has 2^31 entries or more.
    std::vector<int32_t> relsrc;
    std::vector<int32_t> relslot;

    // Refactorization schedule: columns sorted by (DAG level, index).
    std::vector<int32_t> col_order;
    std::vector<int32_t> col_level;  // DAG level of each col_order position (non-decreasing)
    int64_t levels_refactor = 0;
    // Hand-out items of the refactorization, in col_order (level) order: item t covers
    // positions [ref_item[t], ref_item[t + 1]).  In a wide level (more than narrow_columns
    // columns) a lane item holds up to 64 columns with at most kLaneLen entries each,
    // refactored one per lane, and the longer columns go kLaneChunk per item; in a narrow
    // level (the dependency chain at the top of the elimination tree) every column is an item
    // of its own, refactored by a whole wavefront.  Within a level, col_order puts the
    // lane-sized columns first.
    std::vector<int32_t> ref_item;
    std::vector<uint8_t> ref_item_lane;

    RefTiles ref;    // empty when the factor does not qualify (the items above are used then)
    SolveTiles sol;  // empty exactly when ref is (lsched and usched are used then)

    // Row-wise triangles in step space (strict L, strict U), from which the solve schedules
    // are built.  Solve layout T = [L values | strict U values | U diagonal (n, step order)],
    // each triangle's values being its schedule's [packed entries | dense blocks]; f2t maps
    // each F entry to its T index.
    std::vector<int64_t> lrp, urp;  // n+1 each
    std::vector<int32_t> lci, uci;  // column indices (steps), ascending per row
    std::vector<int32_t> f2t;
    int64_t t_size = 0;  // values in T (dense blocks include explicit zeros)

    // Triangular-solve schedules (L forward, U backward).
    TriSchedule lsched, usched;

    // Exchange layout -> F position (for copying device values back).
    std::vector<int64_t> l2f, u2f;

    // Order of the vectors inside a solve (the Krylov basis, residuals, iterates): position k
    // holds original index vperm[k], a reverse Cuthill-McKee order of K + K^T, so that the rows
    // one block of the matrix-vector products handles reference nearby entries.  The Krylov
    // kernels' copy of K is in that order: row k is original row vperm[k], its entries in their
    // original order with columns renumbered by vpinv (each row's terms are still summed in
    // ascending original column), ksrc the original CSR position of each entry.  fsrc_k is
    // fsrc in terms of that copy; prow_k, q_k are prow and q renumbered by vpinv.
    std::vector<int32_t> vperm, vpinv;
    std::vector<int64_t> krp;
    std::vector<int32_t> kci;
    std::vector<int64_t> ksrc, fsrc_k;
    std::vector<int32_t> prow_k, q_k;

    // Device layout with the flat list (phys): F's columns are stored in col_order, so the
    // columns of one hand-out item (the 64 of a lane item in particular) are side by side, and
    // the update lists follow the same order.  pc[p] / pu[p] (n + 1 each, ascending) are the
    // first F position / first update of the column at col_order position p, pnu[p] its
    // diagonal offset.  relpos, relsrc and relslot are then in that order, and relsrc, f2t,
    // fsrc_k, l2f and u2f hold these F positions.  Without the flat list F keeps the column
    // order of fp.
    bool phys = false;
    std::vector<int64_t> pc, pu;
    std::vector<int32_t> pnu;

    double seconds = 0.0;

    int64_t nnz_l() const { return (int64_t)li.size(); }
    int64_t nnz_u() const { return (int64_t)ui.size(); }
    int64_t nnz_f() const { return (int64_t)fi.size(); }
    int64_t updates() const { return (int64_t)relpos.size(); }
};

// Whether the one launch of both sweeps of the solve tiles could write an entry of x over an entry of b
// (n entries each, step k reading b[prow[k]] and writing x[q[k]]) that is still to be read: a U
// tile writes its rows' entries of x as soon as the tiles above it are done, which may be before
// another tree's L tile has read its entries of b.  It cannot where the arrays do not overlap, nor
// where they are one array and every pivot is on the diagonal: a tile then writes only the
// entries that it has read itself, after its own L task.  Callers copy b first where it could.
// (One launch per sweep there needed a variant of the kernel: 33 KB more code, with which other
// kernels of a solve of 500,000 unknowns took 3 us longer in all.)
inline bool may_overwrite(const Analysis &a, const double *b, const double *x) {
    const uintptr_t b0 = (uintptr_t)b, x0 = (uintptr_t)x, bytes = (uintptr_t)a.n * sizeof(double);
    if (b0 + bytes <= x0 || x0 + bytes <= b0) return false;
    return b0 != x0 || a.offdiag_pivots != 0;
}

enum AnalysisStatus { AN_OK = 0, AN_EINVAL = 1, AN_ENOMEM = 2, AN_ESINGULAR = 3 };

// Runs the whole analysis.  On failure returns the status and sets *msg.
int analyze(const AnalysisOptions &opt, int64_t n, const int64_t *rowptr, const int32_t *colidx,
            const double *values, Analysis &out, std::string *msg);

// Exposed for tests of the orderings alone.
void vector_order(int64_t n, const int64_t *rowptr, const int32_t *colidx, std::vector<int32_t> &perm);
int nested_dissection(int64_t n, const int64_t *rowptr, const int32_t *colidx, int64_t leaf,
                      std::vector<int32_t> &q);

}  // namespace kkt
