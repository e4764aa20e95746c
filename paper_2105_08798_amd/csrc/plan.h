// Host planning of the FBC library: plain C++ on geometry and integers only (no HIP types),
// so that the same code builds into the library and, with the address and
// undefined-behaviour sanitizers, into a CPU check program.
//  * distinct column offsets n_b - n_i and their dense lookup (Section 3.2: the Green
//    blocks depend on the offset only);
//  * the order in which offset-table products take columns;
//  * negligible-block windows of the reduced and offset-table products;
//  * cluster trees and the block partition of the H-matrix form (Appendix C).
#pragma once
#include <cstdint>
#include <vector>

// One cell's columns: lattice indices (n1, n2) per column, [n][2].
struct PlanGeom {
    int n_i, n_b;
    const int32_t* cols_i;
    const int32_t* cols_b;
};

// Distinct offsets (d1, d2) = col_b - col_i over every cell, numbered row-major over their
// bounding box [d1min, d1min + w1) x [d2min, d2min + w2); lut[(d1 - d1min) w2 + d2 - d2min]
// is the offset's number, -1 for none.
struct PlanOffsets {
    int d1min = 0, d2min = 0, w1 = 0, w2 = 0;
    std::vector<int32_t> lut, d1, d2;
};
PlanOffsets plan_offsets(const std::vector<PlanGeom>& cells);

// Key of a column, n1 w2 + n2 modulo 2^32 (columns may lie anywhere, their keys past 32 bits).  A pad
// column's key less that of (d1min, d2min) and of an interface column is the pair's index in lut,
// also modulo 2^32: exact for lookups of up to 2^32 entries.
inline uint32_t plan_key(int32_t n1, int32_t n2, int w2) {
    return (uint32_t)n1 * (uint32_t)w2 + (uint32_t)n2;
}

// Order in which the tiles and chunks of an offset-table product take a cell's columns (place ->
// column): by angle about the middle of the interface columns, then distance, where the columns
// come in no neighbourly order -- consecutive ones, on average, farther apart than 3/4 of their mean
// distance from the middle (columns in random order 1.27 of it, by distance 0.9, by lattice index
// 0.3 to 0.55, by angle 0.02) and than four times what they are by angle.  Empty otherwise, and for
// fewer than 65536 pairs of columns.
void plan_order(const PlanGeom& g, std::vector<int32_t>& ord_i, std::vector<int32_t>& ord_b);

// In-plane distance of column a from column b (a = 1, c = a / sqrt 2).
double plan_pair_rho(int32_t a1, int32_t a2, int32_t b1, int32_t b2);

// Negligible-block windows of one cell.  Row tiles of the product: table_form ? 32 pad
// columns : rows_tile rows (mp / tile rows of them); K chunks: table_form ? 8 interface
// columns : 64 of the kp padded reals.  At cell mode m (table mode m * mult, rho_cut
// indexed by table mode) a chunk is negligible for a tile when every (pad, interface)
// pair of the two lies farther than rho_cut; per (mode, tile) the window is the cyclic
// run [win_start, win_start + win_len) of chunks left after removing the longest cyclic
// run of negligible chunks.  mode_skips[m] = 1 when some real chunk of some non-empty
// tile lies outside its window.
struct PlanWindows {
    int n_tiles = 0, n_chunks = 0;
    std::vector<int32_t> win_start, win_len;   // [nm][n_tiles]
    std::vector<uint8_t> mode_skips;           // [nm]
};
// The same for row tiles and K chunks given by their column ranges [lo, hi) (a chunk with lo >= hi is padding).
struct PlanRange {
    int lo, hi;
};
void plan_windows_ranges(const PlanGeom& g, int nm, const std::vector<PlanRange>& tiles,
                         const std::vector<PlanRange>& chunks, int mult, const std::vector<double>& rho_cut,
                         PlanWindows& out);
void plan_windows(const PlanGeom& g, int nm, int mp, int kp, bool table_form, int rows_tile, int mult,
                  const std::vector<double>& rho_cut, PlanWindows& out);

// Boxes of column offsets of the reduced forms' gather jobs.  chunk [n_chunks][4]: smallest and
// largest n1 and largest n2 of the interface columns that a chunk of 32 complex columns (three per
// interface column) touches, one unused; box [n_tiles][4]: smallest n1, range of n1, smallest n2
// of the pad columns that a tile of `rows` rows touches, and the length of a box row (the largest
// range of d2 over the chunks, plus one); largest [n_tiles]: records of the tile's largest box
// (range of d1 plus one, times the row length).  Columns past the last count as the last.
struct PlanBoxes {
    std::vector<int32_t> chunk, box;
    std::vector<int64_t> largest;
};
void plan_boxes(const PlanGeom& g, int n_tiles, int rows, int n_chunks, PlanBoxes& out);

// Cluster tree node: columns in tree order and the bounding box in the integer coordinates
// X = n1, Y = n1 + 2 n2 (in-plane x = X / 2, y = Y / (2 sqrt 2)).
struct PlanNode {
    std::vector<int> idx;
    long long xlo, xhi, ylo, yhi, sx, sy;
    long long n, diam8;               // 8 diam^2 = 2 dX^2 + dY^2
    int child[2] = {-1, -1};
};
// Binary space partitioning of the columns idx: each cluster is cut along the longer side
// of its bounding box at the median (ties by column index) until it holds at most b_min
// columns.  Appends the nodes (root first, children after their parent) and returns the
// index of the subtree's root.
int plan_tree(std::vector<PlanNode>& nodes, const std::vector<int32_t>& cols, std::vector<int> idx, int b_min);
// min(diam t, diam s) <= gamma dist(t, s) on the bounding boxes, in exact integers.
bool plan_admissible(const PlanNode& t, const PlanNode& s, int gamma);

struct PlanBlock {
    int kind;      // 1 low rank, 0 dense
    int t, s;      // tree nodes
};
// Block partition of t x s: admissible blocks low rank, pairs of leaves dense, every other
// block subdivided (a leaf side kept whole).
void plan_partition(const std::vector<PlanNode>& tb, const std::vector<PlanNode>& ti, int t, int s, int gamma,
                    std::vector<PlanBlock>& out);
