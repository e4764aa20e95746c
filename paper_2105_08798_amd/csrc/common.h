// Shared definitions of the FBC library (host plan + device kernels), gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <cstdint>
#include <vector>

#include "../../include/fbc.h"

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));

// Split-FP16 form: power-of-two scale exponent of a line mode's blocks from the largest
// table magnitude of that mode (bit pattern of a non-negative double).  |G - row mean|
// <= 2 max, so 2^e |G - row mean| < 2^14, inside the FP16 range with headroom.
__host__ __device__ inline int split16_exp_a(unsigned long long maxbits) {
    const double m = __longlong_as_double((long long)maxbits);
    return m > 0.0 ? 12 - ilogb(m) : 0;
}
typedef unsigned short us8_t __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------------
// MFMA fragment orders.  A real matrix X[rows][K'] (or the GEMM B operand, indexed
// [col][K'] the same way) is stored as 16-row blocks; inside a block the 64 lanes of a
// wave hold one MFMA operand each, so a wave-wide 16-byte load is 1 KiB contiguous.
//   FP64 16x16x4 : lane l holds X[16 blk + l%16][4 t + l/16]; two k-steps per 16 B.
//   FP32 16x16x4 : same lane map; four k-steps per 16 B.
//   BF16 16x16x32: lane l holds X[16 blk + l%16][32 t + 8 (l/16) + j], j = 0..7;
//                  hi and lo halves of the split are stored as consecutive 1 KiB runs.
// Output of the 16x16 MFMAs: FP64 c[j] = C[4 j + l/16][l%16];
//                            FP32 c[j] = C[4 (l/16) + j][l%16].
// K' is padded to a multiple of 64 for every form (zeros).
// The B operand (the transformed forces, one column per RHS and real/imaginary part)
// keeps each column's four 16-byte units of a block together: lane l's unit sits at
// position bpos(l) = 4 (l % 16) + l / 16 of its 1 KiB block, so the forward transform,
// which produces one column at a time, writes 64-byte runs; a wave still reads the
// whole block (lane order permuted).
// ---------------------------------------------------------------------------------
__host__ __device__ inline int bpos(int lane) { return ((lane & 15) << 2) | (lane >> 4); }

// Round-to-nearest FP64 -> FP16 through FP32.  The result equals direct rounding (FP32
// carries more than twice FP16's precision plus two bits, so the double rounding is
// innocuous).  The empty asm keeps the compiler from merging the two hardware
// conversions into one FP64 -> FP16 conversion, which it expands into a long integer
// sequence.
__device__ inline _Float16 f64_to_f16(double x) {
    float f = (float)x;
    asm volatile("" : "+v"(f));
    return (_Float16)f;
}
__host__ __device__ inline int64_t frag_off_f32(int64_t r, int64_t k, int64_t kp) {
    int64_t blk = r >> 4, rr = r & 15;
    int64_t lane = ((k & 3) << 4) | rr;
    return (((blk * (kp >> 4) + (k >> 4)) * 64 + bpos((int)lane)) << 2) + ((k >> 2) & 3);
}
// element offset (in bf16 units) of the hi part; the lo part is at +512
__host__ __device__ inline int64_t frag_off_bf16(int64_t r, int64_t k, int64_t kp) {
    int64_t blk = r >> 4, rr = r & 15;
    int64_t kk = k & 31;
    int64_t lane = ((kk >> 3) << 4) | rr;
    return ((((blk * (kp >> 5) + (k >> 5)) * 2) * 64 + bpos((int)lane)) << 3) + (kk & 7);
}

// Symmetric 3x3 component index: xx yy zz xy xz yz
__host__ __device__ inline int sym_idx(int c, int d) {
    if (c == d) return c;
    int lo = c < d ? c : d, hi = c < d ? d : c;
    return (lo == 0) ? (hi == 1 ? 3 : 4) : 5;
}

// One work item of the per-mode complex product: JOB_ROWS rows (reduced forms) or TAB_COLS pad
// columns (offset forms) of one mode of one cell over one slice of K (the K split keeps enough work items to fill the chip
// evenly; the partial products of the slices are summed in fixed order by the inverse
// line transform).  Offsets are in elements of the respective arrays.
struct GemmJob {
    int64_t a_off;   // compact store or reduced table (reduced forms), table mode base (offset forms)
    int64_t b_off;   // B fragments of this mode
    int64_t c_off;   // output [ct][mp][nm][16] doubles: this mode's record, K slice
    int32_t mb;      // row blocks of the mode (mp / 16)
    int32_t kp;      // padded K' (row stride of the fragment arrays)
    int32_t rb0;     // first row block of this tile
    int32_t ct;      // column tiles (8 RHS each)
    int32_t cell;    // cell index
    // K' range [k0, k1) (reduced forms) or interface columns [k0, k1) (offset forms, multiples of 16); the
    // range is cyclic: indices at or beyond the padded K wrap to its start (windows around
    // the non-negligible blocks of a tile may straddle the end); k0 == k1: empty (zeros)
    int32_t k0, k1;
    int32_t ct_active;  // column tiles holding RHS of this cell; offset forms: end of the job's
    int32_t crs;        // output row stride (doubles): the modes of a row are adjacent
    int32_t prec;       // offset forms: 1 = this job on FP32 MFMA (options.table_fp32), 0 = FP64
    // reduced forms: 1 = blocks gathered from the reduced table (a_off: byte offset of its mode),
    // 0 = streamed from the compact store; the (mode, tile)'s window has win_len chunks of 64 k',
    // this job starts at chunk win_a of it, and FP32 sums end where vs equal slices of it do
    int32_t gather, win_len, win_a, vs;
    int32_t c0;         // first column tile of the job
};

// Work lists of a persistent product launch: one list consumed by every work group (the
// jobs longest first), or one list per XCD (nl = 8: work group b takes jobs from list
// b mod 8 -- the XCD it runs on under round-robin dispatch -- and, once that list is
// exhausted, from the others in turn).  ctr: device counters, [l] the next job of list
// l, [8] the work groups that have left; all zero between launches.
struct PqLists {
    int* ctr;
    int nl;
    int start[9];      // list l holds the jobs [start[l], start[l + 1])
};

// Physical index of a step of a cyclic K range (idx < 2 n).
__host__ __device__ inline int wrap_k(int idx, int n) { return idx >= n ? idx - n : idx; }

// B fragments of the offset-table products, in the K order of their kernel (chunks of 16
// interface columns; column 16 chunk + 4 q + g in lane group g): per column tile and chunk
// 12 steps (q, d) of 64 units (Re- and Im-part operand), column n's four units of a step
// adjacent as in the reduced forms (bpos).  Element offset of the pair for B column n and
// complex column k = 3 i + d; nch chunks.
__host__ __device__ inline int64_t tab_frag_off(int n, int k, int nch) {
    const int i = k / 3, d = k - 3 * i;
    const int64_t step = ((int64_t)(n >> 4) * nch + (i >> 4)) * 12 + 3 * ((i >> 2) & 3) + d;
    return (step * 64 + (((n & 15) << 2) | (i & 3))) << 1;
}

// Read-only data that a whole wave reads at one address: through the constant address space the
// loads are scalar whatever the kernel stores.
typedef const __attribute__((address_space(4))) int uniform_int;
template <typename T>
__device__ inline T uniform_at(const T* p) {
    T v;
    const uniform_int* src = (const uniform_int*)p;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) ((int*)&v)[k] = src[k];
    return v;
}

// Per-cell device view used by the offset-table product kernel: the column keys (plan_key;
// their differences index the offset lookup), pad columns up to whole tiles of 16 (the last
// column repeated), interface columns up to whole chunks of 16 in the order [chunk][g][q].
struct CellDev {
    int64_t key_b, key_i;    // offsets into TabView::keys
    int64_t order_b;         // pad column of each place in the tiles (the same keys), -1: as they come
    // reduced forms, offsets into RTabView::keys: interface columns (n1, n2) in natural order, the last
    // one repeated past the end; per chunk of 64 k' the smallest and largest n1 and the largest n2 of
    // its columns (four ints); per JOB_ROWS rows the smallest n1, the range of n1, the smallest n2
    // and the row length of their pad columns' boxes (four ints); and these rows by component,
    // then (n1, n2): row - first row | place of the pad column in the box << 16
    int64_t rkey_i, rchunk, rbox, rrow;
};

// Rows of a job of the reduced forms, and the largest box of a chunk (records) that a job gathers.
#define JOB_ROWS 128
#define G_CAP 384

// The reduced forms' table of distinct column offsets: records of 64 bytes (16 of padding) in the
// order xx xy xz yz yy zz, each component eight bytes -- split forms: (re, im) hi halves, (re, im) lo
// halves; FP32: re, im.  Record of offset (d1, d2): (2 W d1 + (d1 + 2 d2) - base) >> 1, so
// consecutive d2 are consecutive records and the offsets' disc fills most of the array.
struct RTabView {
    const char* tab;
    const int32_t* keys;
    int w2, base, nrec;            // 2 W, and the number of records
};
struct RBox {
    int64_t w, base, mode_bytes;   // half range of n1 + 2 n2, smallest index, bytes per table mode
};

// The table of an offset-table product: `tab` starts at element a_base of the whole table
// (generated tables hold a few modes at a time); need (or NULL): offsets present per table
// mode, every other one reads as the record zero_rec of `tab`.
struct TabView {
    const double2* tab;
    int64_t a_base;
    const int32_t* lut;      // offset number by key difference
    const int32_t* keys;     // column keys of every cell (CellDev)
    const int32_t* need;
    int64_t n_off, zero_rec;
};

// Device-side status latch bits
enum { ST_NETFORCE = 1, ST_NONFINITE = 2 };

struct CellPlan {
    int nz, nm, n_i, n_b, R;
    int K, M;            // complex K = 3 n_i, rows M = 3 n_b
    int kp;              // padded real K' = roundup(6 n_i, 64)
    int mp;              // padded rows = roundup(3 n_b, 64 * RB), a whole work-group tile
    int ct;              // column tiles of the B / output layouts (same for every cell)
    int ctr;             // column tiles holding RHS of this cell = ceil(R / 8)
    int64_t f_off, u_off;        // offsets (doubles) into caller's f and u
    int64_t a_off;               // compact store offset (elements of the store type) of mode 0
    int64_t b_off;               // B fragments offset (elements) of mode 0
    int64_t c_off;               // GEMM output offset (doubles) of mode 0, K slice 0
    int64_t c_split;             // doubles per K slice of the GEMM output (nm*ct*mp*16)
    int64_t w_off;               // w scratch offset (doubles)
    int64_t t_off;               // f transpose scratch offset (doubles)
    int64_t red_off;             // reduction scratch offset (doubles)
    int rhs0;                    // first global RHS index
    int tw_n;                    // line length of the twiddle table used (== nz)
    int64_t tw_off;              // twiddle table offset (double2) for nz
    int32_t *cols_i_d, *cols_b_d;
    std::vector<int32_t> cols_i, cols_b;
    // Negligible-block windows: per (mode, row tile) the cyclic range of K chunks that
    // holds every block above the skip tolerance [win_start, win_start + win_len).
    int n_tiles = 0, n_chunks = 0;
    std::vector<int32_t> win_start, win_len;   // [nm][n_tiles]
    std::vector<uint8_t> mode_skips;           // [nm]: some chunk of this mode is skipped
    // offset-table forms: column at each place of the tiles and chunks (plan_order; empty: as they
    // come), and on the device the place of each interface column (NULL: as they come)
    std::vector<int32_t> ord_b, ord_i;
    const int32_t* place_i = nullptr;
    std::vector<uint8_t> gather;               // [nm][n_tiles]: reduced forms: blocks from the reduced table (RTabView)
    // Compact dense store of the tiles that are not gathered: region r = m n_tiles + tl holds the
    // win_len[r] chunk-tiles of that window from chunk-tile reg_pre[r] on (cell-local); n_ct =
    // reg_pre[nm n_tiles].
    std::vector<int64_t> reg_pre;
    int64_t n_ct = 0;
};
