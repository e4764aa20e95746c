// Per-mode complex products w^(m) = G^(m) f^(m) on MFMA (Section 2.3.2,
// eq. flexbc.up=Gpipl*fipl; Section 3.2, eq. impl.up=Gpipl*fipl_mvm, one dense product
// per line mode).  The complex product is one real product: A[row][k'] holds
// (Re, Im) of G^ interleaved along k', and the B operand holds, per RHS, the two
// columns (Re f, -Im f) and (Im f, Re f), so a 16-column output tile carries the real
// parts of 8 RHS in columns 0..7 and their imaginary parts in columns 8..15.
//
// Two kinds of jobs share a launch, 128 rows of one (cell, mode) each:
//  * stream: the tile's blocks are stored (compact store: the K chunks of its window, one
//    contiguous run in MFMA fragment order, each wave-wide 16-byte load 1 KiB contiguous) and
//    streamed once from HBM.  Modes whose rows carry a row gauge take it (the subtracted mean
//    makes an entry depend on the pad column, not on the offset alone), tiles whose boxes do
//    not fit, and every mode of FP32 contexts of eight column tiles.
//  * gather: every other mode reads the table of distinct column offsets in the form's
//    precision: the records of a K chunk's box of offsets are staged through LDS and read back as
//    fragments (gather_job).
// Both run the same MFMAs on the same operand values in the same order, FP32 sums over the
// same K chunks and FP64 across them, so a result does not depend on the kind of its job.
#include <cstdint>

#include "kernels.h"
#include "pq.h"

#include <algorithm>
#include <type_traits>

static __device__ inline void store_c_f32acc(double* __restrict__ c, const GemmJob& jb, int rb,
                                             int ctile, int lane, const d4_t& acc) {
    const int64_t mp = (int64_t)jb.mb * 16;
    const int col = lane & 15;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 16 * rb + 4 * (lane >> 4) + j;      // FP32-accumulator output order
        c[jb.c_off + ((int64_t)(jb.c0 + ctile) * mp + row) * jb.crs + col] = acc[j];
    }
}

// Loads of the stored G^ blocks: every byte is read once per update, so they go out as
// nontemporal (streaming) loads and do not push the f^ fragments, the partial outputs and
// the caller's arrays out of L2 and the Infinity Cache (measured on MI355X: the products
// run 8-11 % faster than with ordinary loads).
__device__ inline float4 ld_stream(const float4* p) {
    const f4_t v = __builtin_nontemporal_load((const f4_t*)p);
    return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline bf8_t ld_stream(const bf8_t* p) { return __builtin_nontemporal_load(p); }
__device__ inline h8_t ld_stream(const h8_t* p) { return __builtin_nontemporal_load(p); }

// Persistent work-queue form of the product kernels (pq.h): as many work groups as fit on
// the chip at once, each taking the next job of its list from a device counter until the
// lists are exhausted (with a list longest first, the groups that finish early take the
// short jobs: dynamic longest-processing-time scheduling of uneven jobs).  With one list
// per XCD (PqLists), the groups of an XCD work through consecutive row tiles of the same
// mode together, so the f^ fragments of their overlapping K windows are fetched into that
// XCD's L2 once; a group whose list is exhausted takes jobs from the other lists in turn.

// Where the FP32 sums go into the FP64 accumulators: after every KC chunks of 64 k', counted
// from the start of a slice, and at a slice's end.  The slices are those of the window cut
// into jb.vs parts (at least the job's own K slices): the sums then do not depend on how many
// of them one job runs through.
struct FlushAt {
    int w, seg0, seg1, v, wl, vs;
    __device__ explicit FlushAt(const GemmJob& jb) : w(jb.win_a), seg0(0), seg1(0), v(-1), wl(jb.win_len), vs(jb.vs) {
        while (seg1 <= w && v + 1 < vs) next();
    }
    __device__ void next() {
        ++v;
        seg0 = seg1;
        seg1 = (int)((unsigned)(wl * (v + 1)) / (unsigned)vs);
    }
    // one more chunk done: true when the sums are due
    template <int KC>
    __device__ bool step() {
        ++w;
        const bool due = ((w - seg0) & (KC - 1)) == 0 || w == seg1;
        while (w == seg1 && v + 1 < vs) next();
        return due;
    }
};

// ------------------------------- FP32 ---------------------------------------------
// FP32 MFMA with FP32 accumulation inside KC chunks of 64 real k, FP64 across chunks.
template <int TRB, int RB, int CT, int PF, int KC>
__device__ inline void gemm_f32_job(const GemmJob& jb,
                                                  const float* __restrict__ A,
                                                  const float* __restrict__ B,
                                                  double* __restrict__ C) {
    static_assert(4 % PF == 0, "ring depth must divide the 4 steps of a 64-k' chunk");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int rbw = jb.rb0 + wave * RB;
    if (rbw >= jb.mb) return;
    FlushAt fl(jb);
    const int kq = jb.kp >> 4;
    const int qb = jb.k0 >> 4, qe = jb.k1 >> 4;
    const float4* a = (const float4*)(A + jb.a_off) + (int64_t)(wave * RB) * 64 + lane;
    const float4* b = (const float4*)(B + jb.b_off) + (int64_t)jb.c0 * kq * 64 + bpos(lane);
    d4_t acc[RB][CT];
    f4_t ac32[RB][CT];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            acc[r][c] = (d4_t){0, 0, 0, 0};
            ac32[r][c] = (f4_t){0, 0, 0, 0};
        }
    if (qe <= qb) {              // empty K slice: its partial output is zero
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) store_c_f32acc(C, jb, rbw + r, c, lane, acc[r][c]);
        return;
    }
    float4 ab[PF][RB], bb[PF][CT];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        const int qw = wrap_k(qb + u, kq);
        const int qa = min(u, qe - qb - 1);       // A: step inside the job's stored run
#pragma unroll
        for (int r = 0; r < RB; ++r) ab[u][r] = ld_stream(a + (((int64_t)qa * TRB + r) * 64));
#pragma unroll
        for (int c = 0; c < CT; ++c) bb[u][c] = b[((int64_t)c * kq + qw) * 64];

        // keeps the ring's loads in slot order (slot 0 first), so the first wait of the main
        // loop leaves the later slots in flight instead of draining every load
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int q0 = qb; q0 < qe; q0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        const float av = h == 0 ? ab[u][r].x : h == 1 ? ab[u][r].y : h == 2 ? ab[u][r].z : ab[u][r].w;
                        const float bv = h == 0 ? bb[u][c].x : h == 1 ? bb[u][c].y : h == 2 ? bb[u][c].z : bb[u][c].w;
                        ac32[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, ac32[r][c], 0, 0, 0);
                    }
            const int ql = min(q0 + u + PF, qe - 1);
            const int qn = wrap_k(ql, kq);
#pragma unroll
            for (int r = 0; r < RB; ++r) ab[u][r] = ld_stream(a + (((int64_t)(ql - qb) * TRB + r) * 64));
#pragma unroll
            for (int c = 0; c < CT; ++c) bb[u][c] = b[((int64_t)c * kq + qn) * 64];

            __builtin_amdgcn_sched_barrier(0);     // the same order in every ring pass
        }
        const bool chunk_end = ((q0 - qb + PF) & 3) == 0;
        if (chunk_end && (fl.template step<KC>() || q0 + PF >= qe)) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[r][c][j] += (double)ac32[r][c][j];
                    ac32[r][c] = (f4_t){0, 0, 0, 0};
                }
        }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) store_c_f32acc(C, jb, rbw + r, c, lane, acc[r][c]);
}

// ------------------------------- split BF16 ---------------------------------------
// G ~ G_hi + G_lo, f ~ f_hi + f_lo; products lo*hi + hi*lo + hi*hi on BF16 MFMA with
// FP32 accumulation inside KC chunks of 64 real k, FP64 across chunks.
// The split-FP16 form runs the same kernel on FP16 MFMA; its operands carry power-of-two
// scales that the inverse transform removes.
__device__ inline f4_t mfma_16x16x32(bf8_t a, bf8_t b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ inline f4_t mfma_16x16x32(h8_t a, h8_t b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

template <typename VT, int TRB, int RB, int CT, int PF, int KC>
__device__ inline void gemm_split_job(const GemmJob& jb,
                                                    const unsigned short* __restrict__ A,
                                                    const unsigned short* __restrict__ B,
                                                    double* __restrict__ C) {
    static_assert(PF == 2, "a ring pass is the 2 steps of a 64-k' chunk");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int rbw = jb.rb0 + wave * RB;
    if (rbw >= jb.mb) return;
    FlushAt fl(jb);
    const int kt = jb.kp >> 5;
    const int tb = jb.k0 >> 5, te = jb.k1 >> 5;
    // 16-byte units: per (block, t): hi run of 64 units then lo run of 64 units
    const VT* a = (const VT*)(A + jb.a_off) + (int64_t)(wave * RB) * 128 + lane;
    const VT* b = (const VT*)(B + jb.b_off) + (int64_t)jb.c0 * kt * 128 + bpos(lane);
    d4_t acc[RB][CT];
    f4_t ac32[RB][CT];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            acc[r][c] = (d4_t){0, 0, 0, 0};
            ac32[r][c] = (f4_t){0, 0, 0, 0};
        }
    if (te <= tb) {              // empty K slice: its partial output is zero
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) store_c_f32acc(C, jb, rbw + r, c, lane, acc[r][c]);
        return;
    }
    VT ah[PF][RB], al[PF][RB], bh[PF][CT], bl[PF][CT];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        const int tw = wrap_k(tb + u, kt);
        const int ta = min(u, te - tb - 1);       // A: step inside the job's stored run
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            ah[u][r] = ld_stream(a + (((int64_t)ta * TRB + r) * 128));
            al[u][r] = ld_stream(a + (((int64_t)ta * TRB + r) * 128 + 64));
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            bh[u][c] = b[((int64_t)c * kt + tw) * 128];
            bl[u][c] = b[((int64_t)c * kt + tw) * 128 + 64];
        }
        // keeps the ring's loads in slot order (slot 0 first), so the first wait of the main
        // loop leaves the later slots in flight instead of draining every load
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int t0 = tb; t0 < te; t0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    ac32[r][c] = mfma_16x16x32(al[u][r], bh[u][c], ac32[r][c]);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    ac32[r][c] = mfma_16x16x32(ah[u][r], bl[u][c], ac32[r][c]);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    ac32[r][c] = mfma_16x16x32(ah[u][r], bh[u][c], ac32[r][c]);
            const int tl = min(t0 + u + PF, te - 1);
            const int tn = wrap_k(tl, kt);
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                ah[u][r] = ld_stream(a + (((int64_t)(tl - tb) * TRB + r) * 128));
                al[u][r] = ld_stream(a + (((int64_t)(tl - tb) * TRB + r) * 128 + 64));
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                bh[u][c] = b[((int64_t)c * kt + tn) * 128];
                bl[u][c] = b[((int64_t)c * kt + tn) * 128 + 64];
            }
            __builtin_amdgcn_sched_barrier(0);     // the same order in every ring pass
        }
        if (fl.template step<KC>() || t0 + PF >= te) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[r][c][j] += (double)ac32[r][c][j];
                    ac32[r][c] = (f4_t){0, 0, 0, 0};
                }
        }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) store_c_f32acc(C, jb, rbw + r, c, lane, acc[r][c]);
}

// Stream job of four column tiles (more than 16 RHS): the B fragments of a K step are the
// same for the NW waves of a work group, so they are loaded once per work group into LDS
// (double buffered) instead of once per wave from L2, and the group meets at one barrier
// per S steps.  A is streamed from HBM into a register ring PFA steps deep.  Each thread
// also keeps its share of B for the same PFA steps in a ring of its own: vector-memory
// loads complete in issue order, so the wait for B before it is copied into LDS would
// otherwise also wait for every A load issued before it, and cut the effective depth of
// the A ring down to the distance at which B was fetched.  K windows and slices hold an
// even number of steps, so S = 2 needs no tail.
template <typename VT, int RB, int CT, int PFA, int KC, int S, int NW>
__device__ inline void gemm_split_lds_job(const GemmJob& jb, const unsigned short* __restrict__ A,
                                          const unsigned short* __restrict__ B, double* __restrict__ C, char* smem) {
    static_assert(CT >= 2 && (CT % 2) == 0, "B staging assumes an even tile count");
    static_assert(S == 1 || S == 2, "one or two K steps per barrier");
    static_assert(PFA >= 2 * S && (PFA % (2 * S)) == 0, "ring depth must be a multiple of 2 S");
    constexpr int NTH = 64 * NW;             // threads of the work group
    constexpr int STEP_UNITS = CT * 128;     // 16-byte units of B per step (hi and lo runs)
    static_assert(STEP_UNITS % NTH == 0, "B units must spread evenly over the threads");
    constexpr int NU = STEP_UNITS / NTH;     // per thread and step
    VT* bs = (VT*)smem;                      // [2][STEP_UNITS * S]
    if (jb.rb0 >= jb.mb) return;             // whole work group (empty job)
    FlushAt fl(jb);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int rbw = jb.rb0 + wave * RB;
    const int kt = jb.kp >> 5;
    const int tb = jb.k0 >> 5, te = jb.k1 >> 5;    // te - tb is even (K slices of 64 k')
    constexpr int TRB = NW * RB;         // row blocks of the tile: the A step stride
    const VT* a = (const VT*)(A + jb.a_off) + (int64_t)(wave * RB) * 128 + lane;
    const VT* b = (const VT*)(B + jb.b_off) + (int64_t)jb.c0 * kt * 128;
    // (two jobs of an 8-tile row block read the same A: ordinary loads, the second finds it in a
    // cache)
    d4_t acc[RB][CT];
    f4_t ac32[RB][CT];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            acc[r][c] = (d4_t){0, 0, 0, 0};
            ac32[r][c] = (f4_t){0, 0, 0, 0};
        }
    if (te <= tb) {              // empty K slice: its partial output is zero
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) store_c_f32acc(C, jb, rbw + r, c, lane, acc[r][c]);
        return;
    }
    // this thread's share of B for step t: LDS in lane order, global in column-run order
    auto load_b = [&](VT (&dst)[NU], int t) {
        const int tw = wrap_k(t, kt);
#pragma unroll
        for (int j = 0; j < NU; ++j) {
            const int u = tid + NTH * j, c = u >> 7, rem = u & 127;
            dst[j] = b[((int64_t)c * kt + tw) * 128 + (rem & 64) + bpos(rem & 63)];
        }
    };
    auto store_b = [&](int buf, int sidx, const VT (&src)[NU]) {
#pragma unroll
        for (int j = 0; j < NU; ++j) bs[(buf * S + sidx) * STEP_UNITS + tid + NTH * j] = src[j];
    };
    // rings: PFA steps of A and of this thread's share of B in flight
    VT ah[PFA][RB], al[PFA][RB], br[PFA][NU];
#pragma unroll
    for (int u = 0; u < PFA; ++u) {
        const int tl = min(tb + u, te - 1);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            ah[u][r] = a[((int64_t)(tl - tb) * TRB + r) * 128];
            al[u][r] = a[((int64_t)(tl - tb) * TRB + r) * 128 + 64];
        }
        load_b(br[u], tl);
    }
#pragma unroll
    for (int u = 0; u < S; ++u) store_b(0, u, br[u]);
    __syncthreads();
    for (int t0 = tb; t0 < te; t0 += PFA) {
#pragma unroll
        for (int u = 0; u < PFA; ++u) {
            const int t = t0 + u;
            if (t >= te) break;                    // same for every wave of the group
            const int sidx = u % S;                // step inside the group of S
            const int buf = (u / S) & 1;           // groups of S alternate (PFA / S even)
            const VT* bb = bs + (buf * S + sidx) * STEP_UNITS;
            // two column tiles at a time, the three products of a tile interleaved with
            // the other tile's, so dependent MFMAs are 2 RB instructions apart
#pragma unroll
            for (int c = 0; c < CT; c += 2) {
                const VT bh0 = bb[c * 128 + lane], bl0 = bb[c * 128 + 64 + lane];
                const VT bh1 = bb[(c + 1) * 128 + lane], bl1 = bb[(c + 1) * 128 + 64 + lane];
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    ac32[r][c] = mfma_16x16x32(al[u][r], bh0, ac32[r][c]);
                    ac32[r][c + 1] = mfma_16x16x32(al[u][r], bh1, ac32[r][c + 1]);
                }
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    ac32[r][c] = mfma_16x16x32(ah[u][r], bl0, ac32[r][c]);
                    ac32[r][c + 1] = mfma_16x16x32(ah[u][r], bl1, ac32[r][c + 1]);
                }
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    ac32[r][c] = mfma_16x16x32(ah[u][r], bh0, ac32[r][c]);
                    ac32[r][c + 1] = mfma_16x16x32(ah[u][r], bh1, ac32[r][c + 1]);
                }
            }
            // slot u is free (its B went to LDS before this group): refill it PFA ahead
            const int tl = min(t + PFA, te - 1);
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                ah[u][r] = a[((int64_t)(tl - tb) * TRB + r) * 128];
                al[u][r] = a[((int64_t)(tl - tb) * TRB + r) * 128 + 64];
            }
            load_b(br[u], tl);
            if (((t - tb) & 1) && (fl.template step<KC>() || t + 1 == te)) {
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[r][c][j] += (double)ac32[r][c][j];
                        ac32[r][c] = (f4_t){0, 0, 0, 0};
                    }
            }
            if (sidx == S - 1) {
                if (t + 1 < te) {                  // next group of S steps, from the ring
#pragma unroll
                    for (int v = 1; v <= S; ++v) store_b(buf ^ 1, v - 1, br[(u + v) % PFA]);
                }
                __syncthreads();
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) store_c_f32acc(C, jb, rbw + r, c, lane, acc[r][c]);
}

typedef unsigned u4_t __attribute__((ext_vector_type(4)));
typedef unsigned u2_t __attribute__((ext_vector_type(2)));

// ------------------------------- gather jobs --------------------------------------
// The blocks come from the table of distinct column offsets.  A job's 128 rows belong to 43 or
// 44 pad columns, a chunk of 64 k' to 11 or 12 interface columns (the first and last maybe in
// part): some 500 pairs, but on neighbouring columns only about a hundred distinct offsets, all
// of them in a box of n1 x n2 of two hundred or so.  So the box, not the pairs, is read per
// chunk: while the group computes a chunk, its threads load the records of the next chunk's box
// into registers, then store them to LDS in six planes of eight bytes (xx xy xz yz yy zz); the
// chunk's B fragments and the places of its columns go the same way.  One buffer and several work groups per CU rather than two buffers: their load, store and
// compute phases overlap.
// A record has 64 bytes (16 of padding): the address unit takes a quad of lanes a clock where
// their 16-byte accesses fill one aligned 64-byte block, and one lane a clock otherwise.
// A fragments are read component by component, at the place of the pad column plus that of the
// interface column (n1 x n2 is linear in both).  The rows are taken in the order of their Cartesian
// component and, within one, so that the 16 of a fragment fall into distinct banks wherever the
// chunk's columns shift them (rows may be permuted freely, the K order may not).  The column and
// the component of k' depend on the lane only through its group g and the chunk number mod 3, so
// they come from three per-lane constants each.  Bound by LDS, the vector operations and MFMA about
// equally (1024 layers, 2048 / 4096 columns, 16 RHS, two column tiles, no row gauge so that every mode
// is gathered, 4.0 ms: busy 60, 50 and 32 %, 27 % of the LDS time bank conflicts; with 16-byte planes
// and rows by place the modes that are gathered with the gauge took 3.1 ms, 2.8 now).
// Bytes of a plane: 16 modulo 64, so that the three pairs of planes that a quad of lanes writes
// fall into distinct banks.
constexpr int G_PL = G_CAP * 8 + 16;
constexpr int G_COLS = (6 * G_PL + 127) / 128 * 128;      // places of the chunk's columns
constexpr int G_B = G_COLS + 128;                         // B fragments, 4 KiB per column tile
constexpr int gather_lds(int ct) { return G_B + 4096 * ct; }

// STG: records of a box that go through registers; of a larger box (up to G_CAP) the rest is
// copied while the chunk is stored.
template <typename VT, int CT, int RG, int KC, int STG>
__device__ inline void gather_job(const GemmJob& jb, const RTabView& tv, const void* __restrict__ Bv,
                                  double* __restrict__ C, const CellDev* __restrict__ cells, char* smem) {
    constexpr bool F32 = sizeof(VT) == 4;                         // VT = float: FP32, else the split halves
    constexpr int NTH = 64 * RG, RB = JOB_ROWS / 16 / RG;
    constexpr int NR = 4 * STG / NTH;
    static_assert(4 * STG % NTH == 0 && STG <= G_CAP, "whole rounds of units");
    constexpr int NBU = CT * 256 / NTH;                           // 16-byte B units per thread
    static_assert(CT * 256 % NTH == 0, "B units must spread evenly over the threads");
    if (jb.rb0 >= jb.mb) return;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4;
    const int nch = jb.kp >> 6, first = jb.k0 >> 6, n = (jb.k1 - jb.k0) >> 6;
    const CellDev cd = cells[jb.cell];
    const int row0 = 16 * jb.rb0, tile = row0 / JOB_ROWS;
    // the rows in the order used here: row - row0, place of the pad column in the box << 16
    const int32_t* rows = tv.keys + cd.rrow + tile * JOB_ROWS;
    d4_t acc[RB][CT];
    f4_t ac32[RB][CT];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            acc[r][c] = (d4_t){0, 0, 0, 0};
            ac32[r][c] = (f4_t){0, 0, 0, 0};
        }
    if (n > 0) {
        FlushAt fl(jb);
        // this lane's complex column is a + 4 g (split; a + g / 2 for FP32, whose steps hold two
        // columns), a the same for every lane, am = a mod 3: its interface column, and the LDS
        // address of its rows' component at the pad column's place
        const int gg = F32 ? g >> 1 : g;
        int base[RB][3], il4[3];
#pragma unroll
        for (int am = 0; am < 3; ++am) il4[am] = G_COLS + 4 * ((am + (F32 ? gg : 4 * gg)) / 3);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int e = rows[16 * (wave * RB + r) + (lane & 15)];
            const int c = (row0 + (e & 0xffff)) % 3;
#pragma unroll
            for (int am = 0; am < 3; ++am) {
                const int d = (am + gg) % 3, lo = min(c, d), hi = max(c, d);
                // slots: xx 0, xy 1, xz 2, yz 3, yy 4, zz 5
                const int slot = lo == 0 ? hi : lo == 1 ? (hi == 1 ? 4 : 3) : 5;
                base[r][am] = slot * G_PL + (e >> 16) * 8 + (F32 ? (g & 1) * 4 : 0);
            }
        }
        const uniform_int* box = (const uniform_int*)(tv.keys + cd.rbox + 4 * tile);
        const int tn1 = box[0], tspan = box[1], tn2 = box[2], L = box[3];   // smallest n1, range of n1, smallest n2
        const uniform_int* chunks = (const uniform_int*)(tv.keys + cd.rchunk);
        const int2* cols = (const int2*)(tv.keys + cd.rkey_i);
        // this thread's units: quarter of a record, and the record's number relative to the box's first
        const int part = tid & 3;
        auto relative = [&](int p) {
            const int r = p / L;
            return r * tv.w2 + r + 2 * (p - r * L);
        };
        int rel[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) rel[k] = relative((tid + NTH * k) >> 2);
        const int at = 2 * part * G_PL + (tid >> 2) * 8;
        const char* tm = tv.tab + jb.a_off;
        const u4_t* bsrc = (const u4_t*)Bv + (F32 ? jb.b_off >> 2 : jb.b_off >> 3);
        u4_t st[NR], sb[NBU];
        int2 xc = make_int2(0, 0);
        auto chunk_at = [&](int t) { return wrap_k(first + t, nch); };
        int cmin1, cmax1, cmax2, pmax1 = 0, pmax2 = 0;            // of the chunk to load, of the chunk loaded
        auto look = [&](int ch) {
            cmin1 = chunks[4 * ch];
            cmax1 = chunks[4 * ch + 1];
            cmax2 = chunks[4 * ch + 2];
        };
        int nu = 0, org = 0;                                      // units of the box loaded, its first record
        auto unit = [&](int rl) {                                 // (records of no offset are read too, inside the table)
            const int rec = max(0, min((rl + org) >> 1, tv.nrec - 1));
            return *(const u4_t*)(tm + (unsigned)(rec * 64 + part * 16));
        };
        auto load = [&](int ch) {
            nu = 4 * L * (tspan + cmax1 - cmin1 + 1);
            const int d1 = tn1 - cmax1, d2 = tn2 - cmax2;         // the box's first offset
            org = d1 * tv.w2 + d1 + 2 * d2 - tv.base;
#pragma unroll
            for (int k = 0; k < NR; ++k) st[k] = unit(rel[k]);
#pragma unroll
            for (int j = 0; j < NBU; ++j) {
                const int u = tid + NTH * j, c = u >> 8, e = u & 255;       // lane order from column-run order
                sb[j] = bsrc[(unsigned)((jb.c0 + c) * jb.kp * 4 + (e & ~63) + bpos(e & 63)) + (unsigned)(256 * ch)];
            }
            if (tid < 12) xc = cols[(32 * ch) / 3 + tid];
            pmax1 = cmax1;
            pmax2 = cmax2;
        };
        auto put = [](char* p, u4_t v) {
            *(u2_t*)p = v.xy;
            *(u2_t*)(p + G_PL) = v.zw;
        };
        auto store = [&]() {
            if (part < 3) {
#pragma unroll
                for (int k = 0; k < NR; ++k) put(smem + at + NTH * k * 2, st[k]);
                if constexpr (STG < G_CAP)
                    for (int u = NTH * NR + tid; u < nu; u += NTH)
                        put(smem + at + (u - tid) * 2, unit(relative(u >> 2)));
            }
#pragma unroll
            for (int j = 0; j < NBU; ++j) *(u4_t*)(smem + G_B + (tid + NTH * j) * 16) = sb[j];
            if (tid < 12) *(int*)(smem + G_COLS + 4 * tid) = 8 * (L * (pmax1 - xc.x) + pmax2 - xc.y);
        };
        auto compute = [&](auto phase) {
            constexpr int PH = decltype(phase)::value;
            const char* bl = smem + G_B + lane * 16;
            if constexpr (F32) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float4 bb[CT];
#pragma unroll
                    for (int c = 0; c < CT; ++c) bb[c] = *(const float4*)(bl + (c * 4 + q) * 1024);
                    float av[4][RB];
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        constexpr int A0 = 32 * PH;
                        const int a = A0 + 8 * q + 2 * h;
                        const int pl = *(const int*)(smem + il4[a % 3] + 4 * (a / 3 - A0 / 3));
#pragma unroll
                        for (int r = 0; r < RB; ++r) av[h][r] = *(const float*)(smem + base[r][a % 3] + pl);
                    }
#pragma unroll
                    for (int h = 0; h < 4; ++h)
#pragma unroll
                        for (int c = 0; c < CT; ++c) {
                            const float bv = h == 0 ? bb[c].x : h == 1 ? bb[c].y : h == 2 ? bb[c].z : bb[c].w;
#pragma unroll
                            for (int r = 0; r < RB; ++r)
                                ac32[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[h][r], bv, ac32[r][c], 0, 0, 0);
                        }
                }
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    VT ah[RB], al[RB];
                    int pl[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        constexpr int A0 = 32 * PH;
                        const int a = A0 + 16 * s + j;
                        pl[j] = *(const int*)(smem + il4[a % 3] + 4 * (a / 3 - A0 / 3));
                    }
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        u4_t h4, l4;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint2 v = *(const uint2*)(smem + base[r][(32 * PH + 16 * s + j) % 3] + pl[j]);
                            h4[j] = v.x;
                            l4[j] = v.y;
                        }
                        ah[r] = __builtin_bit_cast(VT, h4);
                        al[r] = __builtin_bit_cast(VT, l4);
                    }
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        const VT bh = *(const VT*)(bl + (c * 4 + 2 * s) * 1024);
                        const VT bo = *(const VT*)(bl + (c * 4 + 2 * s + 1) * 1024);
#pragma unroll
                        for (int r = 0; r < RB; ++r) ac32[r][c] = mfma_16x16x32(al[r], bh, ac32[r][c]);
#pragma unroll
                        for (int r = 0; r < RB; ++r) ac32[r][c] = mfma_16x16x32(ah[r], bo, ac32[r][c]);
#pragma unroll
                        for (int r = 0; r < RB; ++r) ac32[r][c] = mfma_16x16x32(ah[r], bh, ac32[r][c]);
                    }
                }
            }
        };
        int ch = chunk_at(0);
        look(ch);
        load(ch);
        look(chunk_at(min(1, n - 1)));
        store();
        __syncthreads();
        for (int t = 0; t < n; ++t) {
            const int nx = chunk_at(min(t + 1, n - 1));
            if (t + 1 < n) load(nx);
            const int ph = ch % 3;
            if (ph == 0) compute(std::integral_constant<int, 0>());
            else if (ph == 1) compute(std::integral_constant<int, 1>());
            else compute(std::integral_constant<int, 2>());
            if (fl.template step<KC>() || t + 1 == n) {
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[r][c][j] += (double)ac32[r][c][j];
                        ac32[r][c] = (f4_t){0, 0, 0, 0};
                    }
            }
            __syncthreads();                       // the chunk has been read
            if (t + 1 < n) {
                look(chunk_at(min(t + 2, n - 1)));
                store();
            }
            __syncthreads();
            ch = nx;
        }
    }
    const int64_t mp = (int64_t)jb.mb * 16;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t row = row0 + (rows[16 * (wave * RB + r) + 4 * g + j] & 0xffff);
#pragma unroll
            for (int c = 0; c < CT; ++c)
                C[jb.c_off + ((jb.c0 + c) * mp + row) * jb.crs + (lane & 15)] = acc[r][c][j];
        }
}

// ------------------------------- kernels ------------------------------------------
// Shape of a product class and variant: TRB row blocks per tile of the compact store, RG row
// groups (waves) on a job's 128 rows, CT column tiles, KC chunks of 64 k' per FP32 sum, OCC work groups per CU, STG staged records, and the stream jobs' ring (PF, or PFA
// and K steps per barrier S).
template <typename VT_, int TRB_, int CT_, int RG_, int KC_, int OCC_, int STG_, int PF_, int S_ = 0>
struct Shape {
    using VT = VT_;
    static constexpr int TRB = TRB_, CT = CT_, RG = RG_, KC = KC_, PF = PF_, S = S_, OCC = OCC_, STG = STG_;
    static constexpr int NTH = 64 * RG_, RB = JOB_ROWS / 16 / RG_;
    static constexpr int LDS = CT_ == 8 ? 0 : S_ == 0 ? gather_lds(CT_) : std::max(gather_lds(CT_), 2 * S_ * CT_ * 2048);
    static constexpr int WPE = std::max(1, OCC_ * RG_ / 4);      // waves per SIMD
};

// A job runs the column tiles that hold RHS of its cell, rounded up to a power of two (gather jobs
// also three; jobs of eight tiles, stream jobs all, hold seven or eight): a cell with few RHS beside one with many, or the second job of five tiles, does not
// multiply zeros.
template <typename SH, int CT = SH::CT>
__device__ inline void any_job(const GemmJob& jb, const void* __restrict__ A, const RTabView& tv,
                               const void* __restrict__ B, double* __restrict__ C,
                               const CellDev* __restrict__ cells, char* smem) {
    using VT = typename SH::VT;
    if constexpr (CT > 1 && CT < 8) {
        if (2 * (jb.ct_active - jb.c0) <= CT) {
            any_job<SH, CT / 2>(jb, A, tv, B, C, cells, smem);
            return;
        }
    }
    if (CT < 8 && jb.gather) {
        if constexpr (CT == 4) {
            if (jb.ct_active - jb.c0 == 3) {
                gather_job<VT, 3, SH::RG, SH::KC, SH::STG>(jb, tv, B, C, cells, smem);
                return;
            }
        }
        if constexpr (CT < 8) gather_job<VT, CT, SH::RG, SH::KC, SH::STG>(jb, tv, B, C, cells, smem);
    } else if constexpr (sizeof(VT) == 4) {
        gemm_f32_job<SH::TRB, SH::RB, CT, SH::PF, SH::KC>(jb, (const float*)A, (const float*)B, C);
    } else if constexpr (SH::S == 0 || CT == 1) {
        gemm_split_job<VT, SH::TRB, SH::RB, CT, 2, SH::KC>(
            jb, (const unsigned short*)A, (const unsigned short*)B, C);
    } else {
        gemm_split_lds_job<VT, SH::RB, CT, SH::PF, SH::KC, SH::S, SH::RG>(
            jb, (const unsigned short*)A, (const unsigned short*)B, C, smem);
    }
}

template <typename SH>
__global__ void __launch_bounds__(SH::NTH, SH::WPE) k_gemm(const GemmJob* __restrict__ jobs, const void* __restrict__ A,
                                                  RTabView tv, const void* __restrict__ B, double* __restrict__ C,
                                                  const CellDev* __restrict__ cells) {
    extern __shared__ __attribute__((aligned(128))) char gsm[];
    const GemmJob jb = uniform_at(jobs + blockIdx.x);
    any_job<SH>(jb, A, tv, B, C, cells, gsm);
}
template <typename SH>
__global__ void __launch_bounds__(SH::NTH, SH::WPE) k_gemm_pq(const GemmJob* __restrict__ jobs, int njobs, PqLists q,
                                                     const void* __restrict__ A, RTabView tv,
                                                     const void* __restrict__ B, double* __restrict__ C,
                                                     const CellDev* __restrict__ cells) {
    extern __shared__ __attribute__((aligned(128))) char gsm[];
    __shared__ int slot;
    int cur = 0;
    for (int j = pq_next(q, &slot, cur); j < njobs; j = pq_next(q, &slot, cur)) {
        const GemmJob jb = uniform_at(jobs + j);     // scalar loads, whatever the kernel stores
        any_job<SH>(jb, A, tv, B, C, cells, gsm);
    }
    pq_done(q);
}

// Rows of a tile (16 per row block): the planner pads rows to whole tiles, K' to a multiple of
// 64, takes the windows per tile and lays the compact store out in tiles of this height.  256
// rows at two column tiles, 128 at the others; a job is 128 rows of a tile (JOB_ROWS).
int gemm_tile_rows(int, int jt) { return jt == 2 ? 256 : 128; }

// Kernel variants of a product class (form, column tiles of a job) that the autotuner may choose
// from (jt: 1, 2, 4, or 8).  They share the tile height and the arithmetic order, so every variant
// gives bitwise the same result: variant 0 is the default; variant 1 changes the depth of the stream jobs'
// prefetch ring (FP32) or their K steps per barrier (split products with four column tiles; variant
// 2: half the ring besides).
int gemm_variants(int form, int jt) {
    if (form == FBC_FORM_SPLIT_FP16 || form == FBC_FORM_SPLIT_BF16) return jt <= 2 ? 1 : 3;
    return 2;
}

// Calls fn(Shape) for a product class and variant.  FP32 sums: 2 chunks of 64 k' for split FP16
// (its representation error is ~2^-23, so the FP32 sums must not dominate; 1 chunk at one or
// two column tiles), 4 for split BF16 and FP32.
template <typename F>
static void with_shape(int form, int jt, int variant, F&& fn) {
#define SPLIT_SHAPES(VT, KC12, KC48, OCC2, STG2)                                               \
    if (jt <= 1) fn(Shape<VT, 8, 1, 4, KC12, 4, G_CAP, 2>());                               \
    else if (jt <= 2) fn(Shape<VT, 16, 2, 4, KC12, OCC2, STG2, 2>());                       \
    else if (variant == 2) fn(Shape<VT, 8, 4, 4, KC48, 2, G_CAP, 2, 1>());                     \
    else if (variant == 1) fn(Shape<VT, 8, 4, 4, KC48, 2, G_CAP, 4, 1>());                     \
    else fn(Shape<VT, 8, 4, 4, KC48, 2, G_CAP, 4, 2>());
    if (form == FBC_FORM_FP32) {
        if (jt <= 1) {
            if (variant) fn(Shape<float, 8, 1, 4, 4, 4, G_CAP, 2>());
            else fn(Shape<float, 8, 1, 4, 4, 4, G_CAP, 4>());
        } else if (jt <= 2) {
            if (variant) fn(Shape<float, 16, 2, 4, 4, 3, G_CAP, 2>());
            else fn(Shape<float, 16, 2, 4, 4, 3, G_CAP, 4>());
        } else if (jt > 4) {
            if (variant) fn(Shape<float, 8, 8, 4, 4, 1, 0, 2>());
            else fn(Shape<float, 8, 8, 4, 4, 1, 0, 4>());
        } else {
            if (variant) fn(Shape<float, 8, 4, 4, 4, 2, G_CAP, 4>());
            else fn(Shape<float, 8, 4, 4, 4, 2, G_CAP, 2>());
        }
    } else if (form == FBC_FORM_SPLIT_FP16) {
        SPLIT_SHAPES(h8_t, 1, 2, 4, 256)
    } else {
        SPLIT_SHAPES(bf8_t, 4, 4, 3, G_CAP)
    }
#undef SPLIT_SHAPES
}

// Work groups of a product class that a CU holds.
int gemm_groups_per_cu(int form, int jt) {
    int n = 1;
    with_shape(form, jt, 0, [&](auto sh) { n = decltype(sh)::OCC; });
    return n;
}

// Readable shape of a variant.
std::string gemm_shape(int form, int jt, int variant) {
    char buf[96];
    with_shape(form, jt, variant, [&](auto sh) {
        using SH = decltype(sh);
        snprintf(buf, sizeof buf, "%s rows=%d CT=%d waves=%d KC=%d ring=%d S=%d, %s",
                 form == FBC_FORM_FP32 ? "f32" : form == FBC_FORM_SPLIT_FP16 ? "f16" : "bf16", JOB_ROWS, SH::CT,
                 SH::RG, SH::KC, SH::PF, SH::S, SH::CT == 8 ? "stream" : "gather + stream");
    });
    return buf;
}

// Raises the dynamic-LDS limit of the product kernels of a class on the current device (call
// outside stream capture, e.g. at context creation).
void gemm_kernels_init(int form, int jt) {
    for (int v = 0; v < gemm_variants(form, jt); ++v)
        with_shape(form, jt, v, [&](auto sh) {
            using SH = decltype(sh);
            (void)hipFuncSetAttribute((const void*)k_gemm<SH>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS);
            (void)hipFuncSetAttribute((const void*)k_gemm_pq<SH>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS);
        });
    (void)hipGetLastError();
}

void launch_gemm(hipStream_t st, int form, const GemmJob* jobs, int njobs, int jt, const void* a,
                 const RTabView& tv, const void* b, double* c, const CellDev* cells, const PqLists* q, int variant) {
    if (njobs <= 0) return;
    with_shape(form, jt, variant, [&](auto sh) {
        using SH = decltype(sh);
        if (q)
            hipLaunchKernelGGL(k_gemm_pq<SH>, dim3(std::min(njobs, SH::OCC * device_cus())),
                               dim3(SH::NTH), SH::LDS, st, jobs, njobs, *q, a, tv, b, c, cells);
        else
            hipLaunchKernelGGL(k_gemm<SH>, dim3(njobs), dim3(SH::NTH), SH::LDS, st, jobs, a, tv, b, c, cells);
    });
}
