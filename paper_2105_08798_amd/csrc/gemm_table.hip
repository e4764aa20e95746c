// Per-mode products of the offset-table forms on MFMA (Section 3.2: the entries of G^(m)
// depend on the column offset n_b - n_i only).  No dense store: the blocks are gathered from
// the table of distinct column offsets, six symmetric complex components per record, straight
// into MFMA operand registers.
//
// The row and K orders of the product are free, and chosen so that a gathered record is an
// operand without any exchange between lanes:
//   rows: a row block holds one Cartesian component c of the tile's 16 pad columns, lane l
//         carrying pad column l % 16;
//   K:    a chunk is 16 interface columns, and lane group g = l / 16 carries the columns
//         4 q + g, q = 0..3, of it.
// So a lane gathers the records of its pad column and its four interface columns; component
// (c, d) of record q, real or imaginary part, is the lane's A operand of row block c in the
// K step (q, d, part), each component serving as (c, d) and (d, c).  The B fragments are
// written in the same K order by the forward line transform (tab_frag_off).  Nothing goes
// through LDS, there is no barrier, and every wave runs its own job: one 16-column tile over
// its own negligible-block window.
//
// What bounds it: FP64 MFMA.  A chunk is 72 MFMAs of 64 cycles per column tile, against 24
// 16-byte gathers per lane.  A record's registers are refilled for the next chunk as soon as
// its MFMAs are issued, the table offsets one chunk and the column keys two chunks ahead of
// that, so every load has a chunk's MFMAs to come back in.  Against blocks staged through LDS
// by work groups of two waves on 32 pad columns (a barrier per 8 interface columns, windows
// shared by the group), MI355X: eight uneven cells on one table (1..16 RHS each) 6.35 -> 3.95
// ms, the learned form's products at 256 layers, 1024 / 2048 columns, 16 RHS 1.98 -> 1.4 ms;
// 128 layers, 1024 / 2048 columns, 8 RHS: 0.92 ms = 56 TFLOP/s.
#include <algorithm>
#include <map>
#include <mutex>

#include "kernels.h"
#include "pq.h"

// One job of one wave over its CT column tiles.  DB: B fragments in flight, in (q, d) steps.
// F32: the gathered values and f^ rounded to FP32 on FP32 MFMA, summed in FP32 over 8 interface
// columns and in FP64 across them; their 48 k' run through the MFMAs four at a time in natural order
// (k' = 6 i + 2 d + part), lane group g the fourth's g-th, so values change lanes through LDS: the
// records [interface column][pad column][6][2], f^ [k'][RHS column].
constexpr int F32_REC = 8 * 16 * 12, F32_B = 48 * 16;       // floats; the latter per column tile
constexpr int f32_lds(int ct) { return 4 * (F32_REC + F32_B * ct); }
template <int CT, int DB, bool F32>
__device__ inline void tab_job(const GemmJob& jb, const TabView& tv, const double* __restrict__ B,
                               double* __restrict__ C, const CellDev* __restrict__ cells, float* lds) {
    static_assert(12 % DB == 0, "the B ring must divide the 12 steps of a chunk");
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const CellDev cd = cells[jb.cell];
    const int b0 = (jb.rb0 / 3) * 16;
    const int nch = jb.kp / 96;
    const int p0 = jb.k0 >> 4, n = (jb.k1 - jb.k0) >> 4;      // first chunk, chunks of the (cyclic) window
    d4_t acc[3][CT];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int x = 0; x < CT; ++x) acc[c][x] = (d4_t){0, 0, 0, 0};
    if (n > 0) {
        const double2* tm = tv.tab + (jb.a_off - tv.a_base);
        // generated tables hold only the first need[t] offsets of table mode t; the others are
        // zero by definition and read as the zero record behind the table
        const int o_lim = tv.need ? tv.need[jb.a_off / (6 * tv.n_off)] : 0x7fffffff;
        const int64_t o_zero = tv.zero_rec - (jb.a_off - tv.a_base) / 6;
        const uint32_t kb = tv.keys[cd.key_b + b0 + (lane & 15)];
        const uint32_t* keys = (const uint32_t*)tv.keys + cd.key_i + 4 * g;
        const double2* b = (const double2*)(B + jb.b_off) + (int64_t)jb.c0 * nch * 768 + bpos(lane);
        auto chunk_at = [&](int t) { return wrap_k(p0 + min(t, n - 1), nch); };
        double2 rec[4][6];
        auto load_rec = [&](int q, int o) {
            const int64_t at = o < o_lim ? (int64_t)o : o_zero;
            const double2* s = tm + at * 6;
#pragma unroll
            for (int e = 0; e < 6; ++e) rec[q][e] = s[e];
        };
        double2 bb[DB][CT];
        auto load_b = [&](int slot, int step, int ch) {       // step = 3 q + d of chunk ch
#pragma unroll
            for (int x = 0; x < CT; ++x)
                bb[slot][x] = b[((int64_t)x * nch + ch) * 768 + step * 64];
        };
        // table offsets of the chunk after the next refill's, and the keys of the one after that
        int cur = chunk_at(0), nxt = chunk_at(1), on[4];
        uint32_t key[4];
        {
            const int c2 = chunk_at(2);
            uint32_t k0[4], k1[4];
            int o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                k0[q] = keys[16 * cur + q];
                k1[q] = keys[16 * nxt + q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = tv.lut[kb - k0[q]];
            // the order of the main loop's refills, so that its first pass waits like the others
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 3 * q - (12 - DB); s < 3 * q + 3 - (12 - DB); ++s)
                    if (s >= 0) load_b(s, s, cur);
                load_rec(q, o[q]);
                on[q] = tv.lut[kb - k1[q]];
                key[q] = keys[16 * c2 + q];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int t = 0; t < n; ++t) {
            const int c3 = chunk_at(t + 3);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (F32) {
                    const int il = 4 * (q & 1) + g;
                    float4* ra = (float4*)(lds + (il * 16 + (lane & 15)) * 12);
#pragma unroll
                    for (int e = 0; e < 6; e += 2)
                        ra[e / 2] = make_float4((float)rec[q][e].x, (float)rec[q][e].y, (float)rec[q][e + 1].x,
                                                (float)rec[q][e + 1].y);
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const int step = 3 * q + d, slot = step % DB, sn = step + DB;
                        float* rb = lds + F32_REC + (6 * il + 2 * d) * 16 + (lane & 15);
#pragma unroll
                        for (int x = 0; x < CT; ++x) {
                            rb[x * F32_B] = (float)bb[slot][x].x;
                            rb[x * F32_B + 16] = (float)bb[slot][x].y;
                        }
                        load_b(slot, sn % 12, sn < 12 ? cur : nxt);
                    }
                    if (q & 1) {
                        __builtin_amdgcn_wave_barrier();        // (one wave: its LDS operations are in order)
                        f4_t a32[3][CT];
#pragma unroll
                        for (int c = 0; c < 3; ++c)
#pragma unroll
                            for (int x = 0; x < CT; ++x) a32[c][x] = (f4_t){0, 0, 0, 0};
#pragma unroll
                        for (int n4 = 0; n4 < 12; ++n4) {
                            const int kq = 4 * n4 + g, i = kq / 6, e = kq - 6 * i, d = e >> 1;
                            const float* fa = lds + (i * 16 + (lane & 15)) * 12 + (e & 1);
#pragma unroll
                            for (int c = 0; c < 3; ++c) {
                                const float av = fa[2 * sym_idx(c, d)];
#pragma unroll
                                for (int x = 0; x < CT; ++x)
                                    a32[c][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                        av, lds[F32_REC + x * F32_B + 64 * n4 + lane], a32[c][x], 0, 0, 0);
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int c = 0; c < 3; ++c)
#pragma unroll
                            for (int x = 0; x < CT; ++x)
#pragma unroll
                                for (int j = 0; j < 4; ++j) acc[c][x][j] += (double)a32[c][x][j];
                    }
                } else {
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const int step = 3 * q + d, slot = step % DB;
#pragma unroll
                        for (int part = 0; part < 2; ++part)
#pragma unroll
                            for (int x = 0; x < CT; ++x)
#pragma unroll
                                for (int c = 0; c < 3; ++c) {
                                    const double2 r = rec[q][sym_idx(c, d)];
                                    acc[c][x] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                        part ? r.y : r.x, part ? bb[slot][x].y : bb[slot][x].x, acc[c][x], 0, 0, 0);
                                }
                        const int sn = step + DB;
                        load_b(slot, sn % 12, sn < 12 ? cur : nxt);
                    }
                }
                load_rec(q, on[q]);
                on[q] = tv.lut[kb - key[q]];
                key[q] = keys[16 * c3 + q];
                // keeps the loads in ring order, so that a wait leaves the later ones in flight
                __builtin_amdgcn_sched_barrier(0);
            }
            cur = nxt;
            nxt = chunk_at(t + 2);
        }
    }
    const int64_t mp = (int64_t)jb.mb * 16;
    const int col = lane & 15;
    auto put = [&](auto place) {
#pragma unroll
        for (int x = 0; x < CT; ++x)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // output rows of the 16x16 MFMAs: FP64 4 j + lane / 16, FP32 4 (lane / 16) + j
                const int bl = place(b0 + (F32 ? 4 * g + j : 4 * j + g));
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    C[jb.c_off + ((int64_t)(jb.c0 + x) * mp + 3 * bl + c) * jb.crs + col] = acc[c][x][j];
            }
    };
    const int order_b = __builtin_amdgcn_readfirstlane((int)cd.order_b);
    if (order_b < 0) put([](int b) { return b; });
    else put([&](int b) { return tv.keys[order_b + b]; });
}

// A job runs the column tiles [c0, ct_active) of its cell, rounded up to a power of two; the
// context's count CT is the largest of its cells', so that a cell with few RHS beside one with many
// does not multiply zeros.  B fragments in flight: 12 steps of one column tile, 48 registers, for
// any count but 8 (64).
template <int CT, int MIX>
__device__ inline void tab_any(const GemmJob& jb, const TabView& tv, const double* __restrict__ B,
                               double* __restrict__ C, const CellDev* __restrict__ cells, float* lds) {
    if constexpr (CT > 1) {
        if (2 * (jb.ct_active - jb.c0) <= CT) {
            tab_any<CT / 2, MIX>(jb, tv, B, C, cells, lds);
            return;
        }
    }
    constexpr int DB = CT == 8 ? 2 : 12 / CT;
    if (MIX && jb.prec) tab_job<CT, DB, true>(jb, tv, B, C, cells, lds);
    else tab_job<CT, DB, false>(jb, tv, B, C, cells, lds);
}

// Each wave of a work group (one, or four: variant 1) on its own job; MIX: each job in its
// own precision (options.table_fp32).
template <int CT, int MIX>
__global__ void __launch_bounds__(256, CT <= 2 ? 2 : 1)
k_tab(const GemmJob* __restrict__ jobs, int njobs, TabView tv, const double* __restrict__ B, double* __restrict__ C,
      const CellDev* __restrict__ cells) {
    const int j = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    if (j >= njobs) return;
    const GemmJob jb = jobs[j];
    if (jb.mb == 0) return;
    extern __shared__ __attribute__((aligned(128))) float tab_lds[];
    tab_any<CT, MIX>(jb, tv, B, C, cells, tab_lds + (threadIdx.x >> 6) * (f32_lds(CT) / 4));
}

template <int CT, int MIX>
__global__ void __launch_bounds__(256, CT <= 2 ? 2 : 1)
k_tab_pq(const GemmJob* __restrict__ jobs, int njobs, PqLists q, TabView tv, const double* __restrict__ B,
         double* __restrict__ C, const CellDev* __restrict__ cells) {
    extern __shared__ __attribute__((aligned(128))) float tab_lds[];
    int cur = 0;
    for (int j = pq_next_wave(q, cur); j < njobs; j = pq_next_wave(q, cur)) {
        const GemmJob jb = jobs[j];
        tab_any<CT, MIX>(jb, tv, B, C, cells, tab_lds + (threadIdx.x >> 6) * (f32_lds(CT) / 4));
    }
    pq_done_wave(q);
}

void launch_gemm_dtab(hipStream_t st, const GemmJob* jobs, int njobs, int ct, const TabView& tv, const double* b,
                      double* c, const CellDev* cells, const PqLists* q, int mixed, int variant) {
    if (njobs <= 0) return;
    // one wave per work group: a finished job frees its place at once, where a group of four
    // waits for its longest (128 layers, 1024 / 2048 columns, 8 RHS: 0.89 against 0.92 ms; 32
    // layers, 301 / 613 columns, 3 RHS: 47 against 49 us)
    const int waves = variant == 1 ? 4 : 1, groups = (njobs + waves - 1) / waves;
#define TAB_CASE(CT, MIX)                                                                                     \
    do {                                                                                                      \
        if (q)                                                                                                \
            hipLaunchKernelGGL((k_tab_pq<CT, MIX>),                                                           \
                               dim3(std::min(groups, 4 / waves * pq_groups_of(k_tab_pq<CT, MIX>, 256))),      \
                               dim3(64 * waves), MIX * waves * f32_lds(CT), st, jobs, njobs, *q, tv, b, c, cells);                    \
        else                                                                                                  \
            hipLaunchKernelGGL((k_tab<CT, MIX>), dim3(groups), dim3(64 * waves), MIX * waves * f32_lds(CT), st, jobs,  \
                               njobs, tv, b, c, cells);                                                       \
    } while (0)
#define TAB_CT(CT) do { if (mixed) TAB_CASE(CT, 1); else TAB_CASE(CT, 0); } while (0)
    switch (ct) {
        case 1: TAB_CT(1); break;
        case 2: TAB_CT(2); break;
        case 4: TAB_CT(4); break;
        default: TAB_CT(8); break;
    }
#undef TAB_CT
#undef TAB_CASE
}
