// Learned far-field form (beyond the exact near field): the continuum Green function
// in the line-mode representation (Section 3.1, eq. cgf; Appendix B, lattice function ->
// continuum function beyond a cut-off radius), tabulated once through its homogeneity,
// and a 4-layer MLP for the correction G^_lgf - G^_cgf, with training kernels (forward,
// backward, Adam) and the on-the-fly table generator of the surrogate form.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "elastic.h"
#include "learned.h"

#define NTL 256

__device__ inline void kelvin(const double x[3], const CgfConst& k, const double* __restrict__ cpsi,
                              const double* __restrict__ spsi, double out[6]) {
    kelvin_point(x, k.c11, k.c12, k.c44, k.npsi, cpsi, spsi, out);
}

// G0 = G_K(t) and g1(phi_j) = (r_hat_j . grad) G_K at t (central difference, step h).
__global__ void k_cgf_g(CgfConst k, const double* __restrict__ cpsi, const double* __restrict__ spsi,
                        const double* __restrict__ rhat, double* __restrict__ g0,
                        double* __restrict__ g1) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j > k.nphi) return;
    if (j == k.nphi) {
        kelvin(k.t, k, cpsi, spsi, g0);
        return;
    }
    const double h = 1e-4;
    double xp[3], xm[3], gp[6], gm[6];
    for (int a = 0; a < 3; ++a) {
        xp[a] = k.t[a] + h * rhat[3 * j + a];
        xm[a] = k.t[a] - h * rhat[3 * j + a];
    }
    kelvin(xp, k, cpsi, spsi, gp);
    kelvin(xm, k, cpsi, spsi, gm);
    for (int c = 0; c < 6; ++c) g1[6 * j + c] = (gp[c] - gm[c]) / (2.0 * h);
}

// Remainder R(phi_j, z) = G_K(r_hat_j + z t) - G0/sqrt(z^2+1) - g1_j z/(z^2+1)^{3/2}.
__global__ void __launch_bounds__(NTL) k_cgf_rem(CgfConst k, const double* __restrict__ cpsi,
                                                 const double* __restrict__ spsi,
                                                 const double* __restrict__ rhat,
                                                 const double* __restrict__ g0,
                                                 const double* __restrict__ g1,
                                                 double* __restrict__ rem) {
    const int64_t idx = (int64_t)blockIdx.x * NTL + threadIdx.x;
    if (idx >= (int64_t)k.nphi * k.nzq) return;
    const int j = (int)(idx / k.nzq);
    const int q = (int)(idx - (int64_t)j * k.nzq);
    const double z = -k.zmax + q * k.dz;
    double x[3], g[6];
    for (int a = 0; a < 3; ++a) x[a] = rhat[3 * j + a] + z * k.t[a];
    kelvin(x, k, cpsi, spsi, g);
    const double d = sqrt(z * z + 1.0);
    const double e1 = 1.0 / d, e2 = z / (d * d * d);
    for (int c = 0; c < 6; ++c) rem[idx * 6 + c] = g[c] - g0[c] * e1 - g1[6 * j + c] * e2;
}

// H(s_i, phi_j) = sum_q w_q exp(-i s_i z_q) R(phi_j, z_q) + 2 G0 K0(s) - 2 i s g1 K0(s),
// stored as e^{s_i} H; the phase advances by a complex rotation per node (host tables
// ph0, step).
// Column i = ns holds the regularised kappa = 0 value (real): sum_q w_q R + 2 G0 (log 2 - gamma).
__global__ void __launch_bounds__(NTL) k_cgf_transform(CgfConst k, const double* __restrict__ rem,
                                                       const double* __restrict__ g0,
                                                       const double* __restrict__ g1,
                                                       const double2* __restrict__ ph0,
                                                       const double2* __restrict__ step,
                                                       const double* __restrict__ k0s,
                                                       double2* __restrict__ H) {
    const int idx = blockIdx.x * NTL + threadIdx.x;
    if (idx >= k.nphi * (k.ns + 1)) return;
    const int j = idx / (k.ns + 1);
    const int i = idx - j * (k.ns + 1);
    const double* rj = rem + (int64_t)j * k.nzq * 6;
    double2 acc[6];
    for (int c = 0; c < 6; ++c) acc[c] = make_double2(0, 0);
    if (i < k.ns) {
        double2 ph = ph0[i];
        const double2 st = step[i];
        for (int q = 0; q < k.nzq; ++q) {
            const double w = (q == 0 || q == k.nzq - 1) ? 0.5 * k.dz : k.dz;
            const double pr = w * ph.x, pi = w * ph.y;
            for (int c = 0; c < 6; ++c) {
                const double r = rj[q * 6 + c];
                acc[c].x += pr * r;
                acc[c].y += pi * r;
            }
            ph = make_double2(ph.x * st.x - ph.y * st.y, ph.x * st.y + ph.y * st.x);
        }
        const double K0 = k0s[2 * i], s = k0s[2 * i + 1];      // K0(s_i), s_i (host table)
        // stored times e^{s}: the transform decays roughly like e^{-s}, and the scaled
        // function varies slowly enough for cubic interpolation between nodes
        const double es = exp(s);
        for (int c = 0; c < 6; ++c) {
            acc[c].x = (acc[c].x + 2.0 * g0[c] * K0) * es;
            acc[c].y = (acc[c].y - 2.0 * s * g1[6 * j + c] * K0) * es;
        }
    } else {
        for (int q = 0; q < k.nzq; ++q) {
            const double w = (q == 0 || q == k.nzq - 1) ? 0.5 * k.dz : k.dz;
            for (int c = 0; c < 6; ++c) acc[c].x += w * rj[q * 6 + c];
        }
        for (int c = 0; c < 6; ++c) acc[c].x += 2.0 * g0[c] * (M_LN2 - 0.57721566490153286061);
    }
    for (int c = 0; c < 6; ++c) H[(int64_t)idx * 6 + c] = acc[c];
}

// ----------------------------------------------------------------------------------
// Evaluation of the far-field block at (theta0, dn1, dn2): Catmull-Rom interpolation
// of H in (log s, phi), the small-s logarithm below s_min, zero above s_max.
// ----------------------------------------------------------------------------------
__device__ inline double cr_w(double t, int k) {
    // Catmull-Rom weights for points -1, 0, 1, 2 at parameter t in [0, 1)
    const double t2 = t * t, t3 = t2 * t;
    switch (k) {
        case 0: return 0.5 * (-t3 + 2.0 * t2 - t);
        case 1: return 0.5 * (3.0 * t3 - 5.0 * t2 + 2.0);
        case 2: return 0.5 * (-3.0 * t3 + 4.0 * t2 + t);
        default: return 0.5 * (t3 - t2);
    }
}

__device__ void cgf_eval(const CgfView& v, double theta0, int dn1, int dn2, double2 out[6]) {
    const double x = 0.5 * dn1;
    const double y = (dn1 + 2.0 * dn2) * (0.5 * M_SQRT1_2);
    const double rho = sqrt(x * x + y * y);
    double phi = atan2(y, x);
    if (phi < 0.0) phi += 2.0 * M_PI;
    const double fp = phi / (2.0 * M_PI) * v.nphi;
    int jp = (int)floor(fp);
    const double tp = fp - jp;
    const double inv_c = M_SQRT2;    // 1 / c with c = a / sqrt 2, a = 1
    for (int c = 0; c < 6; ++c) out[c] = make_double2(0, 0);
    if (theta0 == 0.0) {
        for (int a = 0; a < 4; ++a) {
            const int jj = ((jp - 1 + a) % v.nphi + v.nphi) % v.nphi;
            const double wa = cr_w(tp, a);
            for (int c = 0; c < 6; ++c) out[c].x += wa * v.H[((int64_t)jj * (v.ns + 1) + v.ns) * 6 + c].x;
        }
        const double lr = log(rho);
        for (int c = 0; c < 6; ++c) out[c].x = (out[c].x - 2.0 * v.g0[c] * lr) * inv_c;
        return;
    }
    const double kappa = 2.0 * M_PI * theta0 * inv_c;
    const double s = kappa * rho;
    if (s > v.s_max) return;
    double ls = log(s);
    double extra = 0.0;       // below s_min: H(s) = H(s_min) - 2 G0 log(s / s_min)
    if (ls < v.ls_min) {
        extra = ls - v.ls_min;
        ls = v.ls_min;
    }
    const double fs = (ls - v.ls_min) / v.dls;
    int is = (int)floor(fs);
    double ts = fs - is;
    if (is >= v.ns - 1) {
        is = v.ns - 2;
        ts = 1.0;
    }
    for (int a = 0; a < 4; ++a) {
        const int jj = ((jp - 1 + a) % v.nphi + v.nphi) % v.nphi;
        const double wa = cr_w(tp, a);
        for (int b = 0; b < 4; ++b) {
            const int ii = min(max(is - 1 + b, 0), v.ns - 1);
            const double w = wa * cr_w(ts, b);
            const double2* h = v.H + ((int64_t)jj * (v.ns + 1) + ii) * 6;
            for (int c = 0; c < 6; ++c) {
                out[c].x += w * h[c].x;
                out[c].y += w * h[c].y;
            }
        }
    }
    const double unscale = exp(-exp(ls));      // table holds e^{s} H
    for (int c = 0; c < 6; ++c) {
        out[c].x *= unscale;
        out[c].y *= unscale;
    }
    if (extra != 0.0)
        for (int c = 0; c < 6; ++c) out[c].x -= 2.0 * v.g0[c] * extra;
    double sp, cp;
    sincospi(theta0 * dn1, &sp, &cp);
    for (int c = 0; c < 6; ++c) {
        const double re = out[c].x * cp - out[c].y * sp;
        const double im = out[c].x * sp + out[c].y * cp;
        out[c] = make_double2(re * inv_c, im * inv_c);
    }
}

__global__ void __launch_bounds__(NTL) k_cgf_points(CgfView v, const double* __restrict__ theta0,
                                                    const int32_t* __restrict__ d1,
                                                    const int32_t* __restrict__ d2, int n,
                                                    double2* __restrict__ out) {
    const int i = blockIdx.x * NTL + threadIdx.x;
    if (i >= n) return;
    double2 o[6];
    cgf_eval(v, theta0[i], d1[i], d2[i], o);
    for (int c = 0; c < 6; ++c) out[(int64_t)i * 6 + c] = o[c];
}

void launch_cgf_points(hipStream_t st, const CgfView& v, const double* theta0, const int32_t* d1,
                       const int32_t* d2, int n, double2* out) {
    if (n > 0)
        hipLaunchKernelGGL(k_cgf_points, dim3((n + NTL - 1) / NTL), dim3(NTL), 0, st, v, theta0, d1,
                           d2, n, out);
}

void launch_cgf_build(hipStream_t st, const CgfConst& k, const double* cpsi, const double* spsi,
                      const double* rhat, double* g0, double* g1, double* rem, const double2* ph0,
                      const double2* step, const double* k0s, double2* H) {
    hipLaunchKernelGGL(k_cgf_g, dim3((k.nphi + 1 + 63) / 64), dim3(64), 0, st, k, cpsi, spsi, rhat, g0, g1);
    const int64_t nrem = (int64_t)k.nphi * k.nzq;
    hipLaunchKernelGGL(k_cgf_rem, dim3((unsigned)((nrem + NTL - 1) / NTL)), dim3(NTL), 0, st, k, cpsi,
                       spsi, rhat, g0, g1, rem);
    const int nh = k.nphi * (k.ns + 1);
    hipLaunchKernelGGL(k_cgf_transform, dim3((nh + NTL - 1) / NTL), dim3(NTL), 0, st, k, rem, g0, g1, ph0,
                       step, k0s, H);
}

// ----------------------------------------------------------------------------------
// MLP 8 -> 128 -> 128 -> 128 -> 12, SiLU, FP32 training kernels.
// Parameter layout: per layer W [out][in] row-major, then b [out].
//
// A work group takes MT samples through every layer and, for training, back: the contractions
// over a layer run on FP32 MFMA (FP32 operands and sums, as scalar FMAs would), a wave for each 16
// rows of a layer and all MT samples, activations in LDS, z in registers between the two passes.
// Weights go from L2 straight to registers (35k of them, the same for every group).  Weight
// gradients, sums over all samples, are FP64 MFMA products of the stored activations and dz, in
// chunks whose partial sums are added in fixed order.  8192 samples: 8 us each of FP32 and of FP64
// MFMA; loss and gradient in three launches 83 us a call (26, 24 and 4 of kernels), with scalar FMAs
// in a launch per layer and step 782.
// ----------------------------------------------------------------------------------
typedef float f4v_t __attribute__((ext_vector_type(4)));
typedef double d4v_t __attribute__((ext_vector_type(4)));

__device__ inline float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ inline float silu_d(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// Offset of a layer's weights in the parameters; its biases follow them.
__host__ __device__ constexpr int layer_off(int l) {
    return l == 0 ? 0 : MLP_H * (MLP_IN + 1) + (l - 1) * MLP_H * (MLP_H + 1);
}
static_assert(layer_off(3) + MLP_OUT * (MLP_H + 1) == MLP_NPARAMS, "layers end to end");

#define MT 32                       // samples of a work group
#define MT_LD (MLP_H + 4)           // row of a sample in LDS: 16-byte reads of 16 samples spread over the banks
#define OUT_LD 16                   // row of dz of the last layer (12 outputs, zeros)

// Training workspace: a and dz of the three hidden layers, dz of the last (n samples), the loss
// partials of the work groups, the chunks' partial gradients.
struct MlpWs {
    float *a[3], *dz[4];
    double *loss, *part;
};
static const int kMaxChunks = 23;
static int mlp_groups(int n) { return (n + MT - 1) / MT; }
int64_t mlp_workspace_floats(int n) {
    return (int64_t)n * (6 * MLP_H + OUT_LD) + 4LL * mlp_groups(n) + 2LL * kMaxChunks * MLP_NPARAMS;
}
static MlpWs mlp_ws(float* ws, int n) {
    MlpWs w;
    double* d = (double*)ws;                      // the doubles first
    w.part = d;
    w.loss = d + (int64_t)kMaxChunks * MLP_NPARAMS;
    float* p = (float*)(w.loss + 2 * mlp_groups(n));
    for (int l = 0; l < 3; ++l) {
        w.a[l] = p + (int64_t)l * n * MLP_H;
        w.dz[l] = p + (int64_t)(3 + l) * n * MLP_H;
    }
    w.dz[3] = p + (int64_t)6 * n * MLP_H;
    return w;
}

// Output row block wave, samples 16 sb + (lane & 15): D register j is output 16 wave + 4 g + j
// (g = lane >> 4).  K steps take inputs 16 q + 4 g + j, so both operands are 16-byte reads.
template <bool TRAIN>
__global__ void __launch_bounds__(512) k_mlp(const float* __restrict__ par, const float* __restrict__ x,
                                             const float* __restrict__ t, int n, float* __restrict__ y, MlpWs ws) {
    __shared__ __attribute__((aligned(16))) float act[2][MT * MT_LD];
    __shared__ __attribute__((aligned(16))) float dzo[MT * (OUT_LD + 4)];
    constexpr int SB = MT / 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int col = lane & 15, g = lane >> 4, row = 16 * wave + col, o4 = 16 * wave + 4 * g;
    const int s0 = blockIdx.x * MT;
    // forward operand of hidden layer l: its rows' weights along the inputs; backward: along the outputs
    auto load_w = [&](f4v_t (&w)[8], int l) {
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = *(const f4v_t*)(par + layer_off(l) + row * MLP_H + 16 * q + 4 * g);
    };
    auto load_wt = [&](f4v_t (&w)[8], int l) {
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) w[q][j] = par[layer_off(l) + (16 * q + 4 * g + j) * MLP_H + row];
    };
    auto product = [&](f4v_t (&acc)[SB], const f4v_t (&w)[8], const float* in) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            f4v_t b[SB];
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) b[sb] = *(const f4v_t*)(in + (16 * sb + col) * MT_LD + 16 * q + 4 * g);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int sb = 0; sb < SB; ++sb)
                    acc[sb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q][j], b[sb][j], acc[sb], 0, 0, 0);
        }
    };
    // a value of this wave's rows for the next layer (LDS) and for the weight gradients
    auto keep = [&](float* out, float* glob, int sb, const f4v_t& v) {
        const int s = 16 * sb + col;
        if (out) *(f4v_t*)(out + s * MT_LD + o4) = v;
        if (TRAIN && s0 + s < n) *(f4v_t*)(glob + (int64_t)(s0 + s) * MLP_H + o4) = v;
    };
    auto bias = [&](int l, int ni) { return *(const f4v_t*)(par + layer_off(l) + MLP_H * ni + o4); };

    f4v_t w[8], wn[8], z[3][SB];
    load_w(w, 1);
    {
        float w0[2], xv[SB][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            w0[j] = par[row * MLP_IN + 2 * g + j];
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) {
                const int s = s0 + 16 * sb + col;
                const float v = x[(int64_t)min(s, n - 1) * MLP_IN + 2 * g + j];
                xv[sb][j] = s < n ? v : 0.0f;
            }
        }
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            z[0][sb] = bias(0, MLP_IN);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                z[0][sb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[j], xv[sb][j], z[0][sb], 0, 0, 0);
        }
    }
#pragma unroll
    for (int l = 0; l < 3; ++l) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            f4v_t v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = silu(z[l][sb][j]);
            keep(act[l & 1], ws.a[l], sb, v);
        }
        __syncthreads();
        if (l == 2) break;
        if (l == 0) load_w(wn, 2);
        const f4v_t b0 = bias(l + 1, MLP_H);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) z[l + 1][sb] = b0;
        product(z[l + 1], l == 0 ? w : wn, act[l & 1]);
    }
    if (TRAIN) load_wt(w, 2);
    // last layer: a wave for 16 samples, rows 12 .. 15 zero
    if (wave < SB) {
        f4v_t acc = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (4 * g + j < MLP_OUT) acc[j] = par[layer_off(3) + MLP_OUT * MLP_H + 4 * g + j];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            f4v_t wv = *(const f4v_t*)(par + layer_off(3) + min(col, MLP_OUT - 1) * MLP_H + 16 * q + 4 * g);
            const f4v_t b = *(const f4v_t*)(act[0] + (16 * wave + col) * MT_LD + 16 * q + 4 * g);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(col < MLP_OUT ? wv[j] : 0.0f, b[j], acc, 0, 0, 0);
        }
        const int s = s0 + 16 * wave + col;
        const bool on = s < n && g < 3;
        if constexpr (!TRAIN) {
            if (on)
#pragma unroll
                for (int j = 0; j < 4; ++j) y[(int64_t)s * MLP_OUT + 4 * g + j] = acc[j];
        } else {
            // loss: mean over samples of the sum over outputs of (y - t)^2; dy = 2 (y - t) / n
            f4v_t dy = {0, 0, 0, 0};
            double loss = 0.0;
            if (on)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d = acc[j] - t[(int64_t)s * MLP_OUT + 4 * g + j];
                    dy[j] = 2.0f * d / n;
                    loss += (double)d * d;
                }
            for (int m = 32; m > 0; m >>= 1) loss += __shfl_xor(loss, m);
            if (lane == 0) ws.loss[(int64_t)blockIdx.x * SB + wave] = loss;
            *(f4v_t*)(dzo + (16 * wave + col) * (OUT_LD + 4) + 4 * g) = dy;
            if (s < n) *(f4v_t*)(ws.dz[3] + (int64_t)s * OUT_LD + 4 * g) = dy;
        }
    }
    if constexpr (TRAIN) {
        __syncthreads();
        f4v_t da[SB];
        float w3[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float v = par[layer_off(3) + min(4 * g + j, MLP_OUT - 1) * MLP_H + row];
            w3[j] = g < 3 ? v : 0.0f;
        }
        load_wt(wn, 1);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            const f4v_t b = *(const f4v_t*)(dzo + (16 * sb + col) * (OUT_LD + 4) + 4 * g);
            da[sb] = (f4v_t){0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 4; ++j) da[sb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w3[j], b[j], da[sb], 0, 0, 0);
        }
#pragma unroll
        for (int l = 2; l >= 0; --l) {
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) {
                f4v_t v;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = da[sb][j] * silu_d(z[l][sb][j]);
                keep(l ? act[(l + 1) & 1] : nullptr, ws.dz[l], sb, v);
                da[sb] = (f4v_t){0, 0, 0, 0};
            }
            if (l == 0) break;
            __syncthreads();
            product(da, l == 2 ? w : wn, act[(l + 1) & 1]);
        }
    }
}

// Partial gradients of a chunk of samples: dW[o][i] = sum_s dz[s][o] in[s][i], db[o] = sum_s
// dz[s][o], in FP64.  A wave takes 16 outputs x 64 inputs (all 8 of the first layer); the four
// waves of a group share rows or columns.  Column lane & 15 of block c is input 4 (lane & 15) + c,
// so a lane's four operands are one 16-byte load (the input of the network may lie at any float).
#define GRAD_TILES (8 + 16 + 16 + 2)
__global__ void __launch_bounds__(256) k_mlp_grad(const float* __restrict__ x, int n, int chunk, MlpWs ws) {
    const int tile = 4 * blockIdx.x + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= GRAD_TILES) return;
    const int sa = blockIdx.y * chunk, sb = min(n, sa + chunk);
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int l = tile < 16 ? 1 : tile < 32 ? 2 : tile < 40 ? 0 : 3;
    const int ob = l == 1 ? tile >> 1 : l == 2 ? (tile - 16) >> 1 : l == 0 ? tile - 32 : 0;
    const int half = l == 0 ? 0 : tile & 1;
    const int no = l == 3 ? MLP_OUT : MLP_H, ni = l == 0 ? MLP_IN : MLP_H;
    const int ldo = l == 3 ? OUT_LD : MLP_H;
    const float* dz = ws.dz[l] + 16 * ob + col;
    const float* in = l == 0 ? x + 4 * min(col, MLP_IN / 4 - 1) : ws.a[l - 1] + 64 * half + 4 * col;
    d4v_t acc[4] = {};
    double db = 0.0;
    auto run = [&](auto aligned) {
        constexpr int U = 8;
        float a[U];
        f4v_t b[U];
        auto load = [&](int s) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = min(s + 4 * u + g, sb - 1);
                a[u] = dz[q * ldo];
                if constexpr (decltype(aligned)::value)
                    b[u] = *(const f4v_t*)(in + q * MLP_H);
                else
                    for (int c = 0; c < 4; ++c) b[u][c] = in[q * MLP_IN + c];
            }
        };
        load(sa);
        for (int s = sa; s < sb; s += 4 * U) {
            float av[U];
            f4v_t bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool on = s + 4 * u + g < sb;
                av[u] = on ? a[u] : 0.0f;
                for (int c = 0; c < 4; ++c) bv[u][c] = on ? b[u][c] : 0.0f;
            }
            load(s + 4 * U);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                db += av[u];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[u], (double)bv[u][c], acc[c], 0, 0, 0);
            }
        }
    };
    if (l == 0) run(std::false_type());
    else run(std::true_type());
    double* part = ws.part + (int64_t)blockIdx.y * MLP_NPARAMS + layer_off(l);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int o = 16 * ob + 4 * j + g, i = 64 * half + 4 * col + c;      // FP64-accumulator output order
            if (o < no && i < ni) part[o * ni + i] = acc[c][j];
        }
    if (half == 0) {
        db += __shfl_xor(db, 16);
        db += __shfl_xor(db, 32);
        const int o = 16 * ob + col;
        if (g == 0 && o < no) part[no * ni + o] = db;
    }
}

// Adds the chunks in fixed order; the last work group adds the loss partials.
__global__ void __launch_bounds__(NTL) k_mlp_sum(int nchunk, int nloss, int n, MlpWs ws, float* __restrict__ grad,
                                                 float* __restrict__ loss) {
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ double red[NTL];
        double s = 0.0;
        for (int i = threadIdx.x; i < nloss; i += NTL) s += ws.loss[i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int st = NTL / 2; st > 0; st >>= 1) {
            if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = (float)(red[0] / n);
        return;
    }
    const int idx = blockIdx.x * NTL + threadIdx.x;
    if (idx >= MLP_NPARAMS) return;
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < nchunk; ++c) s += ws.part[(int64_t)c * MLP_NPARAMS + idx];
    grad[idx] = (float)s;
}

__global__ void __launch_bounds__(NTL) k_adam(float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, int n,
                                              float lr, float b1, float b2, float eps, float c1,
                                              float c2) {
    const int i = blockIdx.x * NTL + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

void launch_mlp_forward(hipStream_t st, const float* params, const float* x, int n, float* ws,
                        float* y) {
    // samples are read and written group by group: an output over the input goes through the workspace
    const bool over = y < x + (int64_t)n * MLP_IN && x < y + (int64_t)n * MLP_OUT;
    hipLaunchKernelGGL(k_mlp<false>, dim3(mlp_groups(n)), dim3(512), 0, st, params, x, nullptr, n, over ? ws : y, MlpWs{});
    if (over) (void)hipMemcpyAsync(y, ws, (int64_t)n * MLP_OUT * 4, hipMemcpyDeviceToDevice, st);
}

void launch_mlp_loss_grad(hipStream_t st, const float* params, const float* x, const float* t, int n, float* ws,
                          float* grad, float* loss) {
    const MlpWs w = mlp_ws(ws, n);
    // chunks of 32 samples or more; 23 of them at most are a work group for each CU (8192 samples: 24.5
    // us; 32 chunks 27.2, the last round nearly empty; 46 chunks 23.4, but 2 us more to add them up)
    const int chunk = std::max(32, ((n + kMaxChunks - 1) / kMaxChunks + 3) & ~3);
    const int nchunk = (n + chunk - 1) / chunk;
    hipLaunchKernelGGL(k_mlp<true>, dim3(mlp_groups(n)), dim3(512), 0, st, params, x, t, n, nullptr, w);
    hipLaunchKernelGGL(k_mlp_grad, dim3((GRAD_TILES + 3) / 4, nchunk), dim3(256), 0, st, x, n, chunk, w);
    hipLaunchKernelGGL(k_mlp_sum, dim3((MLP_NPARAMS + NTL - 1) / NTL + 1), dim3(NTL), 0, st, nchunk,
                       mlp_groups(n) * (MT / 16), n, w, grad, loss);
}

void launch_adam(hipStream_t st, float* p, const float* g, float* m, float* v, int n, float lr, int step) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((n + NTL - 1) / NTL), dim3(NTL), 0, st, p, g, m, v, n, lr, b1, b2, eps, c1,
                       c2);
}

// ----------------------------------------------------------------------------------
// Training samples and the surrogate table generator.
// Features of (theta0, dn1, dn2): (cos phi, sin phi, cos 2phi, sin 2phi, cos 4phi,
// sin 4phi, r_c / rho, 8 theta0); the low angular harmonics of the cubic anisotropy
// are given explicitly.
// Target / output: exp(-i pi theta0 dn1) (G^_lgf - G^_cgf) / env, 6 complex components
// (xx yy zz xy xz yz) as 12 reals, with env = env_mode[t] = exp(-s_exact) times the
// largest block of table mode t: the learned band starts where the lattice blocks fall
// below that, so the targets are of order one or less and the network's absolute error
// is spread evenly over the band (the continuum is zero beyond kappa rho = 40, where the
// lattice values at large theta0 still matter; a relative envelope would vanish there).
// ----------------------------------------------------------------------------------
__device__ inline void sur_features(double theta0, int dn1, int dn2, double r_c, float f[MLP_IN],
                                    double* rho_out) {
    const double x = 0.5 * dn1;
    const double y = (dn1 + 2.0 * dn2) * (0.5 * M_SQRT1_2);
    const double rho = sqrt(x * x + y * y);
    const double c1 = x / rho, s1 = y / rho;
    const double c2 = c1 * c1 - s1 * s1, s2 = 2.0 * s1 * c1;
    f[0] = (float)c1;
    f[1] = (float)s1;
    f[2] = (float)c2;
    f[3] = (float)s2;
    f[4] = (float)(c2 * c2 - s2 * s2);
    f[5] = (float)(2.0 * s2 * c2);
    f[6] = (float)(r_c / rho);
    f[7] = (float)(8.0 * theta0);
    *rho_out = rho;
}



__global__ void __launch_bounds__(NTL) k_sur_samples(CgfView v, const double2* __restrict__ tab,
                                                     int64_t n_off, int nz_tab,
                                                     const int32_t* __restrict__ d1,
                                                     const int32_t* __restrict__ d2,
                                                     const int32_t* __restrict__ pick_t,
                                                     const int32_t* __restrict__ pick_o, int n,
                                                     double r_c, const double* __restrict__ env_mode,
                                                     float* __restrict__ x, float* __restrict__ t) {
    const int i = blockIdx.x * NTL + threadIdx.x;
    if (i >= n) return;
    const int tm = pick_t[i];
    const int64_t o = pick_o[i];
    const double theta0 = (double)tm / nz_tab;
    double2 g[6];
    cgf_eval(v, theta0, d1[o], d2[o], g);
    float f[MLP_IN];
    double rho;
    sur_features(theta0, d1[o], d2[o], r_c, f, &rho);
    const double env = env_mode[tm];
    double sp, cp;
    sincospi(theta0 * d1[o], &sp, &cp);
    const double2* l = tab + ((int64_t)tm * n_off + o) * 6;
    for (int a = 0; a < MLP_IN; ++a) x[(int64_t)i * MLP_IN + a] = f[a];
    for (int c = 0; c < 6; ++c) {
        const double dr = l[c].x - g[c].x, di = l[c].y - g[c].y;
        // multiply by exp(-i pi theta0 dn1)
        t[(int64_t)i * 12 + 2 * c] = (float)((dr * cp + di * sp) / env);
        t[(int64_t)i * 12 + 2 * c + 1] = (float)((di * cp - dr * sp) / env);
    }
}

void launch_sur_samples(hipStream_t st, const CgfView& v, const double2* tab, int64_t n_off, int nz_tab,
                        const int32_t* d1, const int32_t* d2, const int32_t* pick_t,
                        const int32_t* pick_o, int n, double r_c, const double* env_mode, float* x, float* t) {
    if (n > 0)
        hipLaunchKernelGGL(k_sur_samples, dim3((n + NTL - 1) / NTL), dim3(NTL), 0, st, v, tab, n_off, nz_tab,
                           d1, d2, pick_t, pick_o, n, r_c, env_mode, x, t);
}

// MLP forward of one sample, weights transposed ([in][out], read with wave-uniform
// addresses) in BF16 (inference) or FP32 (the control that isolates the weights'
// rounding), FP32 accumulation.  The hidden vector of each thread lives in its own LDS
// column hl[i * stride]; every layer reads its inputs from there and overwrites them with
// its outputs (the column is private to the thread, so no barrier is needed).
#define MLP_BLOCK 64
__device__ inline float wval(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
__device__ inline float wval(float x) { return x; }

template <typename WT>
struct MlpW {
    const WT* w1t;   // [8][128]
    const WT* w2t;   // [128][128]
    const WT* w3t;   // [128][128]
    const WT* w4t;   // [128][12]
    const float* b1;
    const float* b2;
    const float* b3;
    const float* b4;
};

template <typename WT>
__device__ inline MlpW<WT> mlp_view(const WT* w, const float* bias) {
    MlpW<WT> m;
    m.w1t = w;
    m.w2t = m.w1t + MLP_IN * MLP_H;
    m.w3t = m.w2t + MLP_H * MLP_H;
    m.w4t = m.w3t + MLP_H * MLP_H;
    m.b1 = bias;
    m.b2 = m.b1 + MLP_H;
    m.b3 = m.b2 + MLP_H;
    m.b4 = m.b3 + MLP_H;
    return m;
}

template <typename WT>
__device__ inline void mlp_hidden(const WT* __restrict__ wt, const float* __restrict__ b, float* hl, int stride) {
    float acc[MLP_H];
#pragma unroll
    for (int o = 0; o < MLP_H; ++o) acc[o] = b[o];
    for (int i = 0; i < MLP_H; ++i) {
        const float v = hl[i * stride];
        const WT* w = wt + i * MLP_H;
#pragma unroll
        for (int o = 0; o < MLP_H; ++o) acc[o] = fmaf(wval(w[o]), v, acc[o]);
    }
#pragma unroll
    for (int o = 0; o < MLP_H; ++o) hl[o * stride] = silu(acc[o]);
}

template <typename WT>
__device__ void mlp_eval(const MlpW<WT>& m, const float f[MLP_IN], float* hl, int stride, float y[MLP_OUT]) {
    {
        float acc[MLP_H];
#pragma unroll
        for (int o = 0; o < MLP_H; ++o) {
            float a = m.b1[o];
#pragma unroll
            for (int i = 0; i < MLP_IN; ++i) a = fmaf(wval(m.w1t[i * MLP_H + o]), f[i], a);
            acc[o] = a;
        }
#pragma unroll
        for (int o = 0; o < MLP_H; ++o) hl[o * stride] = silu(acc[o]);
    }
    mlp_hidden(m.w2t, m.b2, hl, stride);
    mlp_hidden(m.w3t, m.b3, hl, stride);
#pragma unroll
    for (int o = 0; o < MLP_OUT; ++o) y[o] = m.b4[o];
    for (int i = 0; i < MLP_H; ++i) {
        const float v = hl[i * stride];
#pragma unroll
        for (int o = 0; o < MLP_OUT; ++o) y[o] = fmaf(wval(m.w4t[i * MLP_OUT + o]), v, y[o]);
    }
}

// Far-field block (CGF, optionally + the network's correction with a unit envelope) at
// arbitrary points.
template <typename WT>
__global__ void __launch_bounds__(MLP_BLOCK) k_sur_points(CgfView v, const WT* __restrict__ wt,
                                                          const float* __restrict__ bias, int use_mlp,
                                                          double r_c, const double* __restrict__ theta0,
                                                          const int32_t* __restrict__ d1,
                                                          const int32_t* __restrict__ d2, int n,
                                                          double2* __restrict__ out) {
    __shared__ float hl[MLP_H * MLP_BLOCK];
    const MlpW<WT> m = mlp_view(wt, bias);
    const int i = blockIdx.x * MLP_BLOCK + threadIdx.x;
    if (i >= n) return;
    double2 g[6];
    cgf_eval(v, theta0[i], d1[i], d2[i], g);
    float f[MLP_IN], y[MLP_OUT];
    double rho;
    sur_features(theta0[i], d1[i], d2[i], r_c, f, &rho);
    if (use_mlp && rho > r_c) {
        mlp_eval(m, f, hl + threadIdx.x, MLP_BLOCK, y);
        double sp, cp;
        sincospi(theta0[i] * d1[i], &sp, &cp);
        for (int c = 0; c < 6; ++c) {
            const double cr = y[2 * c], ci = y[2 * c + 1];
            g[c].x += cr * cp - ci * sp;
            g[c].y += cr * sp + ci * cp;
        }
    }
    for (int c = 0; c < 6; ++c) out[(int64_t)i * 6 + c] = g[c];
}

void launch_sur_points(hipStream_t st, const CgfView& v, const MlpInfer& w, int use_mlp, double r_c,
                       const double* theta0, const int32_t* d1,
                       const int32_t* d2, int n, double2* out) {
    if (n <= 0) return;
    const dim3 grid((n + MLP_BLOCK - 1) / MLP_BLOCK);
    if (w.wf)
        hipLaunchKernelGGL(k_sur_points<float>, grid, dim3(MLP_BLOCK), 0, st, v, w.wf, w.bias, use_mlp, r_c,
                           theta0, d1, d2, n, out);
    else
        hipLaunchKernelGGL(k_sur_points<unsigned short>, grid, dim3(MLP_BLOCK), 0, st, v, w.wb, w.bias, use_mlp,
                           r_c, theta0, d1, d2, n, out);
}

// The exact prefix of each table mode t0 .. t0+nt-1 into the generated slice: one
// contiguous run per mode (ragged table: mode t at ex_off[t], n_exact[t] offsets).
__global__ void __launch_bounds__(256) k_sur_copy_exact(const double2* __restrict__ exact_tab,
                                                        const int64_t* __restrict__ ex_off,
                                                        const int32_t* __restrict__ n_exact, int t0, int64_t n_off,
                                                        double2* __restrict__ out) {
    const int tl = blockIdx.y, tm = t0 + tl;
    const int64_t n = (int64_t)n_exact[tm] * 6;
    const double2* src = exact_tab + ex_off[tm] * 6;
    double2* dst = out + (int64_t)tl * n_off * 6;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}

// Table slice generator of the surrogate form: table modes t0 .. t0+nt-1 for every
// offset o (offsets numbered by increasing rho; every band below is a prefix).
// o < n_exact[t]: the exact lattice value (copied from the ragged table by
// k_sur_copy_exact; this kernel starts at o0, the smallest n_exact of the chunk);
// o < n_learn[t]: continuum + learned correction (only out to rho_learn, the largest distance
// of the training data: no extrapolation); o < n_need[t]: continuum alone; beyond:
// zero, not written (the product treats offsets at or beyond n_need[t] as zero).
template <typename WT>
__global__ void __launch_bounds__(MLP_BLOCK) k_sur_generate(CgfView v, const WT* __restrict__ wt,
                                                            const float* __restrict__ bias, double r_c,
                                                            const double* __restrict__ env_mode, double rho_learn,
                                                            int nz_tab, int t0,
                                                            const int32_t* __restrict__ n_exact,
                                                            const int32_t* __restrict__ n_learn,
                                                            int64_t o0, int64_t n_off,
                                                            const int32_t* __restrict__ n_need,
                                                            const int32_t* __restrict__ d1,
                                                            const int32_t* __restrict__ d2,
                                                            double2* __restrict__ out, int band_done) {
    __shared__ float hl[MLP_H * MLP_BLOCK];
    const MlpW<WT> m = mlp_view(wt, bias);
    const int tl = blockIdx.y;
    const int tm = t0 + tl;
    const int64_t o = o0 + (int64_t)blockIdx.x * MLP_BLOCK + threadIdx.x;
    if (o >= n_off) return;
    double2* dst = out + ((int64_t)tl * n_off + o) * 6;
    if (o < n_exact[tm]) return;      // copied by k_sur_copy_exact
    if (band_done && o < n_learn[tm]) return;     // made by k_sur_learned
    if (o >= n_need[tm]) return;      // zero by definition; the product does not read it
    const double theta0 = (double)tm / nz_tab;
    double2 g[6];
    cgf_eval(v, theta0, d1[o], d2[o], g);
    float f[MLP_IN], y[MLP_OUT];
    double rho;
    sur_features(theta0, d1[o], d2[o], r_c, f, &rho);
    const double env = env_mode[tm];
    if (o < n_learn[tm] && rho <= rho_learn) {
        mlp_eval(m, f, hl + threadIdx.x, MLP_BLOCK, y);
        double sp, cp;
        sincospi(theta0 * d1[o], &sp, &cp);
        for (int c = 0; c < 6; ++c) {
            const double cr = env * y[2 * c], ci = env * y[2 * c + 1];
            g[c].x += cr * cp - ci * sp;
            g[c].y += cr * sp + ci * cp;
        }
    }
    for (int c = 0; c < 6; ++c) dst[c] = g[c];
}

// ----------------------------------------------------------------------------------
// Learned band on MFMA: the network's layers are dense products over a batch of samples,
// run as v_mfma_f32_16x16x32_bf16 (weights and activations in BF16, FP32 accumulation,
// biases and SiLU in FP32).  Weights in fragment order (k_mlp_to_mfma): layer l's
// fragment (row block rb, K block kb) is 64 lanes x 8 BF16, lane L holding
// W[16 rb + L % 16][32 kb + 8 (L / 16) + j]; layers 8 -> 128 (K padded to 32), 128 ->
// 128 twice, 128 -> 12 (rows padded to 16).  One wave takes 64 samples (one per lane for
// the continuum, the features and the final combination) and runs the network on them
// in four groups of 16 (the MFMA columns); between layers the activations go through a
// per-wave LDS buffer [sample][row] (row stride 136: the lanes' 8- and 16-byte accesses
// fall on distinct banks), which turns the accumulator layout (rows 16 rb + 4 (L / 16) +
// j) into the operand layout (rows 32 kb + 8 (L / 16) + j).
// ----------------------------------------------------------------------------------
#define LRN_WAVES 4
#define LRN_ACT 136
#define LRN_FRAGS (8 + 32 + 32 + 4)

__device__ inline unsigned short to_bf16(float x) {
    unsigned u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);       // round to nearest even (finite values)
    return (unsigned short)(u >> 16);
}

__device__ inline bf8_t frag_at(const unsigned short* p) { return *(const bf8_t*)p; }

// bias + SiLU of one layer's accumulators, into the activation buffer act[sample][row]
__device__ inline void put_act(unsigned short* act, const f4_t (&acc)[8], const float* __restrict__ b, int lane) {
    const int n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int rb = 0; rb < 8; ++rb) {
        unsigned short h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = to_bf16(silu(acc[rb][j] + b[16 * rb + 4 * q + j]));
        uint2 pk;
        pk.x = (unsigned)h[0] | ((unsigned)h[1] << 16);
        pk.y = (unsigned)h[2] | ((unsigned)h[3] << 16);
        *(uint2*)(act + n * LRN_ACT + 16 * rb + 4 * q) = pk;
    }
}

// Offsets n_exact[t] .. n_learn[t] - 1 of table modes t0 .. t0 + nt - 1: continuum + the
// network's correction (within rho_learn; the continuum alone beyond), as k_sur_generate.
__global__ void __launch_bounds__(64 * LRN_WAVES) k_sur_learned(CgfView v, const unsigned short* __restrict__ wm,
                                                               const float* __restrict__ bias, double r_c,
                                                               const double* __restrict__ env_mode,
                                                               double rho_learn, int nz_tab, int t0,
                                                               const int32_t* __restrict__ n_exact,
                                                               const int32_t* __restrict__ n_learn, int64_t n_off,
                                                               const int32_t* __restrict__ d1,
                                                               const int32_t* __restrict__ d2,
                                                               double2* __restrict__ out) {
    __shared__ __align__(16) unsigned short feat[LRN_WAVES][64][8];
    __shared__ __align__(16) unsigned short act[LRN_WAVES][16 * LRN_ACT];
    __shared__ float yo[LRN_WAVES][64][MLP_OUT];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tl = blockIdx.y, tm = t0 + tl;
    const int64_t o = (int64_t)n_exact[tm] + ((int64_t)blockIdx.x * LRN_WAVES + wave) * 64 + lane;
    const bool live = o < n_learn[tm];
    const double theta0 = (double)tm / nz_tab;
    double2 g[6];
    float f[MLP_IN];
    double rho = 0.0;
    bool use = false;
    if (live) {
        cgf_eval(v, theta0, d1[o], d2[o], g);
        sur_features(theta0, d1[o], d2[o], r_c, f, &rho);
        use = rho <= rho_learn;
    }
#pragma unroll
    for (int a = 0; a < MLP_IN; ++a) feat[wave][lane][a] = use ? to_bf16(f[a]) : (unsigned short)0;
    const int any = __syncthreads_or(use ? 1 : 0);       // work-group uniform
    if (any) {
        const int n = lane & 15, q = lane >> 4;
        unsigned short* aw = act[wave];
        const f4_t zero = {0.f, 0.f, 0.f, 0.f};
        for (int sb = 0; sb < 4; ++sb) {
            f4_t acc[8];
            // layer 1: the 8 features are K rows 0..7 (the first lane quarter), zeros beyond
            bf8_t b1;
            if (q == 0) b1 = *(const bf8_t*)&feat[wave][16 * sb + n][0];
            else b1 = (bf8_t){};
#pragma unroll
            for (int rb = 0; rb < 8; ++rb)
                acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_at(wm + rb * 512 + lane * 8), b1, zero, 0, 0, 0);
            put_act(aw, acc, bias, lane);
            __syncthreads();
            // layers 2 and 3
            for (int l = 0; l < 2; ++l) {
                bf8_t bk[4];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) bk[kb] = *(const bf8_t*)(aw + n * LRN_ACT + 32 * kb + 8 * q);
                __syncthreads();             // every lane has its operands before any overwrite
                const unsigned short* wl = wm + (8 + 32 * l) * 512;
#pragma unroll
                for (int rb = 0; rb < 8; ++rb) {
                    acc[rb] = zero;
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb)
                        acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_at(wl + (rb * 4 + kb) * 512 + lane * 8),
                                                                          bk[kb], acc[rb], 0, 0, 0);
                }
                put_act(aw, acc, bias + MLP_H * (l + 1), lane);
                __syncthreads();
            }
            // layer 4: 12 outputs (rows 12..15 of the fragment are zero)
            bf8_t bk[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) bk[kb] = *(const bf8_t*)(aw + n * LRN_ACT + 32 * kb + 8 * q);
            f4_t a4 = zero;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                a4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_at(wm + (72 + kb) * 512 + lane * 8), bk[kb], a4, 0, 0,
                                                             0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = 4 * q + j;
                if (row < MLP_OUT) yo[wave][16 * sb + n][row] = a4[j] + bias[3 * MLP_H + row];
            }
            __syncthreads();                 // layer 4 has read act; yo complete after the last group
        }
    }
    if (!live) return;
    if (use) {
        const double env = env_mode[tm];
        double sp, cp;
        sincospi(theta0 * d1[o], &sp, &cp);
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            const double cr = env * yo[wave][lane][2 * c], ci = env * yo[wave][lane][2 * c + 1];
            g[c].x += cr * cp - ci * sp;
            g[c].y += cr * sp + ci * cp;
        }
    }
    double2* dst = out + ((int64_t)tl * n_off + o) * 6;
#pragma unroll
    for (int c = 0; c < 6; ++c) dst[c] = g[c];
}

// FP32 weights -> BF16 fragments of k_sur_learned (round to nearest even; zeros in the
// padding).
__global__ void k_mlp_to_mfma(const float* __restrict__ params, unsigned short* __restrict__ wm) {
    for (int e = threadIdx.x; e < LRN_FRAGS * 512; e += blockDim.x) {
        const int fr = e / 512, rem = e - fr * 512, lane = rem / 8, j = rem - lane * 8;
        int l, rb, kb;
        if (fr < 8) { l = 0; rb = fr; kb = 0; }
        else if (fr < 40) { l = 1; rb = (fr - 8) / 4; kb = (fr - 8) % 4; }
        else if (fr < 72) { l = 2; rb = (fr - 40) / 4; kb = (fr - 40) % 4; }
        else { l = 3; rb = 0; kb = fr - 72; }
        const int ni = (l == 0) ? MLP_IN : MLP_H, no = (l == 3) ? MLP_OUT : MLP_H;
        int64_t off = 0;
        if (l > 0) off += (int64_t)MLP_H * MLP_IN + MLP_H;
        if (l > 1) off += (int64_t)MLP_H * MLP_H + MLP_H;
        if (l > 2) off += (int64_t)MLP_H * MLP_H + MLP_H;
        const int row = 16 * rb + (lane & 15), col = 32 * kb + 8 * (lane >> 4) + j;
        wm[e] = (row < no && col < ni) ? to_bf16(params[off + (int64_t)row * ni + col]) : (unsigned short)0;
    }
}

void launch_mlp_to_mfma(hipStream_t st, const float* params, unsigned short* wm) {
    hipLaunchKernelGGL(k_mlp_to_mfma, dim3(1), dim3(256), 0, st, params, wm);
}

void launch_sur_generate(hipStream_t st, const CgfView& v, const MlpInfer& w, double r_c, const double* env_mode,
                         double rho_learn, int nz_tab, int t0, int nt, const double2* exact_tab, const int64_t* ex_off,
                         const int32_t* n_exact, const int32_t* n_learn, int64_t n_off,
                         const int32_t* n_need, const int32_t* d1, const int32_t* d2, double2* out,
                         int64_t min_exact, int64_t max_exact, int64_t min_learn, int64_t max_band, int64_t max_need) {
    if (nt <= 0) return;
    if (max_exact > 0) {
        const int64_t per = (max_exact * 6 + 255) / 256;
        hipLaunchKernelGGL(k_sur_copy_exact, dim3((unsigned)std::min<int64_t>(per, 1024), nt), dim3(256), 0, st,
                           exact_tab, ex_off, n_exact, t0, n_off, out);
    }
    if (w.wf) {          // FP32 control: the whole non-exact prefix on the SIMT network
        if (max_need <= min_exact) return;
        dim3 grid((unsigned)((max_need - min_exact + MLP_BLOCK - 1) / MLP_BLOCK), nt);
        hipLaunchKernelGGL(k_sur_generate<float>, grid, dim3(MLP_BLOCK), 0, st, v, w.wf, w.bias, r_c, env_mode, rho_learn,
                           nz_tab, t0, n_exact, n_learn, min_exact, n_off, n_need, d1, d2, out, 0);
        return;
    }
    if (max_band > 0) {   // learned band on MFMA
        const int64_t per = (max_band + 64 * LRN_WAVES - 1) / (64 * LRN_WAVES);
        hipLaunchKernelGGL(k_sur_learned, dim3((unsigned)per, nt), dim3(64 * LRN_WAVES), 0, st, v, w.wm, w.bias, r_c,
                           env_mode, rho_learn, nz_tab, t0, n_exact, n_learn, n_off, d1, d2, out);
    }
    if (max_need <= min_learn) return;     // continuum alone beyond the learned band
    dim3 grid((unsigned)((max_need - min_learn + MLP_BLOCK - 1) / MLP_BLOCK), nt);
    hipLaunchKernelGGL(k_sur_generate<unsigned short>, grid, dim3(MLP_BLOCK), 0, st, v, w.wb, w.bias, r_c,
                       env_mode, rho_learn, nz_tab, t0, n_exact, n_learn, min_learn, n_off, n_need, d1, d2, out, 1);
}

// FP32 weights -> transposed bf16 (round to nearest even) and biases, for inference.
__global__ void k_mlp_to_bf16(const float* __restrict__ params, unsigned short* __restrict__ wb,
                              float* __restrict__ bias) {
    const int sizes[5] = {MLP_IN, MLP_H, MLP_H, MLP_H, MLP_OUT};
    int64_t off = 0, ow = 0, ob = 0;
    for (int l = 0; l < 4; ++l) {
        const int ni = sizes[l], no = sizes[l + 1];
        for (int e = threadIdx.x; e < no * ni; e += blockDim.x) {
            const int o = e / ni, i = e - o * ni;           // W [o][i] -> Wt [i][o]
            unsigned u = __float_as_uint(params[off + e]);
            u += 0x7FFFu + ((u >> 16) & 1u);
            wb[ow + (int64_t)i * no + o] = (unsigned short)(u >> 16);
        }
        for (int i = threadIdx.x; i < no; i += blockDim.x) bias[ob + i] = params[off + (int64_t)no * ni + i];
        off += (int64_t)no * ni + no;
        ow += (int64_t)no * ni;
        ob += no;
    }
}

void launch_mlp_to_bf16(hipStream_t st, const float* params, unsigned short* wb, float* bias) {
    hipLaunchKernelGGL(k_mlp_to_bf16, dim3(1), dim3(256), 0, st, params, wb, bias);
}

// FP32 weights -> transposed FP32 weights and biases (the inference control without the
// BF16 rounding of the weights).
__global__ void k_mlp_to_f32t(const float* __restrict__ params, float* __restrict__ wf, float* __restrict__ bias) {
    const int sizes[5] = {MLP_IN, MLP_H, MLP_H, MLP_H, MLP_OUT};
    int64_t off = 0, ow = 0, ob = 0;
    for (int l = 0; l < 4; ++l) {
        const int ni = sizes[l], no = sizes[l + 1];
        for (int e = threadIdx.x; e < no * ni; e += blockDim.x) {
            const int o = e / ni, i = e - o * ni;
            wf[ow + (int64_t)i * no + o] = params[off + e];
        }
        for (int i = threadIdx.x; i < no; i += blockDim.x) bias[ob + i] = params[off + (int64_t)no * ni + i];
        off += (int64_t)no * ni + no;
        ow += (int64_t)no * ni;
        ob += no;
    }
}

void launch_mlp_to_f32t(hipStream_t st, const float* params, float* wf, float* bias) {
    hipLaunchKernelGGL(k_mlp_to_f32t, dim3(1), dim3(256), 0, st, params, wf, bias);
}
