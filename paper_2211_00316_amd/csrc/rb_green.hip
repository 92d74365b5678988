// Green's-function assembly, residual, back-projection scaling and model update (gfx950).
//
// Eq. 2D_greens: g = A exp(i [phi + pi/4]) with A_geom = A_tab / sqrt(k0);
// Eq. phase-discretised: phi = omega T - (pi/2) K (lossless);
// Eq. greens-time-reversed: g_dagger = A^-1 exp(-i [phi + pi/4]);
// Eq. sound_speed_update2: angular weights |d gamma_e / d e| De (central difference over
// neighbouring transducers), pair weight |kbar| |d|kbar|/d omega| = (2k/c)(1 + u_e . u_r)
// split into the three operands H, H u_x, H u_y; scale S = (Domega/(2 pi)^3)(2k/c)/omega^2.
// Eq. residual: g_res = g - data; Section 3.4: m <- m + tau dm, c = m^-1/2 (FP64).
//
// These kernels are elementwise and bound by HBM bandwidth: each reads its table entries
// once and writes the operands with coalesced 8-byte stores; only the phase is in FP64.
#include "rb_internal.h"

namespace {

__device__ __forceinline__ double reduce_phase(double ph) {
    return ph - RB_TWO_PI * floor(ph / RB_TWO_PI);
}

// One thread per mask node q and ROWS consecutive transducers. Bound by HBM: 53 bytes per
// (transducer, node), 21 read and 32 written. The angular weight takes the rays of the two
// neighbouring transducers, 18 bytes more; a thread keeps the directions and flags of three rows
// and moves up, so that only a group's two outer rows are read twice. With one transducer per
// thread the neighbours' rows came from beyond L2 again (512 transducers, 152 053 nodes: 0.72
// against 0.94 ms). Small launches take two rows per thread, for their latency.
// gs (nullable): per-node complex factor applied to G (the frequency step stores
// G sqrt(v), so that the Born term is the plain symmetric product); write_g = 0 skips G.
struct GreenRay {
    float ux, uy;
    bool valid;
    uint8_t f;
};
template <int ROWS>
__global__ void __launch_bounds__(256) green_kernel(rb_tables tb, int N, int n_mask,
                                                    double omega, double c0,
                                                    const float2 *__restrict__ gs,
                                                    const float *__restrict__ gscale, int write_g,
                                                    float2 *__restrict__ G,
                                                    float2 *__restrict__ H) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    const int e0 = blockIdx.y * ROWS;
    if (q >= n_mask) return;
    const size_t plane = (size_t)N * n_mask;
    auto ray = [&](int e) {
        e = e < 0 ? e + N : (e >= N ? e - N : e);
        const size_t o = (size_t)e * n_mask + q;
        GreenRay r;
        r.f = tb.flags[o];
        r.ux = tb.ux[o];
        r.uy = tb.uy[o];
        r.valid = r.f & 0x80;
        return r;
    };
    const double k0 = omega / c0;
    const float sk = (float)sqrt(k0);
    float2 f2 = make_float2(1.f, 0.f);
    float sc = 1.f;
    if (write_g && gs) {
        f2 = gs[q];
        sc = gscale[0];
    }
    GreenRay m = ray(e0 - 1), r = ray(e0);
    double T = tb.T[(size_t)e0 * n_mask + q];
    float A = tb.A[(size_t)e0 * n_mask + q];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int e = e0 + k;
        if (e >= N) break;
        const size_t o = (size_t)e * n_mask + q;
        const GreenRay p = ray(e + 1);
        // the next row's, in flight while this one is worked out
        double Tn = 0.0;
        float An = 0.f;
        if (k + 1 < ROWS && e + 1 < N) {
            Tn = tb.T[o + n_mask];
            An = tb.A[o + n_mask];
        }
        float gr = 0.f, gi = 0.f, hr = 0.f, hi = 0.f;
        if (r.valid) {
            const double ph =
                reduce_phase(omega * T + 0.25 * RB_PI - (double)(r.f & 3) * 0.5 * RB_PI);
            float s, c;
            sincosf((float)ph, &s, &c);
            const float ga = A / sk;
            gr = ga * c;
            gi = ga * s;
            if (write_g && gs) {
                const float tr = (gr * f2.x - gi * f2.y) * sc;
                gi = (gr * f2.y + gi * f2.x) * sc;
                gr = tr;
            }
            // angular weight: angle between the ray directions of the neighbouring transducers
            float a = 0.f;
            if (m.valid && p.valid)
                a = 0.5f * fabsf(atan2f(m.ux * p.uy - m.uy * p.ux, m.ux * p.ux + m.uy * p.uy));
            else if (p.valid)
                a = fabsf(atan2f(r.ux * p.uy - r.uy * p.ux, r.ux * p.ux + r.uy * p.uy));
            else if (m.valid)
                a = fabsf(atan2f(m.ux * r.uy - m.uy * r.ux, m.ux * r.ux + m.uy * r.uy));
            const float ha = a * sk / A;
            hr = ha * c;
            hi = -ha * s;
        }
        // directions of invalid entries are not read as numbers
        const float ux = r.valid ? r.ux : 0.f, uy = r.valid ? r.uy : 0.f;
        if (write_g) G[o] = make_float2(gr, gi);
        H[o] = make_float2(hr, hi);
        H[plane + o] = make_float2(hr * ux, hi * ux);
        H[2 * plane + o] = make_float2(hr * uy, hi * uy);
        m = r;
        r = p;
        T = Tn;
        A = An;
    }
}

// R[e][r] = g_rx + d_born - data on valid pairs with e != r; sum |R|^2 into *norm. One
// workgroup per emitter row e: one atomic per row for the norm.
__global__ void __launch_bounds__(256) residual_kernel(const double *__restrict__ rx_T,
                                                       const float *__restrict__ rx_A,
                                                       const uint8_t *__restrict__ rx_flags,
                                                       int N, double omega, double c0,
                                                       const float2 *__restrict__ d_born,
                                                       const float2 *__restrict__ data,
                                                       float2 *__restrict__ R, double *norm) {
    __shared__ double red[4];
    const int e = blockIdx.x;
    const double isk = 1.0 / sqrt(omega / c0);
    double v = 0.0;
    for (int r = threadIdx.x; r < N; r += blockDim.x) {
        const size_t o = (size_t)e * N + r;
        const uint8_t f = rx_flags[o];
        float2 out = make_float2(0.f, 0.f);
        if ((f & 0x80) && r != e) {
            double ph =
                reduce_phase(omega * rx_T[o] + 0.25 * RB_PI - (double)(f & 3) * 0.5 * RB_PI);
            double sn, cs;
            sincos(ph, &sn, &cs);
            double a = (double)rx_A[o] * isk;
            double gr = a * cs, gi = a * sn;
            if (d_born) {
                gr += d_born[o].x;
                gi += d_born[o].y;
            }
            float2 dd = data[o];
            out = make_float2((float)(gr - dd.x), (float)(gi - dd.y));
        }
        R[o] = out;
        v += (double)out.x * out.x + (double)out.y * out.y;
    }
    if (norm) {
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(norm, (red[0] + red[1]) + (red[2] + red[3]));
    }
}

__global__ void adjoint_finish_kernel(int n_mask, int mblocks, const float *__restrict__ parts,
                                      const float2 *__restrict__ w, float *__restrict__ grad) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask) return;
    float sr = 0.f, si = 0.f;
    for (int b = 0; b < mblocks; ++b) {
        sr += parts[(size_t)b * n_mask + q];
        si += parts[(size_t)(mblocks + b) * n_mask + q];
    }
    float2 ww = w[q];
    grad[q] = ww.x * sr + ww.y * si;  // Re{ conj(w) (sr + i si) }
}

template <typename OutT>
__global__ void backproject_finish_kernel(int n_mask, int mblocks, const float *__restrict__ parts,
                                          const double *__restrict__ c_mask, double omega,
                                          double d_omega, OutT *__restrict__ dm, int accumulate) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask) return;
    double sr = 0.0;
    for (int b = 0; b < mblocks; ++b) sr += (double)parts[(size_t)b * n_mask + q];
    double c = c_mask[q];
    double S = 2.0 * d_omega / (RB_TWO_PI * RB_TWO_PI * RB_TWO_PI * omega * c * c);
    double v = -S * sr;
    if (accumulate) v += (double)dm[q];
    dm[q] = (OutT)v;
}

// c at the mask nodes (double) gathered from the full map.
__global__ void gather_mask(const double *__restrict__ c, const int32_t *__restrict__ mask_index,
                            int n_mask, double *__restrict__ cq) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n_mask) cq[q] = c[mask_index[q]];
}

// sv = sqrt(w delta) at the mask nodes (complex: i sqrt(w |delta|) for delta < 0), with
// w = omega^2 h^2 and delta = m - m_s, where m_s = (n_s / c0)^2 is the squared slowness of
// the smoothed map the rays were traced on. Then sum_q G[e,q] v[q] G[r,q] with v = w delta
// is the symmetric product of G sv with itself.
__global__ void rough_part(const double *__restrict__ cq, const float *__restrict__ n_s,
                           const int32_t *__restrict__ mask_index, int n_mask, double c0,
                           double w, float2 *__restrict__ sv) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask) return;
    double c = cq[q];
    double ns = (double)n_s[mask_index[q]];
    double v = w * (1.0 / (c * c) - ns * ns / (c0 * c0));
    float r = (float)sqrt(fabs(v));
    sv[q] = v >= 0.0 ? make_float2(r, 0.f) : make_float2(0.f, r);
}

// Absorbing media (Szabo's model, Section 2.2; Eq. scattering-potential): sv = sqrt(v) with
// v = Upsilon_m h^2 delta complex, Upsilon_m = omega c k~ = omega^2 z, z = 1 + omega^(y-1)
// c alpha0 (tan(pi y/2) + i) from the model's c and alpha0 at the node. The principal square
// root in the cancellation-free form; with alpha0 = 0 it is the lossless root.
__global__ void rough_part_lossy(const double *__restrict__ cq, const double *__restrict__ aq,
                                 const float *__restrict__ n_s,
                                 const int32_t *__restrict__ mask_index, int n_mask, double c0,
                                 double w, double wy1, double tanpy, float2 *__restrict__ sv) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask) return;
    const double c = cq[q];
    const double ns = (double)n_s[mask_index[q]];
    const double delta = 1.0 / (c * c) - ns * ns / (c0 * c0);
    const double t = wy1 * c * aq[q];
    const double vr = w * (1.0 + t * tanpy) * delta, vi = w * t * delta;
    double sr = 0.0, si = 0.0;
    if (vi == 0.0) {
        const double r = sqrt(fabs(vr));
        if (vr >= 0.0) sr = r;
        else si = r;
    } else {
        const double m = sqrt(vr * vr + vi * vi);
        if (vr >= 0.0) {
            sr = sqrt(0.5 * (m + vr));
            si = vi / (2.0 * sr);
        } else {
            const double u = sqrt(0.5 * (m - vr));
            si = copysign(u, vi);
            sr = fabs(vi) / (2.0 * u);
        }
    }
    sv[q] = make_float2((float)sr, (float)si);
}

// Hessian-free direction of an absorbing medium (Eq. sound_speed_update2 with Section 3.4's
// d|kbar|/domega): S = Domega / (2 pi)^3 (2k/c + 2k y tan(pi y/2) omega^(y-1) alpha0)
// / (omega^2 z), k = omega/c + alpha0 tan(pi y/2) omega^y, z as in rough_part_lossy; S is
// complex and dm = -Re{S (sr + i si)} over the complex double sum of the contraction.
template <typename OutT>
__global__ void backproject_finish_lossy_kernel(int n_mask, int mblocks,
                                                const float *__restrict__ parts,
                                                const double *__restrict__ c_mask,
                                                const double *__restrict__ a_mask, double omega,
                                                double base, double tanpy, double wy, double wy1,
                                                double y, OutT *__restrict__ dm, int accumulate) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask) return;
    double sr = 0.0, si = 0.0;
    for (int b = 0; b < mblocks; ++b) {
        sr += (double)parts[(size_t)b * n_mask + q];
        si += (double)parts[(size_t)(mblocks + b) * n_mask + q];
    }
    const double c = c_mask[q], a0 = a_mask[q];
    const double k = omega / c + a0 * tanpy * wy;
    const double s = base * (2.0 * k / c + 2.0 * k * (y * tanpy * wy1 * a0));  // base: Dw/(2pi)^3 w^2
    const double t = wy1 * c * a0;
    const double zr = 1.0 + t * tanpy, zi = t;
    const double iz = 1.0 / (zr * zr + zi * zi);
    const double Sr = s * zr * iz, Si = -s * zi * iz;
    double v = -(Sr * sr - Si * si);
    if (accumulate) v += (double)dm[q];
    dm[q] = (OutT)v;
}

// m <- m + tau dm (FP64); the candidate c is kept aside until every value is finite.
__global__ void update_kernel(const double *__restrict__ cq, const double *__restrict__ dm,
                              int n_mask, double tau, double *__restrict__ c_new, int *flag) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask) return;
    double c = cq[q];
    double m = 1.0 / (c * c) + tau * dm[q];
    double cn = 1.0 / sqrt(m);
    if (!(m > 0.0) || !isfinite(cn)) atomicOr(flag, 2);
    c_new[q] = cn;
}

// Writes the new model on the mask; with `flag` (deferred checks) only while no error bit
// is set, so a failed step and every later one leave c as it was.
__global__ void commit_kernel(const double *__restrict__ c_new,
                              const int32_t *__restrict__ mask_index, int n_mask,
                              const int32_t *__restrict__ flag, double *__restrict__ c) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_mask || (flag && flag[RB_W_FLAGS] != 0)) return;
    c[mask_index[q]] = c_new[q];
}

// Deferred checks: remember the first step that raised an error bit.
__global__ void note_fail_kernel(int32_t *flag, int step) {
    if (threadIdx.x == 0 && flag[RB_W_FLAGS] != 0 && flag[RB_W_FAIL_STEP] < 0)
        flag[RB_W_FAIL_STEP] = step;
}

// Status of a step for the caller, from the context's device words (no host round trip).
__global__ void report_kernel(const int32_t *__restrict__ flag, rb_report *__restrict__ rep) {
    if (threadIdx.x != 0) return;
    const int32_t fl = flag[RB_W_FLAGS];
    rep->status = fl ? (int32_t)RB_ENONFINITE : (int32_t)RB_OK;
    rep->flags = fl;
    rep->lost_nodes = flag[RB_W_LOST];
    rep->reserved = 0;
    rep->ray_samples = *reinterpret_cast<const int64_t *>(flag + RB_W_SAMPLES);
}

__global__ void fill_i32(int32_t *x, int n, int32_t v) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) x[q] = v;
}

__global__ void zero_f64(double *x, int n) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) x[q] = 0.0;
}

inline unsigned blocks(size_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

rb_status rb_launch_green(rb_ctx *ctx, const rb_tables *tb, double omega, double c0,
                          const rb_green *out, const float *gs, const float *gscale,
                          int write_g) {
    // eight rows per thread where that still makes 32 workgroups per CU
    const unsigned cols = blocks(tb->n_mask);
    const bool deep = (size_t)cols * ((tb->n + 7) / 8) >= 32 * (size_t)ctx->n_cu;
    const int rows = deep ? 8 : 2;
    rb_prof_begin(ctx, ST_GREEN);
    hipLaunchKernelGGL(deep ? green_kernel<8> : green_kernel<2>,
                       dim3(cols, (tb->n + rows - 1) / rows), dim3(256), 0, ctx->stream, *tb,
                       tb->n, tb->n_mask, omega, c0, (const float2 *)gs, gscale, write_g,
                       (float2 *)out->G, (float2 *)out->H);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

rb_status rb_launch_residual(rb_ctx *ctx, const rb_tables *tb, double omega, double c0,
                             const float *d_born, const float *data, float *R,
                             double *residual_norm) {
    rb_prof_begin(ctx, ST_RESIDUAL);
    hipLaunchKernelGGL(residual_kernel, dim3(tb->n), dim3(256), 0, ctx->stream, tb->rx_T, tb->rx_A,
                       tb->rx_flags, tb->n, omega, c0, (const float2 *)d_born,
                       (const float2 *)data, (float2 *)R, residual_norm);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

rb_status rb_launch_adjoint_finish(rb_ctx *ctx, int n_mask, int mblocks, const float *parts,
                                   const float *w, float *grad) {
    rb_prof_begin(ctx, ST_FINISH);
    hipLaunchKernelGGL(adjoint_finish_kernel, dim3(blocks(n_mask)), dim3(256), 0, ctx->stream,
                       n_mask, mblocks, parts, (const float2 *)w, grad);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

rb_status rb_launch_backproject_finish(rb_ctx *ctx, int n_mask, int mblocks, const float *parts,
                                       const double *c_mask, double omega, double d_omega,
                                       float *dm, int accumulate) {
    rb_prof_begin(ctx, ST_FINISH);
    hipLaunchKernelGGL(backproject_finish_kernel<float>, dim3(blocks(n_mask)), dim3(256), 0,
                       ctx->stream, n_mask, mblocks, parts, c_mask, omega, d_omega, dm,
                       accumulate);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

// Internal helpers of rb_frequency_step --------------------------------------------------
rb_status rb_launch_gather_mask(rb_ctx *ctx, const double *c, double *cq) {
    int n = (int)ctx->n_mask;
    hipLaunchKernelGGL(gather_mask, dim3(blocks(n)), dim3(256), 0, ctx->stream, c,
                       ctx->d_mask_index, n, cq);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_rough_part(rb_ctx *ctx, const double *cq, const float *n_s, double c0,
                               double w, float *sv) {
    int n = (int)ctx->n_mask;
    hipLaunchKernelGGL(rough_part, dim3(blocks(n)), dim3(256), 0, ctx->stream, cq, n_s,
                       ctx->d_mask_index, n, c0, w, (float2 *)sv);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_backproject_finish_acc(rb_ctx *ctx, int mblocks, const float *parts,
                                           const double *c_mask, double omega, double d_omega,
                                           double *dm_acc) {
    int n = (int)ctx->n_mask;
    rb_prof_begin(ctx, ST_FINISH);
    hipLaunchKernelGGL(backproject_finish_kernel<double>, dim3(blocks(n)), dim3(256), 0,
                       ctx->stream, n, mblocks, parts, c_mask, omega, d_omega, dm_acc, 1);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

rb_status rb_launch_rough_part_lossy(rb_ctx *ctx, const double *cq, const double *aq,
                                     const float *n_s, double c0, double omega, double y,
                                     double h2, float *sv) {
    int n = (int)ctx->n_mask;
    hipLaunchKernelGGL(rough_part_lossy, dim3(blocks(n)), dim3(256), 0, ctx->stream, cq, aq, n_s,
                       ctx->d_mask_index, n, c0, omega * omega * h2, pow(omega, y - 1.0),
                       tan(0.5 * RB_PI * y), (float2 *)sv);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_backproject_finish_lossy(rb_ctx *ctx, int n_mask, int mblocks,
                                             const float *parts, const double *c_mask,
                                             const double *a_mask, double omega, double d_omega,
                                             double y, double *dm_acc, float *dm,
                                             int accumulate) {
    const double base = d_omega / (RB_TWO_PI * RB_TWO_PI * RB_TWO_PI) / (omega * omega);
    const double tanpy = tan(0.5 * RB_PI * y), wy = pow(omega, y), wy1 = pow(omega, y - 1.0);
    rb_prof_begin(ctx, ST_FINISH);
    if (dm_acc)
        hipLaunchKernelGGL(backproject_finish_lossy_kernel<double>, dim3(blocks(n_mask)),
                           dim3(256), 0, ctx->stream, n_mask, mblocks, parts, c_mask, a_mask,
                           omega, base, tanpy, wy, wy1, y, dm_acc, 1);
    else
        hipLaunchKernelGGL(backproject_finish_lossy_kernel<float>, dim3(blocks(n_mask)),
                           dim3(256), 0, ctx->stream, n_mask, mblocks, parts, c_mask, a_mask,
                           omega, base, tanpy, wy, wy1, y, dm, accumulate);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

rb_status rb_launch_zero_f64(rb_ctx *ctx, double *x, int n) {
    hipLaunchKernelGGL(zero_f64, dim3(blocks(n)), dim3(256), 0, ctx->stream, x, n);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_update(rb_ctx *ctx, const double *cq, const double *dm, double tau,
                           double *c_new) {
    int n = (int)ctx->n_mask;
    rb_prof_begin(ctx, ST_UPDATE);
    hipLaunchKernelGGL(update_kernel, dim3(blocks(n)), dim3(256), 0, ctx->stream, cq, dm, n, tau,
                       c_new, ctx->d_flag);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}

rb_status rb_launch_commit(rb_ctx *ctx, const double *c_new, double *c, const int32_t *flag) {
    int n = (int)ctx->n_mask;
    hipLaunchKernelGGL(commit_kernel, dim3(blocks(n)), dim3(256), 0, ctx->stream, c_new,
                       ctx->d_mask_index, n, flag, c);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_note_fail(rb_ctx *ctx, int step) {
    hipLaunchKernelGGL(note_fail_kernel, dim3(1), dim3(64), 0, ctx->stream, ctx->d_flag, step);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_report(rb_ctx *ctx, rb_report *rep) {
    hipLaunchKernelGGL(report_kernel, dim3(1), dim3(64), 0, ctx->stream, ctx->d_flag, rep);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}

rb_status rb_launch_fill_i32(rb_ctx *ctx, int32_t *x, int n, int32_t value) {
    hipLaunchKernelGGL(fill_i32, dim3(blocks(n)), dim3(256), 0, ctx->stream, x, n, value);
    RB_CHECK_LAUNCH(ctx);
    return RB_OK;
}
