// Seed, propagate and fit kernels: one lane per track, structure-of-arrays
// state so that element k of consecutive tracks is one coalesced access.
//
// arXiv:1906.02253 Sec. 2 (vectorised KF track fitting over sets of small
// matrices), Sec. 3.1 (layer-to-layer propagation with per-layer material in
// a constant field), Sec. 3.2 (seeds provided externally).
#include "kf_fit.hpp"

namespace kfmi {

// ---------------------------------------------------------------- seed
template <typename T>
__global__ __launch_bounds__(256) void seed_kernel(int64_t n, int64_t ld, int64_t n_hits,
                                                   const float* __restrict__ hx,
                                                   const float* __restrict__ hy,
                                                   const float* __restrict__ hz,
                                                   const int32_t* __restrict__ seed_hits, double bz,
                                                   T* __restrict__ par, T* __restrict__ cov,
                                                   T* __restrict__ chi2, int32_t* __restrict__ ndf,
                                                   uint32_t* __restrict__ status)
{
    const int64_t b0 = (int64_t)blockIdx.x * blockDim.x, i = b0 + threadIdx.x;
    if (i >= n) return;
    const int32_t a = seed_hits[i], b = seed_hits[ld + i], c = seed_hits[2 * ld + i];
    if (a < 0 || b < 0 || c < 0 || a >= n_hits || b >= n_hits || c >= n_hits) {
        chi2[i] = T(0);
        ndf[i] = -5;
        status[i] = KF_ST_BADINPUT;
        return;
    }
    // computed in FP64 in every precision mode: the curvature is a small
    // cross product of differences (sagitta << chord for stiff tracks)
    using D = double;
    const D x1 = hx[a], y1 = hy[a], z1 = hz[a];
    const D ax = D(hx[b]) - x1, ay = D(hy[b]) - y1;
    const D bx = D(hx[c]) - x1, by = D(hy[c]) - y1;
    const D d12 = sqrt(ax * ax + ay * ay);
    const D d13 = sqrt(bx * bx + by * by);
    const D ex = D(hx[c]) - D(hx[b]), ey = D(hy[c]) - D(hy[b]);
    const D d23 = sqrt(ex * ex + ey * ey);
    // signed curvature of the circle through the three points
    const D h = D(2) * (ax * by - ay * bx) / (d12 * d23 * d13);
    D w = D(0.5) * h * d13;
    w = w > D(1) ? D(1) : (w < D(-1) ? D(-1) : w);
    const D w2 = w * w;
    const D s13 = fabs(w) < D(1e-4) ? d13 * (D(1) + w2 * (D(1.0 / 6.0) + w2 * D(3.0 / 40.0)))
                                     : d13 * asin(w) / w;
    T p[6];
    T P[21];
    p[0] = T(x1);
    p[1] = T(y1);
    p[2] = T(z1);
    p[3] = T(-h / (kKappa * D(bz)));
    p[4] = T(wrap_phi(atan2(by, bx) - D(0.5) * h * s13));
    p[5] = T(atan2(s13, D(hz[c]) - z1));
#pragma unroll
    for (int k = 0; k < 21; ++k) P[k] = T(0);
    P[pk(0, 0)] = P[pk(1, 1)] = P[pk(2, 2)] = T(1);
    P[pk(3, 3)] = T(4);
    P[pk(4, 4)] = P[pk(5, 5)] = T(0.01);
    store_state<T, T, T>(par, cov, ld, b0, threadIdx.x, p, P);
    chi2[i] = T(0);
    ndf[i] = -5;
    status[i] = 0;
}

// ---------------------------------------------------------------- propagate
// LEARN: every lane of the wave runs to the network call (uniform control
// flow around the matrix-core instructions).
template <typename T, typename C, typename U, bool LEARN, bool FIELD, bool MAT>
__global__ __launch_bounds__(256) void propagate_kernel(int64_t n, int64_t ld, T* __restrict__ par,
                                                        T* __restrict__ cov,
                                                        uint32_t* __restrict__ status,
                                                        const int32_t* __restrict__ target,
                                                        const kf_layer* __restrict__ layers,
                                                        int n_layers, kf_params prm, int material,
                                                        MatMap mat, float* __restrict__ path_len,
                                                        int32_t* __restrict__ iters, MlpDev mlp)
{
    const int64_t b0 = (int64_t)blockIdx.x * blockDim.x, i = b0 + threadIdx.x;
    if (!LEARN && i >= n) return;
    const bool inb = i < n;
    const int32_t l = inb ? target[i] : -1;
    uint32_t st = inb ? status[i] : 0u;
    if (l >= n_layers) st |= KF_ST_BADINPUT;
    const bool active = inb && l >= 0 && !(st & kFreezeMask);
    if (!LEARN && !active) {
        status[i] = st;
        if (path_len) path_len[i] = 0.0f;
        if (iters) iters[i] = 0;
        return;
    }
    U p[6];
    C P[21];
    StepLayer<T> L{};
    if (active) {
        load_state(par, cov, ld, b0, threadIdx.x, p, P);
        L = step_layer<T>(layers[l]);
    }
    T s_init = T(-1);
    if (LEARN) {
        float f[kMlpIn] = {0, 0, 0, 0, 0, 0, 0, 0};
        const bool want = active && L.kind == 0;
        if (want) {
            T pt[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) pt[k] = T(p[k]);
            mlp_features(pt, L, prm, f);
        }
        const uint64_t wmask = __ballot(want);
        const float y = wmask ? mlp_wave(mlp, f, wmask) : 0.0f;
        if (want) s_init = T(mlp_guess(f, y));
        if (!inb) return;
        if (!active) {
            status[i] = st;
            if (path_len) path_len[i] = 0.0f;
            if (iters) iters[i] = 0;
            return;
        }
    }
    T s = T(0);
    int ev = 0, fb = 0;
    const bool finite = wave_all(all_finite(P));
    int r = propagate_to<T, C, U, FIELD, MAT>(p, P, L, prm, material != 0, mat, finite, s_init, &s, &ev, &fb);
    if (fb) st |= KF_ST_FALLBACK;
    if (r) {
        st |= (uint32_t)r;
    } else {
        store_state(par, cov, ld, b0, threadIdx.x, p, P);
    }
    status[i] = st;
    if (path_len) path_len[i] = float(s);
    if (iters) iters[i] = ev;
}

// ---------------------------------------------------------------- launchers
static inline dim3 grid_for(int64_t n, int block) { return dim3((unsigned)((n + block - 1) / block)); }

hipError_t launch_seed(const kf_ctx* ctx, const kf_hits* h, const int32_t* seed_hits,
                       kf_tracks* out, int flags, hipStream_t s)
{
    if (out->n == 0) return hipSuccess;
    const int prec = flags & KF_PREC_MASK;
    dim3 g = grid_for(out->n, 256);
    if (prec == KF_PREC_FP64)
        seed_kernel<double><<<g, 256, 0, s>>>(out->n, out->ld, h->n, h->x, h->y, h->z, seed_hits,
                                              ctx->params.bz, (double*)out->par, (double*)out->cov,
                                              (double*)out->chi2, out->ndf, out->status);
    else
        seed_kernel<float><<<g, 256, 0, s>>>(out->n, out->ld, h->n, h->x, h->y, h->z, seed_hits,
                                             ctx->params.bz, (float*)out->par, (float*)out->cov,
                                             (float*)out->chi2, out->ndf, out->status);
    return hipGetLastError();
}

hipError_t launch_propagate(const kf_ctx* ctx, kf_tracks* t, const int32_t* target, float* path_len,
                            int32_t* iters, int flags, hipStream_t s)
{
    if (t->n == 0) return hipSuccess;
    const int prec = flags & KF_PREC_MASK;
    const int material = (flags & KF_NO_MATERIAL) ? 0 : 1;
    const bool learn = (flags & KF_INIT_MLP) != 0;
    const MlpDev m = ctx->mlp.dev();
    dim3 g = grid_for(t->n, 256);
    const bool field = ctx->params.field_z0 > 0.0, map = ctx->mat.x0 != nullptr;
#define KF_PROP1(TT, CC, UU, LL, FF, MM)                                                             \
    propagate_kernel<TT, CC, UU, LL, FF, MM><<<g, 256, 0, s>>>(t->n, t->ld, (TT*)t->par, (TT*)t->cov, \
                                                               t->status, target, ctx->d_layers,   \
                                                               ctx->n_layers, ctx->params,         \
                                                               material, ctx->mat, path_len, iters, \
                                                               m)
#define KF_PROP(TT, CC, UU, LL)                                                                      \
    do {                                                                                             \
        if (field) {                                                                                 \
            if (map) KF_PROP1(TT, CC, UU, LL, true, true);                                           \
            else KF_PROP1(TT, CC, UU, LL, true, false);                                              \
        } else {                                                                                     \
            if (map) KF_PROP1(TT, CC, UU, LL, false, true);                                          \
            else KF_PROP1(TT, CC, UU, LL, false, false);                                             \
        }                                                                                            \
    } while (0)
    if (prec == KF_PREC_FP64) {
        if (learn) KF_PROP(double, double, double, true);
        else KF_PROP(double, double, double, false);
    } else if (prec == KF_PREC_FP32) {
        if (learn) KF_PROP(float, float, float, true);
        else KF_PROP(float, float, float, false);
    } else {
        if (learn) KF_PROP(float, double, double, true);
        else KF_PROP(float, double, double, false);
    }
#undef KF_PROP
#undef KF_PROP1
    return hipGetLastError();
}

// 64 bits.  At most one workgroup (four waves) a compute unit: one wave a SIMD
// with all its registers; more tracks: two waves (kf_fit64.hip).  Uniform 1 ..
// 10 GeV tracks, hits in random order: 60,000 tracks 70 us by one wave and 74 by
// two, 65,537 110 and 89, 200,000 267 and 254.
template <bool LEARN>
static void fit_launch_fp64(const FitArgs& a, dim3 g, int n_cu, int k0, int k1, int init, bool field,
                            bool map, hipStream_t s)
{
    if ((int64_t)g.x <= n_cu) fit_launch<double, double, double, LEARN, kAnySteps, 1>(a, g, k0, k1, init, field, map, s);
    else launch_fit64(a, g, k0, k1, init, LEARN, field, map, s);
}

hipError_t launch_fit(const kf_ctx* ctx, kf_tracks* t, const kf_hits* h, const int32_t* layer_seq,
                      const int32_t* hit_idx, int32_t max_steps, int flags, hipStream_t s)
{
    if (t->n == 0) return hipSuccess;
    FitArgs a;
    a.n = t->n;
    a.ld = t->ld;
    a.par = t->par;
    a.cov = t->cov;
    a.chi2 = t->chi2;
    a.ndf = t->ndf;
    a.status = t->status;
    a.hx = h->x;
    a.hy = h->y;
    a.hz = h->z;
    a.hsu = h->su;
    a.hsv = h->sv;
    a.layer_seq = layer_seq;
    a.hit_idx = hit_idx;
    a.n_hits = h->n;
    a.layers = ctx->d_layers;
    a.n_layers = ctx->n_layers;
    a.prm = ctx->params;
    a.material = (flags & KF_NO_MATERIAL) ? 0 : 1;
    a.mat = ctx->mat;
    a.mlp = ctx->mlp.dev();
    const bool learn = (flags & KF_INIT_MLP) != 0;
    const int prec = flags & KF_PREC_MASK;
    dim3 g = grid_for(t->n, kFitThreads);
    a.index_ahead = (int64_t)g.x <= ctx->n_cu || (int64_t)g.x > 3 * (int64_t)ctx->n_cu;
    const bool per_layer = (flags & KF_PER_LAYER) != 0;
    const bool field = ctx->params.field_z0 > 0.0, map = ctx->mat.x0 != nullptr;
    const int nlaunch = per_layer ? max_steps : 1;
    for (int k = 0; k < nlaunch; ++k) {
        const int k0 = per_layer ? k : 0;
        const int k1 = per_layer ? k + 1 : max_steps;
        const int init = k == 0;
        if (prec == KF_PREC_FP64) {
            if (learn) fit_launch_fp64<true>(a, g, ctx->n_cu, k0, k1, init, field, map, s);
            else fit_launch_fp64<false>(a, g, ctx->n_cu, k0, k1, init, field, map, s);
        } else if (prec == KF_PREC_FP32) {
            if (learn) fit_launch<float, float, float, true, kAnySteps, 2>(a, g, k0, k1, init, field, map, s);
            else fit_launch<float, float, float, false, kAnySteps, 2>(a, g, k0, k1, init, field, map, s);
        } else if (k1 - k0 == 1) {
            if (learn) fit_launch<float, double, double, true, kOneStep, 2>(a, g, k0, k1, init, field, map, s);
            else fit_launch<float, double, double, false, kOneStep, 2>(a, g, k0, k1, init, field, map, s);
        } else {
            if (learn) fit_launch<float, double, double, true, kManySteps, 2>(a, g, k0, k1, init, field, map, s);
            else fit_launch<float, double, double, false, kManySteps, 2>(a, g, k0, k1, init, field, map, s);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kfmi
