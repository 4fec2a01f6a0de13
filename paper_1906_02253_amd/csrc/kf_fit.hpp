// The fit kernel and what the propagation shares with it.
#pragma once

#include "kf_internal.hpp"
#include "kf_math.hpp"
#include "kf_mlp.hpp"

namespace kfmi {

// par and cov are stored in T, the state precision (FP32 in the mixed and
// FP32 modes); in registers the state is held in U (the update precision) and
// the covariance in C (the covariance-arithmetic precision).
// A workgroup's elements start at b0 and lane i takes element b0 + i.  The row
// stride is made opaque at each use, so that the compiler steps one scalar
// address from row to row there instead of keeping all 27 rows' addresses in
// 54 vector registers from the load to the store.
__device__ inline int64_t opaque(int64_t v)
{
    asm volatile("" : "+s"(v));
    return v;
}

template <typename T, typename C, typename U>
__device__ inline void load_state(const T* par, const T* cov, int64_t ld, int64_t b0, unsigned i, U p[6],
                                  C P[21])
{
    const int64_t row = opaque(ld);
    const T* q = par + b0;
#pragma unroll
    for (int k = 0; k < 6; ++k, q += row) p[k] = U(q[i]);
    q = cov + b0;
#pragma unroll
    for (int k = 0; k < 21; ++k, q += row) P[k] = C(q[i]);
}

template <typename T, typename C, typename U>
__device__ inline void store_state(T* par, T* cov, int64_t ld, int64_t b0, unsigned i, const U p[6],
                                   const C P[21])
{
    const int64_t row = opaque(ld);
    T* q = par + b0;
#pragma unroll
    for (int k = 0; k < 6; ++k, q += row) q[i] = T(p[k]);
    q = cov + b0;
#pragma unroll
    for (int k = 0; k < 21; ++k, q += row) q[i] = T(P[k]);
}

// A layer as propagate_to reads it.
template <typename T>
struct StepLayer {
    int32_t kind;
    T r_or_z, x0;
};

template <typename T>
__device__ inline StepLayer<T> step_layer(const kf_layer& L)
{
    return StepLayer<T>{L.kind, T(L.r_or_z), T(L.x0)};
}

// Propagate (p, P) to layer L.  The surface solve, the helix and the
// transport Jacobian run in T on the state rounded to T; the state itself
// stays in U (transport adds the T increments in U) and the covariance in C.
// s_init < 0: straight-line start; otherwise the learned start with
// prm.mlp_max_iter evaluations before the fallback to the straight-line
// start (counted in *fallbacks).
// FIELD: the parametrised field (kf_params.field_z0 > 0); MAT: the r-z material
// map.  Both are compile-time variants so that the uniform-field, per-layer
// material instantiation keeps its register budget.  finite: see transport.
template <typename T, typename C, typename U, bool FIELD, bool MAT>
__device__ inline int propagate_to(U p[6], C P[21], const StepLayer<T>& L, const kf_params& prm,
                                   bool material, const MatMap& mat, bool finite, T s_init, T* s_out,
                                   int* evals, int* fallbacks)
{
    const T kb = T(kKappa) * T(prm.bz);
    T pt[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) pt[k] = T(p[k]);
    T s;
    if constexpr (FIELD) {
        // parametrised field: Runge-Kutta transport to the barrel's radius or
        // the disk's z; the covariance is carried by the helix Jacobian in the
        // path's mean effective axial field
        const T sth = Tr<T>::sin_(pt[5]);
        T l;
        T q[6];
        int st;
        if (L.kind != 0) {
            st = solve_disk_field(pt, T(L.r_or_z), prm, &l, q, evals);
        } else {
            T bx, by, bz0;
            field_at(T(prm.bz), T(prm.field_z0), pt[0], pt[1], pt[2], &bx, &by, &bz0);
            const T kb0 = T(kKappa) * bz0;
            st = solve_barrel_field(pt, T(L.r_or_z), prm, kb0, s_init >= T(0) ? s_init / sth : T(-1),
                                    prm.mlp_max_iter, &l, q, evals, fallbacks);
        }
        if (st) return st;
        field_transport(p, P, q, l, prm, L.kind, T(L.r_or_z), finite);
        if (material) {
            if constexpr (MAT)
                add_material(p, P, L, mat, T(prm.mass));
            else
                add_scatter(p, P, L.kind, T(L.x0), T(prm.mass));
        }
        if (s_out) *s_out = l * sth;
        bool fin = true;
#pragma unroll
        for (int k = 0; k < 6; ++k) fin &= isfinite(p[k]);
        return fin ? 0 : KF_ST_NAN;
    }
    T st_, ct_;
    Tr<T>::sincos_(pt[5], &st_, &ct_);
    if (L.kind == 0) {
        const T h = -kb * pt[3];
        T sph, cph;
        Tr<T>::sincos_(pt[4], &sph, &cph);
        int st = reach_barrel(pt, h, cph, sph, T(L.r_or_z), prm, s_init, prm.mlp_max_iter, &s, evals,
                              fallbacks);
        if (st) return st;
    } else {
        if (ct_ == T(0)) return KF_ST_UNREACHABLE;
        s = (T(L.r_or_z) - pt[2]) * st_ / ct_;
        *evals += 1;
        if (s < T(0)) return KF_ST_UNREACHABLE;
    }
    transport(p, P, s, kb, L.kind, T(L.r_or_z), st_, ct_, finite);
    if (material) {
        if constexpr (MAT)
            add_material(p, P, L, mat, T(prm.mass));
        else
            add_scatter(p, P, L.kind, T(L.x0), T(prm.mass), st_, ct_);
    }
    if (s_out) *s_out = s;
    bool fin = true;
#pragma unroll
    for (int k = 0; k < 6; ++k) fin &= isfinite(p[k]);
    return fin ? 0 : KF_ST_NAN;
}

// ---------------------------------------------------------------- fit
struct FitArgs {
    int64_t n, ld;
    void* par;
    void* cov;
    void* chi2;
    int32_t* ndf;
    uint32_t* status;
    const float *hx, *hy, *hz, *hsu, *hsv;
    const int32_t* layer_seq;
    const int32_t* hit_idx;
    int64_t n_hits;
    const kf_layer* layers;
    int n_layers;
    kf_params prm;
    int material;
    MatMap mat;                  // r-z material map (x0 == nullptr: none)
    MlpDev mlp;                  // learned guess (KF_INIT_MLP)
    bool index_ahead;            // FP32: load a step's indices in the step before
};

constexpr int kFitThreads = 256;
static_assert(kMaxLayers <= kFitThreads, "a workgroup's LDS holds every layer");

// What a step reads besides the state: its layer and hit index, and the hit.
struct FitIndex {
    int32_t l, hi;
};
struct FitHit {
    float x, y, z, su, sv;
};

// What the fit kernel is built for: several steps, one (k0), or either.
enum { kManySteps, kOneStep, kAnySteps };

// Steps [k0, k1) of the fit.  init: start a fresh fit (chi2 = 0, ndf = -5).
// LEARN: every lane of the wave walks all steps (finished lanes idle), so
// that the network call at each step is in uniform control flow.
//
// Loads: a step's layer and hit indices come in the step before, its hit at its
// start, to be waited for at the update.  A hit a step earlier still gained
// nothing where hits come in order (4,000,000 mixed fits 1506 us, now 1485) and
// cost where they come in any order and the memory is the limit (80,000 mixed
// fits 98 and 90), except among the Runge-Kutta steps of the field (300,000
// mixed fits 832 us with it, 870 without).  FP32 fits, with the least
// arithmetic, do not read the indices ahead either where two or three
// workgroups share a compute unit and all are resident (with and without, hits
// in any order: 50,000 tracks 52 us and 55, 80,000 89 and 84, 130,000 128 and
// 123, 196,608 199 and 198; in order: 100,000 58 and 59, 1,000,000 326 and 336).
//
// The layers wait in LDS.  A launch of one step reads the one layer that each
// lane needs instead: all of them, staged behind a barrier before the first
// load, were what a small fit by layers waited for.  Loads return in order, so
// the hit's come last.  Mixed fits, whose state is rounded between launches
// anyway, have a kernel for one step and one for several; the same kernel serves
// both where one launch and one a layer give the same bits (two copies are
// fused differently by the compiler).  Fits by layers with all layers staged and
// now: 2000 tracks in FP32 72 and 69 us, in 64 bits 110 and 87; 50,000 in 64
// bits 173 and 113; 200,000 mixed 331 and 322, in 64 bits 540 and 394.
//
// WAVES: waves on a SIMD that the registers have to leave room for.
template <typename T, typename C, typename U, bool LEARN, bool FIELD, bool MAT, int STEPS, int WAVES>
__global__ __launch_bounds__(kFitThreads, WAVES) void fit_kernel(FitArgs a, int k0, int k1, int init)
{
    __shared__ StepLayer<T> sl[STEPS == kOneStep ? 1 : STEPS == kAnySteps ? kFitThreads : kMaxLayers];
    if constexpr (STEPS == kOneStep) k1 = k0 + 1;
    const bool one = STEPS == kAnySteps ? k1 - k0 == 1 : STEPS == kOneStep;
    if (!one) {
        for (int l = threadIdx.x; l < a.n_layers; l += blockDim.x) sl[l] = step_layer<T>(a.layers[l]);
        __syncthreads();
    }
    const int64_t b0 = (int64_t)blockIdx.x * blockDim.x;
    const unsigned i = threadIdx.x;
    if (!LEARN && b0 + i >= a.n) return;
    const bool inb = b0 + i < a.n;
    const int64_t ld = a.ld;
    T* par = (T*)a.par;
    T* cov = (T*)a.cov;
    T* chi2p = (T*)a.chi2 + b0;
    uint32_t* stp = a.status + b0;
    int32_t* ndfp = a.ndf + b0;
    uint32_t st = (init || !inb) ? 0u : stp[i];
    int32_t ndf = (init || !inb) ? -5 : ndfp[i];
    U chi2 = (init || !inb) ? U(0) : U(chi2p[i]);
    bool alive = inb && !(st & kFreezeMask);
    if (!LEARN && !alive) return;
    const bool was_alive = alive;
    auto load_index = [&](int k) {
        FitIndex x{-1, -1};
        if (alive && k < k1) {
            x.l = a.layer_seq ? (a.layer_seq + (k * ld + b0))[i] : k;
            x.hi = (a.hit_idx + (k * ld + b0))[i];
        }
        return x;
    };
    auto load_hit = [&](const FitIndex& x) {
        FitHit h{};
        if (x.l >= 0 && x.hi >= 0 && x.hi < a.n_hits) {
            h.x = a.hx[x.hi];
            h.y = a.hy[x.hi];
            h.z = a.hz[x.hi];
            h.su = a.hsu[x.hi];
            h.sv = a.hsv[x.hi];
        }
        return h;
    };
    constexpr bool kHitAhead = STEPS == kOneStep || (STEPS == kManySteps && FIELD);
    const bool index_ahead = sizeof(U) == 8 || a.index_ahead;
    FitIndex now = load_index(k0), next{-1, -1};
    if (kHitAhead) next = load_index(k0 + 1);
    StepLayer<T> own{};
    if (one && now.l >= 0 && now.l < a.n_layers) own = step_layer<T>(a.layers[now.l]);
    // the state stays in U between steps (rounded to T only when stored)
    U p[6];
    C P[21];
    if (alive) load_state(par, cov, ld, b0, i, p, P);
    if constexpr (STEPS == kAnySteps) {
        if (one) sl[i] = own;
    }
    FitHit hit{};
    if (kHitAhead) hit = load_hit(now);
    const bool finite = wave_all(!alive || all_finite(P));
    bool touched = false;
    for (int k = k0; k < k1; ++k) {
        if (!LEARN && !alive) break;
        if (!kHitAhead) {
            if (!index_ahead && k > k0) now = load_index(k);
            hit = load_hit(now);
        }
        const int32_t l = now.l, hi = now.hi;
        FitHit h = hit;
        if (kHitAhead) {
            now = next;
            hit = load_hit(next);
            next = load_index(k + 2);
        } else if (index_ahead) {
            now = load_index(k + 1);
        }
        if (alive) {
            if (l < 0) {
                alive = false;
            } else if (l >= a.n_layers) {
                st |= KF_ST_BADINPUT;
                alive = false;
            }
        }
        StepLayer<T> L{};
        if (alive) L = STEPS == kOneStep ? own : sl[one ? i : (unsigned)l];
        T s_init = T(-1);
        if (LEARN) {
            float f[kMlpIn] = {0, 0, 0, 0, 0, 0, 0, 0};
            const bool want = alive && L.kind == 0;
            if (want) {
                T pt[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) pt[q] = T(p[q]);
                mlp_features(pt, L, a.prm, f);
            }
            const uint64_t wmask = __ballot(want);
            const float y = wmask ? mlp_wave(a.mlp, f, wmask) : 0.0f;
            if (want) s_init = T(mlp_guess(f, y));
        }
        if (!alive) continue;
        int ev = 0, fb = 0;
        int r = propagate_to<T, C, U, FIELD, MAT>(p, P, L, a.prm, a.material != 0, a.mat, finite,
                                                   s_init, (T*)nullptr, &ev, &fb);
        touched = true;
        if (fb) st |= KF_ST_FALLBACK;
        if (r) {
            st |= (uint32_t)r;
            alive = false;
            continue;
        }
        if (hi >= a.n_hits) {
            st |= KF_ST_BADINPUT;
            alive = false;
            continue;
        }
        if (hi >= 0) {
            // (keeps the conversions, and with them the wait, from moving up to the loads)
            asm volatile("" : "+v"(h.x), "+v"(h.y), "+v"(h.z), "+v"(h.su), "+v"(h.sv));
            HitFrame<U> f = hit_frame<U>(h.x, h.y, h.z, h.su, h.sv);
            U c2 = U(0);
            r = kf_update<U, C, U>(p, P, f, L.kind, &c2);
            if (r) {
                st |= (uint32_t)r;
                alive = false;
                continue;
            }
            // rounded to storage precision every step, so one launch per step
            // and one launch for all steps give identical results
            chi2 = U(T(chi2 + c2));
            ndf += 2;
        }
    }
    if (!was_alive) return;
    // on failure the registers hold the last good state (a failed solve or
    // update leaves them untouched)
    if (touched) store_state(par, cov, ld, b0, i, p, P);
    chi2p[i] = T(chi2);
    ndfp[i] = ndf;
    stp[i] = st;
}

template <typename T, typename C, typename U, bool LEARN, int STEPS, int WAVES>
inline void fit_launch(const FitArgs& a, dim3 g, int k0, int k1, int init, bool field, bool map,
                       hipStream_t s)
{
    if (field) {
        if (map) fit_kernel<T, C, U, LEARN, true, true, STEPS, WAVES><<<g, kFitThreads, 0, s>>>(a, k0, k1, init);
        else fit_kernel<T, C, U, LEARN, true, false, STEPS, WAVES><<<g, kFitThreads, 0, s>>>(a, k0, k1, init);
    } else {
        if (map) fit_kernel<T, C, U, LEARN, false, true, STEPS, WAVES><<<g, kFitThreads, 0, s>>>(a, k0, k1, init);
        else fit_kernel<T, C, U, LEARN, false, false, STEPS, WAVES><<<g, kFitThreads, 0, s>>>(a, k0, k1, init);
    }
}

// Fits in 64 bits of more tracks than one wave a SIMD holds (kf_fit64.hip).
void launch_fit64(const FitArgs& a, dim3 g, int k0, int k1, int init, bool learn, bool field, bool map,
                  hipStream_t s);

}  // namespace kfmi
