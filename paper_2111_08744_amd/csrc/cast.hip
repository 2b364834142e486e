// cast.hip -- forward ray-casting kernels for gfx950.
//
// One lane integrates one photon (Sect. 2.2: photons are independent), or four
// lanes do where the rays are few (QuadRay).  Two schedules share the per-ray
// code:
//   static      one launch with one lane per ray (or four); rays of a wave are
//               neighbouring NESTED pixels of one observer, so their
//               stencil gathers hit the same cache lines near the observer;
//   persistent  a grid sized to the resident capacity of the GPU; every lane
//               that finishes its ray takes the next one from a global
//               queue (one atomic per wave per refill, ballot-aggregated), so
//               rays of uneven length (many observers, many source
//               redshifts, AMR) do not leave lanes idle.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device.h"

namespace mpath {
namespace {

constexpr int kWave = 64;
// Occupancy target of the integration kernels: 4 waves per SIMD (128
// registers).  A wave stalls on every stage where one of its lanes enters a
// new stencil, so latency hiding pays more than the few values the bound
// spills (measured on the AMR workload with an earlier form of the field
// cache: 3 waves 102.6 ms, 4 waves 89.5 ms per cast).
constexpr int kMinWavesPerSimd = 4;

// Step-start hook of RayRun::advance that does nothing (plain casts).
struct NoSample {
    template <class FC>
    __device__ __forceinline__ void at_step(const CastArgs&, const RayGeom&, const GeoState&, int, const FC&) {}
    template <class Run>
    __device__ __forceinline__ bool at_surface(const CastArgs&, Run&) { return false; }
};

// Everything one lane carries for its current ray (DP: the form of dPhi/dl).
template <bool AMR, class FC = FieldCache<AMR>, class DP = ChainRule>
struct RayRun {
    static constexpr int C = FC::kComp;   // components of geo, y and the gradient that this lane holds
    int64_t ray;          // -1: no ray
    RayGeom geo;
    double eta_s;
    float phi_o;
    GeoState y;
    int32_t n_steps;
    uint32_t hash;
    int status;           // -1 while running
    double isw;           // int dPhi/deta |d eta| so far (time-dependent potential; else 0)
    double lam;           // affine parameter (iso-lambda stops)
    double p_cur, dp_cur; // stop parameter and its lambda-derivative at y (iso-chi, iso-z stops)
    DP dp;
    FC F;

    template <bool CKPT = false>
    __device__ __forceinline__ bool advance(const CastArgs& a, int max_iter)
    {
        NoSample none;
        return advance<CKPT, NoSample>(a, max_iter, none);
    }

    __device__ __forceinline__ void start(const CastArgs& a, int64_t r)
    {
        ray = r;
        // observer owning the ray (observers are few; linear scan from the end)
        int j = a.n_obs - 1;
        while (j > 0 && a.obs[j].ray_first > r) --j;
        const ObsDev& ob = a.obs[j];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            geo.vo[i] = ldexp(ob.x[FC::own_axis(i)] / a.grid.h0, a.grid.max_level + 1);
            geo.n[i] = a.dirs[3 * r + FC::own_axis(i)];
        }
        eta_s = a.ray_stop ? a.ray_stop[r].x : ob.eta_s;
        F.reset();
        n_steps = 0;
        hash = kFnvOffset;
        status = -1;
        isw = 0.0;
        if constexpr (DP::kDiff) dp.dl_prev = 0.0;
        float G[C];
        int leafl, l;
        phi_o = __builtin_nanf("");
        if (F.eval(a.grid, geo.vo, G, leafl, l)) status = MPATH_RAY_LEFT_DOMAIN;
        else phi_o = F.phi(a.grid);
        // k0 = -1 (backward in time); |k| from the null condition
        const double po = (double)phi_o;
        const double kmag = sqrt((1.0 + 2.0 * po) / (1.0 - 2.0 * po));
        y.eta = a.cosmo_eta0;
        y.K = 1.0;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            y.d[i] = (float)(geo.n[i] * (kmag - 1.0));
            y.dx[i] = 0.0f;
        }
    }

    // Advance by at most max_iter steps; returns true when the ray is done.
    // With CKPT the state before every K-th step is stored for the adjoint.
    // smp.at_step(y, L, F) sees the state at every step start (after the leaf
    // level L there is known and F evaluated there, before the step is taken).
    template <bool CKPT = false, class Smp = NoSample>
    __device__ __forceinline__ bool advance(const CastArgs& a, int max_iter, Smp& smp)
    {
        if (status >= 0) return true;
        const GridDev& g = a.grid;
        const int max_steps = (int)a.max_steps;     // at most 2^31 - 1
        int it = 0;
        for (;;) {
            // the field at the step start (stage 0 of the step, and of every
            // landing pass, which all start there)
            Stage0 s0;
            // regular steps up to the one that would cross the stop surface
            for (;; ++it) {
                if (it >= max_iter) return false;
                if (n_steps >= max_steps) { status = MPATH_RAY_MAX_STEPS; return true; }
                if (CKPT && n_steps % a.ckpt_every == 0) {
                    GeoState& k = a.ckpt[(n_steps / a.ckpt_every) * a.n_rays + ray];
                    k.eta = y.eta;
                    k.K = y.K;
                    FC::whole_vector(y.dx, k.dx);
                    FC::whole_vector(y.d, k.d);
                }
                // leaf level at the step start sets the step length (N steps
                // per cell); the same evaluation gives stage 0's field
                double v[C];
                grid_coords<C>(g, geo, y.eta, y.dx, v);
                int L;
                s0.bad = F.eval(g, v, s0.G, L, s0.l);
                if constexpr (DP::kDiff) s0.phi = F.phi(g);
                if constexpr (FC::kTime) s0.tv = F.tv;
                if (L < 0) { status = MPATH_RAY_LEFT_DOMAIN; return true; }
                hash = fnv(hash, (uint32_t)L);
                smp.at_step(a, geo, y, L, F);
                const double dl = quotient(step_length(a, L), y.K);
                if (fma(-y.K, dl, y.eta) < eta_s) break;
                GeoState yn;
                if (rk4_step_dp<FC, DP, true>(g, a.cosmo, F, geo, y, dl, yn, hash, dp, &s0)) {
                    status = MPATH_RAY_LEFT_DOMAIN;
                    return true;
                }
                if constexpr (FC::kTime) isw += (double)F.isw_step;
                if (!finite_state<FC>(yn)) { status = MPATH_RAY_NONFINITE; return true; }
                y = yn;
                ++n_steps;
                if constexpr (DP::kDiff) {
                    dp.phi_prev = dp.phi0;
                    dp.dl_prev = dl;
                }
            }
            ++it;
            // landing on the iso-eta surface: Newton on eta_RK4(dl) = eta_s
            // with derivative -K at the trial end, two iterations, then the step
            double dlx = (y.eta - eta_s) / y.K;
            GeoState yn;
#pragma unroll 1
            for (int k = 0; k < 3; ++k) {
                if (rk4_step_dp<FC, DP, false>(g, a.cosmo, F, geo, y, dlx, yn, hash, dp, &s0)) {
                    status = MPATH_RAY_LEFT_DOMAIN;
                    return true;
                }
                if (k < 2) dlx = dlx + (yn.eta - eta_s) / yn.K;
            }
            const bool fin = finite_state<FC>(yn);
            if constexpr (FC::kTime) isw += (double)F.isw_step;
            y = yn;
            ++n_steps;
            if constexpr (!std::is_same<Smp, NoSample>::value)
                if (fin && smp.at_surface(a, *this)) continue;   // on to the next stop surface
            status = fin ? MPATH_RAY_REACHED : MPATH_RAY_NONFINITE;
            return true;
        }
    }

    // Stop parameter of state s and its lambda-derivative (iso-chi: the
    // comoving distance r from the observer, d/dl = K r.m / r; iso-z:
    // ln(1 + z5) with z5 of the end-point formula at s, d/dl =
    // K (a'/a - m.G), the first-order rate of a K (1 + Phi)).  Returns false
    // when the field has no stencil there.
    template <int SURF>
    __device__ __forceinline__ bool stop_param(const CastArgs& a, const GeoState& s, double& p, double& dp)
    {
        const double sp = a.grid.eta0 - s.eta;
        double r[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) r[i] = fma(sp, geo.n[i], (double)s.dx[i]);
        if constexpr (SURF == MPATH_SURFACE_CHI) {
            const double rr = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
            double rm = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) rm += r[i] * (geo.n[i] + (double)s.d[i]);
            p = rr;
            dp = s.K * rm / rr;
            return true;
        } else {
            double v[3];
            grid_coords(a.grid, geo, s.eta, s.dx, v);
            float G[3];
            int leafl, l;
            if (F.eval(a.grid, v, G, leafl, l)) return false;
            const float phi = F.phi(a.grid);
            const double sa = scale_factor(a.cosmo, s.eta);
            p = log(sa * s.K * (1.0 + (double)phi) / (1.0 + (double)phi_o));
            HubbleCubic Hc;
            Hc.init(a.cosmo, s.eta);
            double mG = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) mG += (geo.n[i] + (double)s.d[i]) * (double)G[i];
            dp = s.K * (Hc(a.cosmo, s.eta) - mG);
            return true;
        }
    }

    // The integration to an iso-chi, iso-lambda or iso-z surface (SURF): the
    // regular steps of advance; the step that reaches the surface is taken
    // again from its start with the length from two Newton iterations on
    // p(RK4(dl)) - p_s (iso-lambda: the remaining length exactly).
    template <int SURF>
    __device__ __forceinline__ void advance_stop(const CastArgs& a, double p_s)
    {
        if (status >= 0) return;
        const GridDev& g = a.grid;
        lam = 0.0;
        if constexpr (SURF == MPATH_SURFACE_CHI) {
            // at the observer: chi = 0, rising at |k| = K |n + d|
            p_cur = 0.0;
            dp_cur = 1.0 + (geo.n[0] * y.d[0] + geo.n[1] * y.d[1] + geo.n[2] * y.d[2]);
        }
        for (;;) {
            if (n_steps >= a.max_steps) { status = MPATH_RAY_MAX_STEPS; return; }
            double v[3];
            grid_coords(g, geo, y.eta, y.dx, v);
            const int L = F.leaf(g, v);
            if (L < 0) { status = MPATH_RAY_LEFT_DOMAIN; return; }
            hash = fnv(hash, (uint32_t)L);
            const double dl = quotient(step_length(a, L), y.K);
            GeoState yn;
            if constexpr (SURF == MPATH_SURFACE_LAMBDA) {
                if (lam + dl >= p_s) {
                    const double dlx = p_s - lam;
                    if (rk4_step<FC>(g, a.cosmo, F, geo, y, dlx, yn, hash)) { status = MPATH_RAY_LEFT_DOMAIN; return; }
                    y = yn;
                    lam += dlx;
                    ++n_steps;
                    status = finite_state(y) ? MPATH_RAY_REACHED : MPATH_RAY_NONFINITE;
                    return;
                }
            }
            if (rk4_step<FC>(g, a.cosmo, F, geo, y, dl, yn, hash)) { status = MPATH_RAY_LEFT_DOMAIN; return; }
            if (!finite_state(yn)) { status = MPATH_RAY_NONFINITE; return; }
            if constexpr (SURF != MPATH_SURFACE_LAMBDA) {
                bool check = true;
                if constexpr (SURF == MPATH_SURFACE_Z) {
                    // interpolation weights are convex, so Phi <= phi_max anywhere (up
                    // to float32 rounding) and 1 + z5 <= a K (1 + phi_max) / (1 + Phi_o):
                    // below 1 + z_s (with a relative margin of 1e-9) the surface is not
                    // reached and the field need not be evaluated
                    const double bound = scale_factor(a.cosmo, yn.eta) * yn.K * (1.0 + (double)g.phi_max) /
                                         (1.0 + (double)phi_o);
                    check = bound >= exp(p_s) * (1.0 - 1e-9);
                }
                double pn = 0.0, dpn = 0.0;
                if (check && !stop_param<SURF>(a, yn, pn, dpn)) { status = MPATH_RAY_LEFT_DOMAIN; return; }
                if (check && pn >= p_s) {
                    if constexpr (SURF == MPATH_SURFACE_Z) {
                        // the parameter and its rate at the step start (the previous
                        // step's end), skipped while far from the surface
                        if (!stop_param<SURF>(a, y, p_cur, dp_cur)) { status = MPATH_RAY_LEFT_DOMAIN; return; }
                    }
                    // two Newton passes, then the step
                    double dlx = (p_s - p_cur) / dp_cur;
#pragma unroll 1
                    for (int it = 0; it < 3; ++it) {
                        if (rk4_step<FC>(g, a.cosmo, F, geo, y, dlx, yn, hash)) { status = MPATH_RAY_LEFT_DOMAIN; return; }
                        if (it < 2) {
                            double pt, dpt;
                            if (!stop_param<SURF>(a, yn, pt, dpt)) { status = MPATH_RAY_LEFT_DOMAIN; return; }
                            dlx = dlx - (pt - p_s) / dpt;
                        }
                    }
                    y = yn;
                    lam += dlx;
                    ++n_steps;
                    status = finite_state(y) ? MPATH_RAY_REACHED : MPATH_RAY_NONFINITE;
                    return;
                }
                if constexpr (SURF == MPATH_SURFACE_CHI) {
                    p_cur = pn;
                    dp_cur = dpn;
                }
            }
            y = yn;
            lam += dl;
            ++n_steps;
        }
    }

    // advance() for a plain cast (iso-eta stop, chain rule, static
    // potential) with a stage recorder T that also sees every step's start
    // and end: T.begin_step(y, dl, regular) before the RK4 pass it records
    // (every regular step; of the landing only the final pass) and
    // T.end_step(y, yn) after it.  The steps, their decisions and the
    // primal arithmetic are those of advance(), bit for bit.
    template <class Tan>
    __device__ __forceinline__ void advance_recorded(const CastArgs& a, Tan& T)
    {
        if (status >= 0) return;
        const GridDev& g = a.grid;
        ChainRule cr;
        constexpr bool kUnrolled = C == 1;
        for (;;) {
            if (n_steps >= a.max_steps) { status = MPATH_RAY_MAX_STEPS; return; }
            double v[C];
            grid_coords<C>(g, geo, y.eta, y.dx, v);
            int L;
            Stage0 s0;                 // the field at the step start: stage 0
            s0.bad = F.eval(g, v, s0.G, L, s0.l);
            if (L < 0) { status = MPATH_RAY_LEFT_DOMAIN; return; }
            hash = fnv(hash, (uint32_t)L);
            const double dl = quotient(step_length(a, L), y.K);
            if (fma(-y.K, dl, y.eta) < eta_s) break;
            GeoState yn;
            T.begin_step(y, dl, true);
            if (rk4_core<FC, Tan, ChainRule, kUnrolled>(g, a.cosmo, F, geo, y, dl, yn, hash, T, true, cr, &s0)) {
                status = MPATH_RAY_LEFT_DOMAIN;
                return;
            }
            if (!finite_state<FC>(yn)) { status = MPATH_RAY_NONFINITE; return; }
            T.end_step(y, yn);
            y = yn;
            ++n_steps;
        }
        // landing on the iso-eta surface (as advance())
        double dlx = (y.eta - eta_s) / y.K;
        GeoState yn;
        for (int k = 0; k < 3; ++k) {
            if (k == 2) T.begin_step(y, dlx, false);
            if (rk4_core<FC, Tan, ChainRule, false>(g, a.cosmo, F, geo, y, dlx, yn, hash, T, k == 2, cr)) {
                status = MPATH_RAY_LEFT_DOMAIN;
                return;
            }
            if (k < 2) dlx = dlx + (yn.eta - eta_s) / yn.K;
        }
        const bool fin = finite_state<FC>(yn);
        T.end_step(y, yn);
        y = yn;
        ++n_steps;
        status = fin ? MPATH_RAY_REACHED : MPATH_RAY_NONFINITE;
    }

    // Outputs at the end of advance_stop: the end point's own scale factor.
    __device__ __forceinline__ void finish_stop(const CastArgs& a)
    {
        int j = a.n_obs - 1;
        while (j > 0 && a.obs[j].ray_first > ray) --j;
        const double ae = scale_factor(a.cosmo, y.eta);
        write_outputs(a, ray, j, ae, 1.0 / ae - 1.0, status);
    }

    // Redshift observables (Sect. 2.5) and the end state; the angular
    // observables follow in observables_kernel, which keeps the FP64
    // transcendental functions out of the integration kernel's registers.
    __device__ __forceinline__ void finish(const CastArgs& a)
    {
        int j = a.n_obs - 1;
        while (j > 0 && a.obs[j].ray_first > ray) --j;
        const ObsDev& ob = a.obs[j];
        const double a_s = a.ray_stop ? a.ray_stop[ray].y : ob.a_s;
        write_outputs(a, ray, j, a_s, a.ray_stop ? 1.0 / a_s - 1.0 : ob.z0, status);
    }

    // Outputs of the current state at output slot `slot` (observer j, stop
    // surface with scale factor a_s and FLRW redshift z0) with ray status st
    // (MPATH_RAY_REACHED: the ray is on that surface).
    __device__ __forceinline__ void write_outputs(const CastArgs& a, int64_t slot, int j, double a_s, double z0,
                                                  int st)
    {
        const bool ok = st == MPATH_RAY_REACHED;
        double v[C];
        grid_coords<C>(a.grid, geo, y.eta, y.dx, v);
        float phi_s = __builtin_nanf(""), G[C];
        int leafl, l;
        if (!F.eval(a.grid, v, G, leafl, l)) phi_s = F.phi(a.grid);
        const OutDev& o = a.out;
        if (o.z5)
            o.z5[slot] = ok ? a_s * y.K * (1.0 + (double)phi_s) / (1.0 + (double)phi_o) - 1.0 : __builtin_nan("");
        if (o.z0) o.z0[slot] = ok ? z0 : __builtin_nan("");
        const double z1 = z0 + (1.0 + z0) * ((double)phi_o - (double)phi_s);
        if (o.z1) o.z1[slot] = ok ? z1 : __builtin_nan("");
        // z4 = z1 - 2 (a0 / a_s) int_{eta_s}^{eta_0} dPhi/deta d eta (Sect. 2.5, v = 0)
        if (o.z4) o.z4[slot] = ok ? z1 - 2.0 * (1.0 + z0) * isw : __builtin_nan("");
        if (o.isw) o.isw[slot] = ok ? isw : __builtin_nan("");
        if (o.phi_src) o.phi_src[slot] = phi_s;
        if (o.n_steps) o.n_steps[slot] = (int32_t)n_steps;
        if (o.status) o.status[slot] = st;
        if (o.hash) o.hash[slot] = hash;
        RayEnd e;
        e.eta = y.eta;
        FC::whole_vector(y.dx, e.dx);
        e.obs = j;
        a.ends[slot] = e;
    }
};

// Initial directions: HEALPix NESTED pixel centres (Sect. 2.4), computed once
// per cast so that the integration kernel does not carry the FP64 sincos.
__global__ __launch_bounds__(256) void ray_dirs_kernel(CastArgs a)
{
    const int64_t ray = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (ray >= a.n_rays) return;
    int j = a.n_obs - 1;
    while (j > 0 && a.obs[j].ray_first > ray) --j;
    const ObsDev& ob = a.obs[j];
    double n[3];
    healpix_nest_dir(a.nside, ob.pix_first + (ray - ob.ray_first), n);
    a.dirs[3 * ray] = n[0];
    a.dirs[3 * ray + 1] = n[1];
    a.dirs[3 * ray + 2] = n[2];
}

// Lens equation (Sect. 2.3): beta from the end point r = x_s - x_obs, and the
// deflection alpha = theta - beta as the tangent vector at theta pointing
// away from beta with the great-circle angle as length, on e1 = e_phi,
// e2 = -e_theta.
__global__ __launch_bounds__(256) void observables_kernel(CastArgs a)
{
    const int64_t ray = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (ray >= a.n_rays) return;
    const RayEnd e = a.ends[ray];
    const double n[3] = {a.dirs[3 * ray], a.dirs[3 * ray + 1], a.dirs[3 * ray + 2]};
    const double s = a.cosmo_eta0 - e.eta;
    double r[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) r[i] = s * n[i] + (double)e.dx[i];
    const double chi = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    const OutDev& o = a.out;
    if (o.chi) o.chi[ray] = chi;
    if (o.beta) {
        o.beta[2 * ray] = atan2(hypot(r[0], r[1]), r[2]);
        o.beta[2 * ray + 1] = atan2(r[1], r[0]);
    }
    if (o.alpha) {
        const double rh[3] = {r[0] / chi, r[1] / chi, r[2] / chi};
        const double c = rh[0] * n[0] + rh[1] * n[1] + rh[2] * n[2];
        double t[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) t[i] = rh[i] - c * n[i];
        const double st2 = t[0] * t[0] + t[1] * t[1] + t[2] * t[2];
        double fac = 0.0;
        if (st2 > 0.0) {
            const double st = sqrt(st2);
            fac = -atan2(st, c) / st;
        }
        const double ph = atan2(n[1], n[0]);
        const double th = atan2(hypot(n[0], n[1]), n[2]);
        double sp, cp, stt, ctt;
        sincos(ph, &sp, &cp);
        sincos(th, &stt, &ctt);
        const double e1[3] = {-sp, cp, 0.0};
        const double e2[3] = {-cp * ctt, -sp * ctt, stt};
        o.alpha[2 * ray] = (float)(fac * (t[0] * e1[0] + t[1] * e1[1] + t[2] * e1[2]));
        o.alpha[2 * ray + 1] = (float)(fac * (t[0] * e2[0] + t[1] * e2[1] + t[2] * e2[2]));
    }
}

// TIME: the grid carries dPhi/deta (time-dependent potential).
template <bool AMR, bool TIME>
__global__ __launch_bounds__(kBlock, kMinWavesPerSimd) void cast_static_kernel(CastArgs a)
{
    extern __shared__ float coef_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    RayRun<AMR, FieldCache<AMR, TIME>> R;
    R.F.bind(coef_lds);
    R.start(a, r);
    R.advance(a, 0x7fffffff);
    R.finish(a);
}

// Four lanes per ray (QuadRay), with CKPT checkpoints for the adjoint: for
// casts that leave a SIMD no more than a wave or a few, where the length of a
// step's instruction sequence decides and not the number of waves.  A step
// takes about 390 vector instructions against 582 (uniform grid).
template <bool AMR, bool CKPT>
__global__ __launch_bounds__(kBlock, kMinWavesPerSimd) void cast_quad_kernel(CastArgs a)
{
    int64_t r;
    if (!lane_ray<4>(a, a.n_rays, r)) return;
    RayRun<AMR, QuadCache<AMR>> R;
    R.start(a, r);
    R.template advance<CKPT>(a, 0x7fffffff);
    R.finish(a);
}

// Static schedule storing checkpoints for the adjoint.
template <bool AMR>
__global__ __launch_bounds__(kBlock, kMinWavesPerSimd) void cast_ckpt_kernel(CastArgs a)
{
    extern __shared__ float coef_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    RayRun<AMR> R;
    R.F.bind(coef_lds);
    R.start(a, r);
    R.template advance<true>(a, 0x7fffffff);
    R.finish(a);
}

template <bool AMR, bool TIME>
__global__ __launch_bounds__(kBlock, kMinWavesPerSimd) void cast_persistent_kernel(CastArgs a)
{
    extern __shared__ float coef_lds[];
    const int lane = threadIdx.x & (kWave - 1);
    RayRun<AMR, FieldCache<AMR, TIME>> R;
    R.F.bind(coef_lds);
    R.ray = -1;
    bool exhausted = false;
    for (;;) {
        // refill every lane without a ray (one atomic per wave)
        const bool need = R.ray < 0 && !exhausted;
        const unsigned long long want = __ballot(need);
        if (want) {
            const int cnt = __popcll(want);
            const int leader = __ffsll((long long)want) - 1;
            unsigned long long base = 0;
            if (lane == leader) base = atomicAdd(a.queue, (unsigned long long)cnt);
            base = __shfl(base, leader);
            if (base + (unsigned long long)cnt >= (unsigned long long)a.n_rays) exhausted = true;
            if (need) {
                const unsigned long long mine = base + __popcll(want & ((1ull << lane) - 1ull));
                if (mine < (unsigned long long)a.n_rays) R.start(a, (int64_t)mine);
            }
        }
        if (!__ballot(R.ray >= 0)) break;          // queue drained and every lane idle
        if (R.ray >= 0 && R.advance(a, a.batch)) {
            R.finish(a);
            R.ray = -1;
        }
    }
}

// 1/sqrt(x) for x of moderate size in double precision (the hardware's
// estimate and two Newton steps).
__device__ __forceinline__ double inv_sqrt(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    r = r * fma(-h * r, r, 1.5);
    return r * fma(-h * r, r, 1.5);
}

// Infinitesimal-beam distortion matrix (Sect. 2.3.1): along the path,
//   A_ab = delta_ab - 2 int_0^chi_s (chi_s - chi) chi / chi_s T_ab dchi,
// T_ab = e_a . H e_b with H the Hessian of Phi from centred differences of
// the interpolated gradient, H_ij = (G_j(x + h e_i) - G_j(x - h e_i)) / 2h
// (mixed derivatives symmetrised), h the size of the leaf cell holding x,
// and (e_1, e_2) = (e_phi, -e_theta) at the direction of x - x_obs.  The
// integrand is sampled at every step start and at the end point and
// integrated by the trapezoid rule in chi; with w = chi - chi^2 / chi_s the
// two sums int chi T and int chi^2 T are carried so that chi_s is needed only
// at the end.
//
// On a refined grid the six probes are evaluated through a second stencil
// cache, so that the integration's own is left in place.  On a uniform grid
// x +- h e_i lies at the same offsets in the neighbouring stencils b +- e_i,
// so the six independent entries of H are the trilinear interpolants of the
// differences of the cells' gradients one cell to either side of x's own
// stencil cells: 48 words a lane, formed from 32 cells when x enters a new
// stencil and evaluated with 84 instructions a step, where six probes, each
// almost always in another stencil than the last, were six resolutions and
// gathers: 49,152 rays to z = 1 on a 64^3 grid 23.3 -> 10.9 ms, the Born beam
// 16.2 -> 7.2.  The differences are rounded once, as the probes' were (the mixed
// entries' sums are formed in double precision), and the eight values
// interpolated, whose weights are convex: float32 differences of the records'
// trilinear coefficients (13.0 and 8.0 ms) gave A's mixed entry 1.5 to 1.7 times
// the error (3,072 rays to z = 0.1, against 64 bits: six probes 9.8e-12, the
// coefficients 1.66e-11, this 9.3e-12).
// ALONE: no integration beside it (the Born beam).
template <bool AMR, bool ALONE = false>
struct InfBeam {
    static constexpr int kFloats = AMR ? FieldCache<AMR>::kFloats : 48;   // LDS words per lane
    FieldCache<AMR> P;           // AMR: the probes' stencils
    float4* c;                   // uniform: entry p of H (00, 01, 02, 11, 12, 22) at the stencil's cells 0..3 at
                                 // c[64 2 p] and 4..7 at c[64 (2 p + 1)]
    int base;                    // uniform: the stencil they belong to
    double chi_p, Tp[3], Up[3];  // previous sample: chi T and chi^2 T (T11, T12, T22)
    double J1[3], J2[3];         // trapezoid sums of chi T and chi^2 T
    int n;

    // lds: kFloats * kBlock floats of the block
    __device__ __forceinline__ void init(float* lds)
    {
        if constexpr (AMR) {
            P.bind(lds);
            P.reset();
        } else {
            c = reinterpret_cast<float4*>(lds) + (threadIdx.x >> 6) * (64 * kFloats / 4) + (threadIdx.x & 63);
            base = -1;
        }
        n = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) J1[k] = J2[k] = 0.0;
    }

    // Uniform grid: H (times 2 h; the mixed entries times 4 h) at the 8 cells of
    // F's stencil.  A probe without a complete stencil (the edge of a
    // non-periodic box) leaves a zero row, a point without one a zero H.
    __device__ __forceinline__ void load(const GridDev& g, const FieldCache<AMR>& F)
    {
        bool ok[3] = {true, true, true};
        if (!g.periodic) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                ok[i] = F.leafL >= 0;
                if (ok[i]) {
                    const int b = (int)F.kd[i];
                    ok[i] = b >= 1 && b + 2 < g.n0;
                }
            }
        }
        if (ok[0] && ok[1] && ok[2]) form<false>(g, (uint32_t)F.base, ok);
        else form<true>(g, (uint32_t)F.base, ok);
        base = F.base;
    }

    // The same with (EDGE) or without rows left out.
    template <bool EDGE>
    __device__ __forceinline__ void form(const GridDev& g, uint32_t from, const bool (&ok)[3])
    {
        const uint32_t bits = (1u << (3 * __builtin_ctz((unsigned)g.n0))) - 1u;
        // per axis the interleaved coordinates of the cells -1, 0, 1, 2 (wrapping)
        uint32_t at[3][4];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t lanes = (0x49249249u << i) & bits, m = from & lanes;
            at[i][0] = (m - (1u << i)) & lanes;
            at[i][1] = m;
            at[i][2] = step_up(m, lanes, 1u << i) & lanes;
            at[i][3] = step_up(at[i][2], lanes, 1u << i) & lanes;
        }
        auto cell = [&](int x, int y, int z, float G[3]) {      // its gradient
            const float4 q = g.payload[at[0][x] | at[1][y] | at[2][z]];
            G[0] = q.y; G[1] = q.z; G[2] = q.w;
        };
        auto put = [&](int p, const auto* h) {
            c[64 * 2 * p] = make_float4((float)h[0], (float)h[1], (float)h[2], (float)h[3]);
            c[64 * (2 * p + 1)] = make_float4((float)h[4], (float)h[5], (float)h[6], (float)h[7]);
        };
        // the corners, and the cells beyond them along axis i.  The Born kernel
        // needs the barriers to have the eight in flight together (it waits for
        // each load without them: 8.2 -> 13.7 ms, with them 7.2); in the cast
        // the compiler requests 24 at once, and barriers make it spill 39
        // registers (10.9 -> 15.0 ms).
        float in[8][3], out[8][3];
#pragma unroll
        for (int o = 0; o < 8; ++o) cell(1 + (o & 1), 1 + ((o >> 1) & 1), 1 + (o >> 2), in[o]);
        double X[3][8];                 // the mixed entries 01, 02, 12, rounded once
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                int k[3] = {1 + (o & 1), 1 + ((o >> 1) & 1), 1 + (o >> 2)};
                k[i] = (o >> i) & 1 ? 3 : 0;
                cell(k[0], k[1], k[2], out[o]);
            }
            if constexpr (ALONE) asm volatile("" ::: "memory");
            float D[8];
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                const int up = (o >> i) & 1;
                const float* hi = up ? out[o] : in[o ^ (1 << i)];
                const float* lo = up ? in[o ^ (1 << i)] : out[o];
                D[o] = !EDGE || ok[i] ? hi[i] - lo[i] : 0.0f;
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    if (j == i) continue;
                    const double d = !EDGE || ok[i] ? (double)hi[j] - (double)lo[j] : 0.0;
                    double& x = X[i + j - 1][o];
                    x = i < j ? d : x + d;
                }
            }
            put(i == 0 ? 0 : 2 * i + 1, D);      // 00, 11, 22
            if (i == 1) put(1, X[0]);
        }
        put(2, X[1]);
        put(4, X[2]);
    }

    // Trilinear interpolant of the values a (cells 0..3) and b (4..7).
    static __device__ __forceinline__ float interpolate(const float4 a, const float4 b, const float t[3])
    {
        #pragma clang fp contract(off)
        const float x0 = fmaf(t[0], a.y - a.x, a.x), x1 = fmaf(t[0], a.w - a.z, a.z);
        const float x2 = fmaf(t[0], b.y - b.x, b.x), x3 = fmaf(t[0], b.w - b.z, b.z);
        const float y0 = fmaf(t[1], x1 - x0, x0), y1 = fmaf(t[1], x3 - x2, x2);
        return fmaf(t[2], y1 - y0, y0);
    }

    // The Hessian's entries (00, 01, 02, 11, 12, 22) at the point v, F's last
    // evaluated one, with the derivation step of a leaf of level L.
    __device__ __forceinline__ void hessian(const GridDev& g, const double v[3], int L, const FieldCache<AMR>& F,
                                            double H[6])
    {
        if constexpr (AMR) {
            // h = h0 / 2^L; in fine-grid units 2^(max_level + 1 - L), exact
            const double i2h = 0.5 * ldexp(g.inv_h0, L);
            const double hf = ldexp(1.0, g.max_level + 1 - L);
            double D[3][3];
#pragma unroll 1
            for (int i = 0; i < 3; ++i) {
                double vp[3] = {v[0], v[1], v[2]}, vm[3] = {v[0], v[1], v[2]};
                vp[i] += hf;
                vm[i] -= hf;
                float gp[3], gm[3];
                int l0, l1;
                const bool bad = P.eval(g, vp, gp, l0, l1) != 0 || P.eval(g, vm, gm, l0, l1) != 0;
#pragma unroll
                for (int j = 0; j < 3; ++j) D[i][j] = bad ? 0.0 : ((double)gp[j] - (double)gm[j]) * i2h;
            }
            H[0] = D[0][0]; H[3] = D[1][1]; H[5] = D[2][2];
            H[1] = 0.5 * (D[0][1] + D[1][0]);
            H[2] = 0.5 * (D[0][2] + D[2][0]);
            H[4] = 0.5 * (D[1][2] + D[2][1]);
        } else {
            if (F.base != base) load(g, F);
            const double i2h = 0.5 * g.inv_h0;
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                const float f = interpolate(c[64 * 2 * p], c[64 * (2 * p + 1)], F.t);
                H[p] = (double)f * (p == 0 || p == 3 || p == 5 ? i2h : 0.5 * i2h);
            }
        }
    }

    __device__ __forceinline__ void at_step(const CastArgs& a, const RayGeom& geo, const GeoState& y, int L,
                                            const FieldCache<AMR>& F)
    {
        const GridDev& g = a.grid;
        double v[3];
        grid_coords(g, geo, y.eta, y.dx, v);
        double H[6];
        hessian(g, v, L, F, H);
        const double s = g.eta0 - y.eta;
        double r[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) r[i] = s * geo.n[i] + (double)y.dx[i];
        const double c2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
        double chi = 0.0, d[3] = {geo.n[0], geo.n[1], geo.n[2]};      // unit direction
        if (c2 > 0.0) {
            const double ic = inv_sqrt(c2);
            chi = c2 * ic;
#pragma unroll
            for (int i = 0; i < 3; ++i) d[i] = r[i] * ic;
        }
        const double st2 = d[0] * d[0] + d[1] * d[1];
        double cp = 1.0, sp = 0.0, st = 0.0;
        if (st2 > 0.0) {
            const double is = inv_sqrt(st2);
            cp = d[0] * is;
            sp = d[1] * is;
            st = st2 * is;
        }
        // e1 = (-sp, cp, 0), e2 = (-cp ct, -sp ct, st); T_ab = e_a . H e_b
        const double ct = d[2];
        const double u0 = cp * H[1] - sp * H[0], u1 = cp * H[3] - sp * H[1], u2 = cp * H[4] - sp * H[2];
        const double q0 = cp * H[0] + sp * H[1], q1 = cp * H[1] + sp * H[3], q2 = cp * H[2] + sp * H[4];
        const double w0 = st * H[2] - ct * q0, w1 = st * H[4] - ct * q1, w2 = st * H[5] - ct * q2;
        double T[3];
        T[0] = cp * u1 - sp * u0;
        T[1] = st * u2 - ct * (cp * u0 + sp * u1);
        T[2] = st * w2 - ct * (cp * w0 + sp * w1);
        const double dc = 0.5 * (chi - chi_p);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double t1 = chi * T[k], t2 = chi * t1;
            if (n > 0) {
                J1[k] += dc * (Tp[k] + t1);
                J2[k] += dc * (Up[k] + t2);
            }
            Tp[k] = t1;
            Up[k] = t2;
        }
        chi_p = chi;
        ++n;
    }

    template <class Run>
    __device__ __forceinline__ bool at_surface(const CastArgs&, Run&) { return false; }

    // A at the end of a ray that reached the source (after the end-point
    // sample); NaN otherwise or without two samples.
    __device__ __forceinline__ void write(float* A, bool reached) const
    {
        if (!reached || n < 2) {
            A[0] = A[1] = A[2] = A[3] = __builtin_nanf("");
            return;
        }
        const double cs = chi_p;
        const double I11 = J1[0] - J2[0] / cs, I12 = J1[1] - J2[1] / cs, I22 = J1[2] - J2[2] / cs;
        A[0] = (float)(1.0 - 2.0 * I11);
        A[1] = (float)(-2.0 * I12);
        A[2] = (float)(-2.0 * I12);
        A[3] = (float)(1.0 - 2.0 * I22);
    }
};

// One lane per ray: the static cast with the infinitesimal-beam samples
// (two stencil caches in LDS, so fewer resident waves than the plain cast).
template <bool AMR>
__global__ __launch_bounds__(kBlock, 2) void cast_infbeam_kernel(CastArgs a, float* A)
{
    extern __shared__ float coef_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    RayRun<AMR> R;
    R.F.bind(coef_lds);
    InfBeam<AMR> B;
    B.init(coef_lds + FieldCache<AMR>::kFloats * kBlock);
    R.start(a, r);
    R.template advance<false, InfBeam<AMR>>(a, 0x7fffffff, B);
    const bool reached = R.status == MPATH_RAY_REACHED;
    if (reached) {
        // end-point sample: leaf level of the end point
        double v[3];
        grid_coords(a.grid, R.geo, R.y.eta, R.y.dx, v);
        const int L = R.F.leaf(a.grid, v);       // -1 outside a non-periodic box
        B.at_step(a, R.geo, R.y, L < 0 ? 0 : L, R.F);
    }
    B.write(A + 4 * r, reached);
    R.finish(a);
}

// One lane per ray with dPhi/dl from the difference of Phi between step
// starts (the second form of the geodesic equations).
template <bool AMR>
__global__ __launch_bounds__(kBlock, kMinWavesPerSimd) void cast_diff_kernel(CastArgs a)
{
    extern __shared__ float coef_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    RayRun<AMR, FieldCache<AMR, false, true>, StepDifference> R;
    R.F.bind(coef_lds);
    R.start(a, r);
    R.advance(a, 0x7fffffff);
    R.finish(a);
}

// One lane per ray to an iso-chi, iso-lambda or iso-z surface (SURF).  At four
// waves per SIMD the iso-chi and iso-z kernels spill 32 to 60 of the 128
// registers, which gained them less from the unrolled stages than the plain
// cast: 196,608 rays to z = 1 on a uniform 64^3 grid 14.9 -> 13.8 and 15.3 ->
// 12.5 ms, iso-lambda without spills 13.5 -> 10.4.
template <bool AMR, int SURF>
__global__ __launch_bounds__(kBlock, kMinWavesPerSimd) void cast_stop_kernel(CastArgs a)
{
    extern __shared__ float coef_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    RayRun<AMR> R;
    R.F.bind(coef_lds);
    R.start(a, r);
    int j = a.n_obs - 1;
    while (j > 0 && a.obs[j].ray_first > r) --j;
    R.template advance_stop<SURF>(a, a.obs[j].p_s);
    R.finish_stop(a);
}

// Intermediate stop surfaces of a cast (the paper's maps at several source
// redshifts from one run): landing on surface k < n_extra writes the ray's
// observables there to output block k and sends the ray on to surface k + 1;
// the observer's own stop is the last surface (block n_extra).
struct Surfaces {
    const double2* surf;    // [n_obs][n_extra] (eta_s, a_s), nearest first
    int n_extra;
    int k;

    template <class FC>
    __device__ __forceinline__ void at_step(const CastArgs&, const RayGeom&, const GeoState&, int, const FC&) {}

    template <class Run>
    __device__ __forceinline__ bool at_surface(const CastArgs& a, Run& R)
    {
        if (k >= n_extra) return false;
        int j = a.n_obs - 1;
        while (j > 0 && a.obs[j].ray_first > R.ray) --j;
        const double a_s = surf[j * n_extra + k].y;
        R.write_outputs(a, (int64_t)k * a.n_rays + R.ray, j, a_s, 1.0 / a_s - 1.0, MPATH_RAY_REACHED);
        ++k;
        R.eta_s = k < n_extra ? surf[j * n_extra + k].x : a.obs[j].eta_s;
        return true;
    }
};

template <bool AMR>
__global__ __launch_bounds__(kBlock, 2) void cast_surfaces_kernel(CastArgs a, Surfaces S)
{
    extern __shared__ float coef_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    RayRun<AMR> R;
    R.F.bind(coef_lds);
    R.start(a, r);
    int j = a.n_obs - 1;
    while (j > 0 && a.obs[j].ray_first > r) --j;
    R.eta_s = S.surf[j * S.n_extra].x;
    S.k = 0;
    R.template advance<false, Surfaces>(a, 0x7fffffff, S);
    // a ray that stopped before some surface: those slots get its status
    for (int k = S.k; k < S.n_extra; ++k) {
        const double a_s = S.surf[j * S.n_extra + k].y;
        R.write_outputs(a, (int64_t)k * a.n_rays + r, j, a_s, 1.0 / a_s - 1.0, R.status);
    }
    const ObsDev& ob = a.obs[j];
    R.write_outputs(a, (int64_t)S.n_extra * a.n_rays + r, j, ob.a_s, ob.z0, R.status);
}

// Born approximation of the infinitesimal-beam matrix: the same
// line-of-sight integral taken along the straight line x_obs + chi n from the
// observer to the stop surface's comoving distance chi_s = eta_0 - eta_s,
// sampled at chi_{i+1} = min(chi_i + ds_i, chi_s), ds_i the integration's
// step length at x(chi_i) (N steps per leaf or coarse cell).
template <bool AMR>
__global__ __launch_bounds__(kBlock, 2) void born_beam_kernel(CastArgs a, float* A, int32_t* status_out)
{
    extern __shared__ float born_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    const GridDev& g = a.grid;
    int j = a.n_obs - 1;
    while (j > 0 && a.obs[j].ray_first > r) --j;
    const ObsDev& ob = a.obs[j];
    RayGeom geo;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        geo.vo[i] = ldexp(ob.x[i] / g.h0, g.max_level + 1);
        geo.n[i] = a.dirs[3 * r + i];
    }
    const double eta_s = a.ray_stop ? a.ray_stop[r].x : ob.eta_s;
    const double chis = a.cosmo_eta0 - eta_s;
    InfBeam<AMR, true> B;
    FieldCache<AMR> F;
    B.init(born_lds);
    F.bind(born_lds + InfBeam<AMR>::kFloats * kBlock);
    F.reset();
    GeoState y;
    y.K = 1.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) { y.d[i] = 0.0f; y.dx[i] = 0.0f; }
    double chi = 0.0;
    int status = MPATH_RAY_MAX_STEPS;
    for (int64_t steps = 0;; ++steps) {
        y.eta = a.cosmo_eta0 - chi;
        double v[3];
        grid_coords(g, geo, y.eta, y.dx, v);
        const int L = F.leaf(g, v);
        if (L < 0) { status = MPATH_RAY_LEFT_DOMAIN; break; }
        B.at_step(a, geo, y, L, F);
        if (chi >= chis) { status = MPATH_RAY_REACHED; break; }
        if (steps >= a.max_steps) break;
        const double ds = step_length(a, L);
        chi = chi + ds < chis ? chi + ds : chis;
    }
    B.write(A + 4 * r, status == MPATH_RAY_REACHED);
    if (status_out) status_out[r] = status;
}

// Static schedule with the NGP (ORDER 0) or TSC (ORDER 2) field evaluator.
template <bool AMR, int ORDER>
__global__ __launch_bounds__(kBlock, 2) void cast_order_kernel(CastArgs a)
{
    extern __shared__ float order_lds[];
    int64_t r;
    if (!lane_ray(a, a.n_rays, r)) return;
    using FC = typename std::conditional<ORDER == 0, NgpCache<AMR>, TscCache<AMR>>::type;
    RayRun<AMR, FC> R;
    R.F.bind(order_lds);
    R.start(a, r);
    R.advance(a, 0x7fffffff);
    R.finish(a);
}

__global__ void zero_u64(unsigned long long* p) { *p = 0ull; }

__global__ void permute_values_kernel(float4* payload, const int64_t* perm, const float4* values, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) payload[i] = values[perm[i]];
}

// ---------------------------------------------------------------------------
// Forward-mode derivative of the cast with respect to the initial direction
// theta: two tangents, b = 1, 2, moving the initial unit vector n along
// e1 = e_phi, e2 = -e_theta (the screen basis at theta).  Written in the
// physical variables (eta, x, k0 = -K, k) of the geodesic equations
// (Sect. 2.2), whose RK4 map equals the split one of the kernels; the
// tangent of a state is kept as
//   (deta, dK, dX = dx - s e_b, dQ = dk - K e_b),   s = eta_0 - eta,
// so that the parts of order one (the unlensed change s e_b of the position
// and K e_b of the wave vector, carried exactly by the primal s and K) never
// enter float32 arithmetic, and only lensing-sized quantities do.  With
// F = dy/dl, psi = G.k and G, JG the interpolated gradient and its spatial
// derivative (the trilinear interpolant of the stencil),
//   deta' = -dK
//   dK'   = 2 H' K^2 deta + (4 H K - 2 psi) dK - 2 K dpsi
//   dX'   = dQ
//   dQ'   = 2 H' deta K k + 2 H dK k + (2 H K + 2 psi) dQ + 2 dpsi k
//           - 2 dG K^2 - 4 G K dK + 4 psi K e_b,
//   dG = JG (s e_b + dX),  dpsi = dG.k + K G.e_b + G.dQ,
// and RK4 is differentiated stage by stage, including the step length
// dl = ds / K (d(dl) = -dl dK / K: the term rho (Y_i - y), rho = -dK/K,
// with Y_i - y = c_i dl F_{i-1}).  The landing step's length is set by the
// source surface; its pass is differentiated at fixed length and the end
// tangent projected along the flow afterwards (tangent_observables_kernel).
// ---------------------------------------------------------------------------
//
// The kernels are bound by instruction issue, so a stage's factors common to
// both tangents are formed once, the three scalar products in dpsi are one sum
// over the axes, and the scale of JG goes onto the displacement it multiplies.
// Every operation is written out (no contraction), so that one and four lanes
// a ray (Form) give the same bits.
//
// A step's increments are formed in float32 and summed over the steps in double
// precision.  Summed in float32 over the 3,000 steps of 8,192 rays to z = 1
// (uniform 64^3) they left dz5/dtheta a median error of 1.3e-8 against 64 bits
// (rms of the values 2.6e-2) and A one of 1.0e-8, in double 2.6e-9 and 2.4e-9, a
// reverse sweep of three columns 3.0e-9 and 3.8e-9.  It takes no more time for
// 4,096 to 131,072 rays (within 0.5 per cent) and 1.5 to 2 per cent more for
// 2^20 and 2^25.6 (101.0 -> 102.5 ms, 7.12 -> 7.26 s).
template <class Form>
struct TangentPair {
    static constexpr int C = Form::kComp;
    float n[C];                                   // initial direction
    float e[2][C];                                // e_b
    double dEta[2], dK[2], dX[2][C], dQ[2][C];    // tangents at the step start
    float fEta[2], fK[2], fX[2][C], fQ[2][C];     // their derivative at the previous stage
    float aEta[2], aK[2], aX[2][C], aQ[2][C];     // sum of w_i times it over the stages
    float rho[2];                                  // d(dl)/dl of the recorded pass
    float dlf;                                     // its affine length
    double eta0;
    float inv_h0;

    // v: the initial direction
    __device__ __forceinline__ void init(const CastArgs& a, const double v[3], float phi_o)
    {
        #pragma clang fp contract(off)
        eta0 = a.cosmo_eta0;
        inv_h0 = (float)a.grid.inv_h0;
        const double rh = hypot(v[0], v[1]);
        const double cp = rh > 0.0 ? v[0] / rh : 1.0, sp = rh > 0.0 ? v[1] / rh : 0.0;
        const double ct = v[2], st = rh;
        const double eb[2][3] = {{-sp, cp, 0.0}, {-cp * ct, -sp * ct, st}};
        // k = kmag n at the observer, so dk = kmag e_b there and dQ = (kmag - 1) e_b
        const double po = (double)phi_o;
        const float km1 = (float)(sqrt((1.0 + 2.0 * po) / (1.0 - 2.0 * po)) - 1.0);
        auto own = [&](const double* u, int i) {
            const int ax = Form::own_axis(i);
            return (float)(ax == 0 ? u[0] : ax == 1 ? u[1] : u[2]);
        };
#pragma unroll
        for (int i = 0; i < C; ++i) n[i] = own(v, i);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            dEta[b] = 0.0;
            dK[b] = 0.0;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                e[b][i] = own(eb[b], i);
                dX[b][i] = 0.0;
                dQ[b][i] = km1 * e[b][i];
            }
        }
    }

    __device__ __forceinline__ void begin_step(const GeoState& y, double dl, bool regular)
    {
        dlf = (float)dl;
        const float invK = 1.0f / (float)y.K;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            rho[b] = regular ? -(float)dK[b] * invK : 0.0f;
            aEta[b] = 0.0f;
            aK[b] = 0.0f;
#pragma unroll
            for (int i = 0; i < C; ++i) { aX[b][i] = 0.0f; aQ[b][i] = 0.0f; }
        }
    }

    // Y - y in the physical variables: (eta, K, x, k) differences
    __device__ __forceinline__ void diff(const GeoState& y, const GeoState& Y, float& De, float& DK, float Dx[C],
                                         float Dk[C]) const
    {
        #pragma clang fp contract(off)
        De = (float)(Y.eta - y.eta);
        DK = (float)(Y.K - y.K);
        const float KY = (float)Y.K, Ky = (float)y.K;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            Dx[i] = fmaf(-De, n[i], Y.dx[i] - y.dx[i]);
            Dk[i] = fmaf(DK, n[i], fmaf(KY, Y.d[i], -Ky * y.d[i]));
        }
    }

    template <class FC>
    __device__ __forceinline__ void stage(int st, const GeoState& y, const GeoState& yi, const FC& F,
                                          const float* G, const HubbleCubic& Hc, const CosmoDev& cz)
    {
        #pragma clang fp contract(off)
        const float c = st == 0 ? 0.0f : (st == 3 ? 1.0f : 0.5f);
        const float cdl = c * dlf;
        const float w = (st == 0 || st == 3) ? 1.0f : 2.0f;
        const float Kf = (float)yi.K;
        float k[C], Gk[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            k[i] = Kf * (n[i] + yi.d[i]);
            Gk[i] = G[i] * k[i];
        }
        const float s = (float)(eta0 - yi.eta);
        const float H = (float)Hc(cz, yi.eta), dH = (float)Hc.deriv(cz, yi.eta);
        const float psi = Form::sum(Gk);
        float De, DK, Dx[C], Dk[C];
        diff(y, yi, De, DK, Dx, Dk);
        // spatial derivative of the interpolated gradient: the t-derivatives
        // of the stencil's trilinear interpolant times 2^lvl / h0
        float t[3];
        F.offsets(t);
        const float sc = ldexpf(inv_h0, F.lvl);
        float JG[C][3];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            float4 p, q;            // c0..c3, c4..c7
            F.coefs(j, p, q);
            JG[j][0] = fmaf(t[2], q.y, fmaf(t[1], fmaf(t[2], q.w, q.x), p.y));
            JG[j][1] = fmaf(t[2], q.z, fmaf(t[0], fmaf(t[2], q.w, q.x), p.z));
            JG[j][2] = fmaf(t[1], q.z, fmaf(t[0], fmaf(t[1], q.w, q.y), p.w));
        }
        const float K2 = Kf + Kf;
        const float hk = dH * K2;                         // 2 H' K
        const float hk2 = hk * Kf;                        // 2 H' K^2
        const float h2 = H + H;
        const float cq = fmaf(h2, Kf, psi + psi);         // 2 H K + 2 psi
        const float ck0 = fmaf(h2, K2, -(psi + psi));     // 4 H K - 2 psi
        const float cg = -K2 * Kf, cK = -(K2 + K2);       // -2 K^2, -4 K
        const float ce = (K2 + K2) * psi;                 // 4 psi K
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float te = (float)dEta[b], tK = (float)dK[b], tX[C], tQ[C];
#pragma unroll
            for (int i = 0; i < C; ++i) { tX[i] = (float)dX[b][i]; tQ[i] = (float)dQ[b][i]; }
            if (st > 0) {
                te = fmaf(rho[b], De, fmaf(cdl, fEta[b], te));
                tK = fmaf(rho[b], DK, fmaf(cdl, fK[b], tK));
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    tX[i] = fmaf(rho[b], Dx[i], fmaf(cdl, fX[b][i], tX[i]));
                    tQ[i] = fmaf(rho[b], Dk[i], fmaf(cdl, fQ[b][i], tQ[i]));
                }
            }
            float dx[C], dxf[3], dG[C], pk[C];
#pragma unroll
            for (int i = 0; i < C; ++i) dx[i] = sc * fmaf(s, e[b][i], tX[i]);
            Form::whole_vector(dx, dxf);
#pragma unroll
            for (int j = 0; j < C; ++j) {
                dG[j] = fmaf(JG[j][2], dxf[2], fmaf(JG[j][1], dxf[1], JG[j][0] * dxf[0]));
                pk[j] = fmaf(G[j], fmaf(Kf, e[b][j], tQ[j]), dG[j] * k[j]);
            }
            const float dpsi = Form::sum(pk);
            fEta[b] = -tK;
            fK[b] = fmaf(hk2, te, fmaf(ck0, tK, -K2 * dpsi));
            const float ck = fmaf(hk, te, fmaf(h2, tK, dpsi + dpsi));
            const float cG = cK * tK;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                fX[b][i] = tQ[i];
                fQ[b][i] = fmaf(ck, k[i], fmaf(cq, tQ[i], fmaf(cg, dG[i], fmaf(cG, G[i], ce * e[b][i]))));
            }
            aEta[b] = fmaf(w, fEta[b], aEta[b]);
            aK[b] = fmaf(w, fK[b], aK[b]);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                aX[b][i] = fmaf(w, fX[b][i], aX[b][i]);
                aQ[b][i] = fmaf(w, fQ[b][i], aQ[b][i]);
            }
        }
    }

    // t + (rho D + h6 sum), the increment in float32
    static __device__ __forceinline__ double advanced(double t, float rho, float D, float h6, float sum)
    {
        #pragma clang fp contract(off)
        return t + (double)fmaf(rho, D, h6 * sum);
    }

    __device__ __forceinline__ void end_step(const GeoState& y, const GeoState& yn)
    {
        #pragma clang fp contract(off)
        float De, DK, Dx[C], Dk[C];
        diff(y, yn, De, DK, Dx, Dk);
        const float h6 = dlf * (1.0f / 6.0f);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            dEta[b] = advanced(dEta[b], rho[b], De, h6, aEta[b]);
            dK[b] = advanced(dK[b], rho[b], DK, h6, aK[b]);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                dX[b][i] = advanced(dX[b][i], rho[b], Dx[i], h6, aX[b][i]);
                dQ[b][i] = advanced(dQ[b][i], rho[b], Dk[i], h6, aQ[b][i]);
            }
        }
    }
};

// The cast with the two tangents: the primal outputs of the plain cast (bit
// for bit) and the tangent end states for tangent_observables_kernel.
// The tangents take registers the plain cast has not: two waves per SIMD.
// QUAD: four lanes per ray.  S: the precision the end states are kept in.
template <bool AMR, bool QUAD, class S>
__global__ __launch_bounds__(kBlock, 2) void cast_tangent_kernel(CastArgs a, TanEndOf<S>* te)
{
    extern __shared__ float coef_lds[];
    using FC = typename std::conditional<QUAD, QuadCache<AMR>, FieldCache<AMR>>::type;
    int64_t r;
    if (!lane_ray<QUAD ? 4 : 1>(a, a.n_rays, r)) return;
    RayRun<AMR, FC> R;
    if constexpr (!QUAD) R.F.bind(coef_lds);
    R.start(a, r);
    TangentPair<FC> T;
    T.init(a, a.dirs + 3 * r, R.phi_o);
    R.advance_recorded(a, T);
    R.finish(a);           // leaves the end point's stencil in R.F
    TanEndOf<S> e;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        double dX[3];
        FC::whole_vector(T.dX[b], dX);
        e.deta[b] = (S)T.dEta[b];
        e.dK[b] = (S)T.dK[b];
#pragma unroll
        for (int i = 0; i < 3; ++i) e.dX[b][i] = (S)dX[i];
    }
    FC::whole_vector(R.y.d, e.d);
    e.phi_o = R.phi_o;
    e.K = R.y.K;
    e.base = R.F.base;
    e.lvl = R.F.lvl;
    e.status = R.status;
    e.pad = 0;
    te[r] = e;
}

// Distortion matrix and dz5/dtheta from the tangent end states (double
// precision).  The landing step ends on eta = eta_s whatever theta is, so
// the end tangent is projected along the flow F(y_f) until deta = 0:
// dy_f += F(y_f) deta / K_f.  Then, with r = x_f - x_obs,
//   A_ab = e~_a(beta) . (s_f e_b + dX_b) / |r|     (Sect. 2.3, rows on the
//          screen basis at the end direction, columns on the one at theta)
//   dz5_b = a_s / (1 + Phi_o) [dK_b (1 + Phi_s) + K_f dPhi_s_b],
// dPhi_s_b the derivative of the interpolated Phi along the end tangent
// (Sect. 2.5, z5 with v = 0).
template <class S>
__global__ __launch_bounds__(256) void tangent_observables_kernel(CastArgs a, const TanEndOf<S>* te, float* jac,
                                                                  float* dz)
{
    const int64_t ray = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (ray >= a.n_rays) return;
    const float q = __builtin_nanf("");
    const TanEndOf<S> T = te[ray];
    if (T.status != MPATH_RAY_REACHED) {
        if (jac) {
#pragma unroll
            for (int i = 0; i < 4; ++i) jac[4 * ray + i] = q;
        }
        if (dz) { dz[2 * ray] = q; dz[2 * ray + 1] = q; }
        return;
    }
    const GridDev& g = a.grid;
    const RayEnd e = a.ends[ray];
    const ObsDev& ob = a.obs[e.obs];
    const double n[3] = {a.dirs[3 * ray], a.dirs[3 * ray + 1], a.dirs[3 * ray + 2]};
    const double s = a.cosmo_eta0 - e.eta;
    double r[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) r[i] = s * n[i] + (double)e.dx[i];
    const double chi = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    // bases: e_b at theta, e~_a at the end direction
    auto basis = [](const double v[3], double e1[3], double e2[3]) {
        const double rh = hypot(v[0], v[1]), rr = sqrt(rh * rh + v[2] * v[2]);
        const double cp = rh > 0.0 ? v[0] / rh : 1.0, sp = rh > 0.0 ? v[1] / rh : 0.0;
        const double ct = v[2] / rr, st = rh / rr;
        e1[0] = -sp; e1[1] = cp; e1[2] = 0.0;
        e2[0] = -cp * ct; e2[1] = -sp * ct; e2[2] = st;
    };
    double eb[2][3], ea[2][3];
    basis(n, eb[0], eb[1]);
    basis(r, ea[0], ea[1]);
    // the interpolant at the end point: Phi, its gradient and grad Phi
    double v[3];
    {
        RayGeom geo;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            geo.vo[i] = ldexp(ob.x[i] / g.h0, g.max_level + 1);
            geo.n[i] = n[i];
        }
        grid_coords(g, geo, e.eta, e.dx, v);
    }
    const double sl = ldexp(1.0, T.lvl - g.max_level - 1);
    double t[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double u = v[d] * sl - 0.5;
        t[d] = u - floor(u);
    }
    const float4* rec = g.dual + 8 * (int64_t)T.base;
    double cf[4][8];             // phi, gx, gy, gz
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        const float4 c4 = rec[o];
        double* q = cf[(o / 2 + 1) & 3] + 4 * (o & 1);
        q[0] = c4.x; q[1] = c4.y; q[2] = c4.z; q[3] = c4.w;
    }
    auto tri = [&](const double* c, double& f, double& fx, double& fy, double& fz) {
        const double tx = t[0], ty = t[1], tz = t[2];
        f = c[0] + tx * (c[1] + ty * (c[4] + tz * c[7]) + tz * c[5]) + ty * (c[2] + tz * c[6]) + tz * c[3];
        fx = c[1] + ty * c[4] + tz * c[5] + ty * tz * c[7];
        fy = c[2] + tx * c[4] + tz * c[6] + tx * tz * c[7];
        fz = c[3] + tx * c[5] + ty * c[6] + tx * ty * c[7];
    };
    const double scale = ldexp(g.inv_h0, T.lvl);
    double phis, gp[3], G[3], dum[3];
    tri(cf[0], phis, gp[0], gp[1], gp[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) gp[i] *= scale;
#pragma unroll
    for (int j = 0; j < 3; ++j) tri(cf[j + 1], G[j], dum[0], dum[1], dum[2]);
    HubbleCubic Hc;
    Hc.init(a.cosmo, e.eta);
    const double H = Hc(a.cosmo, e.eta);
    const double K = T.K;
    double k[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) k[i] = K * (n[i] + (double)T.d[i]);
    const double psi = G[0] * k[0] + G[1] * k[1] + G[2] * k[2];
    const double FK = 2.0 * H * K * K - 2.0 * psi * K;
    const double a_s = a.ray_stop ? a.ray_stop[ray].y : ob.a_s;
    const double pref = a_s / (1.0 + (double)T.phi_o);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const double tau = (double)T.deta[b] / K;
        double dr[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) dr[i] = s * eb[b][i] + ((double)T.dX[b][i] + tau * k[i]);
        const double dKb = (double)T.dK[b] + tau * FK;
        if (jac) {
#pragma unroll
            for (int aa = 0; aa < 2; ++aa)
                jac[4 * ray + 2 * aa + b] = (float)((ea[aa][0] * dr[0] + ea[aa][1] * dr[1] + ea[aa][2] * dr[2]) / chi);
        }
        if (dz) {
            const double dphi = gp[0] * dr[0] + gp[1] * dr[1] + gp[2] * dr[2];
            dz[2 * ray + b] = (float)(pref * (dKb * (1.0 + phis) + K * dphi));
        }
    }
}

}  // namespace

// A cast's rays take four lanes each where that needs at most two waves per
// SIMD on a uniform grid, four on a tree.  A quad's wave issues two
// thirds of the instructions of a step, and waits for no coefficients from
// LDS, but carries a quarter of the rays; on a tree it also gathers and
// diverges for 16 rays and not for 64.  One lane against four, uniform 64^3,
// to z = 0.3: 3,072 rays 1.59 ms and 1.02, 12,288 1.86 and 1.21, 32,768 (two
// waves) 2.02 and 1.66, 49,152 2.13 and 2.19; 64^3 + 5 levels: 3,072 1.44 and
// 1.09, 32,768 2.33 and 1.76, 65,536 (four) 2.58 and 2.14, 98,304 2.51 and
// 2.96.  With checkpoints the same.
static int quad_waves(const CastArgs& a) { return a.grid.max_level > 0 ? 4 : 2; }

template <bool CKPT>
static hipError_t launch_cast_quad(const CastArgs& args, hipStream_t s)
{
    const bool amr = args.grid.max_level > 0;
    const CastArgs a = spread_rays(args, args.form_rays, amr ? 2 : 1, kWave / 4);
    const dim3 grid = ray_grid(a, a.n_rays), blk(kBlock);
    if (amr) hipLaunchKernelGGL((cast_quad_kernel<true, CKPT>), grid, blk, 0, s, a);
    else hipLaunchKernelGGL((cast_quad_kernel<false, CKPT>), grid, blk, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_cast_static(const CastArgs& args, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const bool amr = args.grid.max_level > 0, td = args.grid.tdual != nullptr;
    if (!td && by_quads(args, args.form_rays, quad_waves(args))) return launch_cast_quad<false>(args, s);
    const CastArgs a = spread_rays(args, args.form_rays, amr ? 2 : 1);
    const size_t lds = (size_t)(td ? FieldCache<true, true>::kFloats : FieldCache<true>::kFloats) * kBlock *
                       sizeof(float);
    const dim3 grid = ray_grid(a, a.n_rays), blk(kBlock);
    if (td) {
        if (amr) hipLaunchKernelGGL((cast_static_kernel<true, true>), grid, blk, lds, s, a);
        else hipLaunchKernelGGL((cast_static_kernel<false, true>), grid, blk, lds, s, a);
    } else {
        if (amr) hipLaunchKernelGGL((cast_static_kernel<true, false>), grid, blk, lds, s, a);
        else hipLaunchKernelGGL((cast_static_kernel<false, false>), grid, blk, lds, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_cast_checkpointed(const CastArgs& args, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    if (by_quads(args, args.form_rays, quad_waves(args))) return launch_cast_quad<true>(args, s);
    const CastArgs a = spread_rays(args, args.form_rays, 1);
    const size_t lds = (size_t)FieldCache<true>::kFloats * kBlock * sizeof(float);
    if (a.grid.max_level > 0)
        hipLaunchKernelGGL(cast_ckpt_kernel<true>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a);
    else
        hipLaunchKernelGGL(cast_ckpt_kernel<false>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_cast_infbeam(const CastArgs& args, float* A, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const CastArgs a = spread_rays(args, args.form_rays, 1);
    const size_t lds = (size_t)(FieldCache<true>::kFloats + std::max(InfBeam<true>::kFloats, InfBeam<false>::kFloats)) *
                       kBlock * sizeof(float);
    if (a.grid.max_level > 0)
        hipLaunchKernelGGL(cast_infbeam_kernel<true>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a, A);
    else
        hipLaunchKernelGGL(cast_infbeam_kernel<false>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a, A);
    return hipGetLastError();
}

template <class T>
hipError_t launch_cast_tangent(const CastArgs& args, TanEndOf<T>* te, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    // four lanes a ray up to two waves per SIMD (registers admit no more):
    // 12,288 rays 3.51 ms and 2.06, 32,768 3.68 and 3.25, 49,152 3.82 and 4.59
    // (uniform); 2.85 and 1.93, 3.29 and 2.38, 3.34 and 3.60 (tree)
    const bool quad = by_quads(args, args.form_rays, 2);
    const CastArgs a = spread_rays(args, args.form_rays, 1, quad ? kWave / 4 : kWave);
    const bool amr = a.grid.max_level > 0;
    const size_t lds = quad ? 0 : (size_t)FieldCache<true>::kFloats * kBlock * sizeof(float);
    const dim3 grid = ray_grid(a, a.n_rays), blk(kBlock);
    if (quad) {
        if (amr) hipLaunchKernelGGL((cast_tangent_kernel<true, true, T>), grid, blk, lds, s, a, te);
        else hipLaunchKernelGGL((cast_tangent_kernel<false, true, T>), grid, blk, lds, s, a, te);
    } else {
        if (amr) hipLaunchKernelGGL((cast_tangent_kernel<true, false, T>), grid, blk, lds, s, a, te);
        else hipLaunchKernelGGL((cast_tangent_kernel<false, false, T>), grid, blk, lds, s, a, te);
    }
    return hipGetLastError();
}

template <class T>
hipError_t launch_tangent_observables(const CastArgs& a, const TanEndOf<T>* te, float* jac, float* dz_dtheta,
                                      hipStream_t s)
{
    if (a.n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(tangent_observables_kernel<T>, dim3((unsigned)((a.n_rays + 255) / 256)), dim3(256), 0, s, a, te,
                       jac, dz_dtheta);
    return hipGetLastError();
}

template hipError_t launch_cast_tangent(const CastArgs&, TanEnd*, hipStream_t);
template hipError_t launch_cast_tangent(const CastArgs&, TanEnd64*, hipStream_t);
template hipError_t launch_tangent_observables(const CastArgs&, const TanEnd*, float*, float*, hipStream_t);
template hipError_t launch_tangent_observables(const CastArgs&, const TanEnd64*, float*, float*, hipStream_t);

hipError_t launch_cast_order(const CastArgs& args, int order, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const CastArgs a = spread_rays(args, args.form_rays, args.grid.max_level > 0 ? 2 : 1);
    const size_t lds = 0;
    const dim3 grid = ray_grid(a, a.n_rays), block(kBlock);
    const bool amr = a.grid.max_level > 0;
    if (order == 0) {
        if (amr) hipLaunchKernelGGL((cast_order_kernel<true, 0>), grid, block, lds, s, a);
        else hipLaunchKernelGGL((cast_order_kernel<false, 0>), grid, block, lds, s, a);
    } else {
        if (amr) hipLaunchKernelGGL((cast_order_kernel<true, 2>), grid, block, lds, s, a);
        else hipLaunchKernelGGL((cast_order_kernel<false, 2>), grid, block, lds, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_born_beam(const CastArgs& args, float* A, int32_t* status, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const CastArgs a = spread_rays(args, args.form_rays, 1);
    const size_t lds = (size_t)(FieldCache<true>::kFloats + std::max(InfBeam<true>::kFloats, InfBeam<false>::kFloats)) *
                       kBlock * sizeof(float);
    if (a.grid.max_level > 0)
        hipLaunchKernelGGL(born_beam_kernel<true>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a, A, status);
    else
        hipLaunchKernelGGL(born_beam_kernel<false>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a, A, status);
    return hipGetLastError();
}

hipError_t launch_cast_surfaces(const CastArgs& args, const double2* surf, int n_extra, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const CastArgs a = spread_rays(args, args.form_rays, 1);
    const size_t lds = (size_t)FieldCache<true>::kFloats * kBlock * sizeof(float);
    Surfaces S;
    S.surf = surf;
    S.n_extra = n_extra;
    S.k = 0;
    if (a.grid.max_level > 0)
        hipLaunchKernelGGL(cast_surfaces_kernel<true>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a, S);
    else
        hipLaunchKernelGGL(cast_surfaces_kernel<false>, ray_grid(a, a.n_rays), dim3(kBlock), lds, s, a, S);
    return hipGetLastError();
}

hipError_t launch_cast_stop(const CastArgs& args, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const CastArgs a = spread_rays(args, args.form_rays, 1);
    const dim3 grid = ray_grid(a, a.n_rays), blk(kBlock);
    const size_t lds = (size_t)FieldCache<true>::kFloats * kBlock * sizeof(float);
    const bool amr = a.grid.max_level > 0;
    switch (a.surface) {
        case MPATH_SURFACE_CHI:
            if (amr) hipLaunchKernelGGL((cast_stop_kernel<true, MPATH_SURFACE_CHI>), grid, blk, lds, s, a);
            else hipLaunchKernelGGL((cast_stop_kernel<false, MPATH_SURFACE_CHI>), grid, blk, lds, s, a);
            break;
        case MPATH_SURFACE_LAMBDA:
            if (amr) hipLaunchKernelGGL((cast_stop_kernel<true, MPATH_SURFACE_LAMBDA>), grid, blk, lds, s, a);
            else hipLaunchKernelGGL((cast_stop_kernel<false, MPATH_SURFACE_LAMBDA>), grid, blk, lds, s, a);
            break;
        case MPATH_SURFACE_Z:
            if (amr) hipLaunchKernelGGL((cast_stop_kernel<true, MPATH_SURFACE_Z>), grid, blk, lds, s, a);
            else hipLaunchKernelGGL((cast_stop_kernel<false, MPATH_SURFACE_Z>), grid, blk, lds, s, a);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_cast_diff(const CastArgs& args, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    const CastArgs a = spread_rays(args, args.form_rays, 1);
    const dim3 grid = ray_grid(a, a.n_rays), blk(kBlock);
    const size_t lds = (size_t)FieldCache<true, false, true>::kFloats * kBlock * sizeof(float);
    if (a.grid.max_level > 0) hipLaunchKernelGGL(cast_diff_kernel<true>, grid, blk, lds, s, a);
    else hipLaunchKernelGGL(cast_diff_kernel<false>, grid, blk, lds, s, a);
    return hipGetLastError();
}

hipError_t launch_ray_dirs(const CastArgs& a, hipStream_t s)
{
    if (a.n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(ray_dirs_kernel, dim3((unsigned)((a.n_rays + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_observables(const CastArgs& a, hipStream_t s)
{
    if (a.n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(observables_kernel, dim3((unsigned)((a.n_rays + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_cast_persistent(const CastArgs& a, int block, int blocks, hipStream_t s)
{
    if (a.n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_u64, dim3(1), dim3(1), 0, s, a.queue);
    const bool amr = a.grid.max_level > 0, td = a.grid.tdual != nullptr;
    const size_t lds = (size_t)(td ? FieldCache<true, true>::kFloats : FieldCache<true>::kFloats) * block *
                       sizeof(float);
    const dim3 grid(blocks), blk(block);
    if (td) {
        if (amr) hipLaunchKernelGGL((cast_persistent_kernel<true, true>), grid, blk, lds, s, a);
        else hipLaunchKernelGGL((cast_persistent_kernel<false, true>), grid, blk, lds, s, a);
    } else {
        if (amr) hipLaunchKernelGGL((cast_persistent_kernel<true, false>), grid, blk, lds, s, a);
        else hipLaunchKernelGGL((cast_persistent_kernel<false, false>), grid, blk, lds, s, a);
    }
    return hipGetLastError();
}

int cast_occupancy_blocks_per_cu(int block, bool amr, bool time_dep)
{
    int nb = 0;
    const size_t lds = (size_t)(time_dep ? FieldCache<true, true>::kFloats : FieldCache<true>::kFloats) * block *
                       sizeof(float);
    hipError_t e;
    if (time_dep)
        e = amr ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, cast_persistent_kernel<true, true>, block, lds)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, cast_persistent_kernel<false, true>, block, lds);
    else
        e = amr ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, cast_persistent_kernel<true, false>, block, lds)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, cast_persistent_kernel<false, false>, block, lds);
    return e == hipSuccess ? nb : 0;
}

hipError_t launch_permute_values(float4* payload, const int64_t* perm, const float4* values, int64_t n,
                                 hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(permute_values_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, payload, perm,
                       values, n);
    return hipGetLastError();
}

}  // namespace mpath
