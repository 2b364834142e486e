// adjoint.hip -- reverse-mode derivative of the ray-casting map on gfx950.
//
// The forward cast (with checkpoints) stores every ray's state before steps
// 0, K, 2K, ...  The reverse sweep then runs, per ray, segment by segment from
// the source back to the observer: it recomputes the steps of the segment from
// its checkpoint (the same code as the forward, so every leaf level, stencil
// and landing decision is replayed exactly) into a per-ray tape, and for every
// step in reverse order re-records the four RK4 stages and applies the
// transposed Jacobian of the step.
//
// The derivative is that of the discrete map: classical RK4 on the null
// geodesic equations of Sect. 2.2 with CIC interpolation (piecewise
// trilinear, so grad Phi has a piecewise-constant spatial derivative), step
// length h_leaf / N with affine step ds / |k0| (differentiated through k0),
// and the landing step on the source iso-eta surface (implicit step length).
// It is taken on the physical variables (eta, x, k0, k), whose RK4 map equals
// the split one of the forward kernels.  Precision follows the forward: the
// cotangent of the state is accumulated in double precision, while the
// per-stage products (stage Jacobians applied to small cotangent increments)
// run in single precision, like the stage arithmetic of the forward.
//
// Cotangent columns:
//   L                adjoint_loss_kernel: a scalar loss through the per-ray
//                    cotangents (dL/dalpha, dL/dz5); its cotangents of the
//                    interpolated (Phi, grad Phi) at every sub-step are
//                    scattered to the cells with the CIC weights (dL/d cell
//                    values)
//   beta_1, beta_2   adjoint_kernel: e~_a(beta) . x / |x_s - x_obs|; their
//                    values at the observer, contracted with d k / d theta_b,
//                    give the distortion matrix A_ab = d beta_a / d theta_b
//                    (Sect. 2.3).  Only the finder's Newton steps take it so:
//                    the two tangents of cast_tangent_kernel, which cost two
//                    forwards, give the other products.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"

namespace mpath {
namespace {

// Physical state (eta, x, k0, k) or a cotangent of it, in precision T.
template <class T>
struct PhysT {
    T eta, x[3], k0, k[3];
};
using Phys = PhysT<double>;
using Phys32 = PhysT<float>;

template <class T>
__device__ __forceinline__ void phys_zero(PhysT<T>& a)
{
    a.eta = T(0); a.k0 = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) { a.x[i] = T(0); a.k[i] = T(0); }
}

template <class T, class U>
__device__ __forceinline__ void phys_axpy(PhysT<T>& a, T s, const PhysT<U>& b)
{
    a.eta += s * (T)b.eta; a.k0 += s * (T)b.k0;
#pragma unroll
    for (int i = 0; i < 3; ++i) { a.x[i] += s * (T)b.x[i]; a.k[i] += s * (T)b.k[i]; }
}

template <class T>
__device__ __forceinline__ T phys_dot(const PhysT<T>& a, const PhysT<T>& b)
{
    T s = a.eta * b.eta + a.k0 * b.k0;
#pragma unroll
    for (int i = 0; i < 3; ++i) s += a.x[i] * b.x[i] + a.k[i] * b.k[i];
    return s;
}

__device__ __forceinline__ Phys32 to32(const Phys& a)
{
    Phys32 r;
    r.eta = (float)a.eta; r.k0 = (float)a.k0;
#pragma unroll
    for (int i = 0; i < 3; ++i) { r.x[i] = (float)a.x[i]; r.k[i] = (float)a.k[i]; }
    return r;
}

// What the forward computed at one RK4 stage: the state, the interpolated
// gradient and the stencil (lowest-corner id, level, offsets of the point).
struct StageData {
    GeoState y;
    float G[3], t[3];
    int base, lvl;
};

struct RayCtx {
    RayGeom geo;
};

// What the transposed stage Jacobian needs at one stage (single precision).
struct Jet32 {
    float k0, k[3];
    float G[3];
    float JG[3][3];     // dG_j / dx_l of the trilinear interpolant
    float H, dH;        // a'/a and its eta-derivative
    float t[3];         // CIC offsets (weights) at the stencil level
    int base, lvl;
};

// The four stages of one RK4 step for the Jacobian sweep (two columns),
// kept in this lane's LDS slots.  Word w of stage i is at p[(i * kWords + w) kBlock].
struct LdsRecord {
    static constexpr int kWords = 18;
    float* p;

    __device__ __forceinline__ void put(float* q, int w, float v) const { q[w * kBlock] = v; }
    __device__ __forceinline__ void put64(float* q, int w, double v) const
    {
        const unsigned long long b = (unsigned long long)__double_as_longlong(v);
        q[w * kBlock] = __uint_as_float((unsigned)b);
        q[(w + 1) * kBlock] = __uint_as_float((unsigned)(b >> 32));
    }
    __device__ __forceinline__ double get64(const float* q, int w) const
    {
        const unsigned long long lo = __float_as_uint(q[w * kBlock]);
        const unsigned long long hi = __float_as_uint(q[(w + 1) * kBlock]);
        return __longlong_as_double((long long)(lo | (hi << 32)));
    }

    template <class FC>
    __device__ __forceinline__ void stage(int i, const GeoState&, const GeoState& yi, const FC& F, const float* G,
                                          const HubbleCubic&, const CosmoDev&)
    {
        float* q = p + i * kWords * kBlock;
        put64(q, 0, yi.eta);
        put64(q, 2, yi.K);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            put(q, 4 + k, yi.d[k]);
            put(q, 7 + k, yi.dx[k]);
            put(q, 10 + k, G[k]);
            put(q, 13 + k, F.t[k]);
        }
        put(q, 16, __int_as_float(F.base));
        put(q, 17, __int_as_float(F.lvl));
    }

    template <int I>
    __device__ __forceinline__ StageData get() const
    {
        const float* q = p + I * kWords * kBlock;
        StageData d;
        d.y.eta = get64(q, 0);
        d.y.K = get64(q, 2);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            d.y.d[k] = q[(4 + k) * kBlock];
            d.y.dx[k] = q[(7 + k) * kBlock];
            d.G[k] = q[(10 + k) * kBlock];
            d.t[k] = q[(13 + k) * kBlock];
        }
        d.base = __float_as_int(q[16 * kBlock]);
        d.lvl = __float_as_int(q[17 * kBlock]);
        return d;
    }

    // the stage's jet, without the gradient's derivatives
    template <int I>
    __device__ __forceinline__ void jet(const CosmoDev& cz, const RayCtx& R, const HubbleCubic& Hc, Jet32& J) const
    {
        const StageData d = get<I>();
        const float K = (float)d.y.K;
        J.k0 = -K;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            J.k[i] = K * ((float)R.geo.n[i] + d.y.d[i]);
            J.G[i] = d.G[i];
            J.t[i] = d.t[i];
        }
        J.H = (float)Hc(cz, d.y.eta);
        J.dH = (float)Hc.deriv(cz, d.y.eta);
        J.base = d.base;
        J.lvl = d.lvl;
    }

    // the gradient's derivatives
    template <int I>
    __device__ __forceinline__ void gradient(const GridDev& g, Jet32& J) const;
};

// The same for the loss sweep (one column), in local variables: 13 or 14 words
// a stage.  With the stages unrolled every index is a constant, and without the
// records in LDS two waves fit a SIMD.  They do not all stay in registers: see
// adjoint_loss_kernel.
struct RegRecord {
    float K[4], H[4], dH[4], k[4][3], G[4][3], t[4][3];
    int base[4], lvl[4];

    template <class FC>
    __device__ __forceinline__ void stage(int i, const GeoState& y, const GeoState& yi, const FC& F, const float* g,
                                          const HubbleCubic& Hc, const CosmoDev& cz)
    {
        K[i] = (float)yi.K;
        H[i] = (float)Hc(cz, yi.eta);
        dH[i] = (float)Hc.deriv(cz, yi.eta);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            k[i][q] = yi.d[q];
            G[i][q] = g[q];
            t[i][q] = F.t[q];
        }
        base[i] = F.base;
        lvl[i] = FC::kUniform ? 0 : F.lvl;
    }

    template <int I>
    __device__ __forceinline__ void jet(const RayCtx& R, Jet32& J) const
    {
        J.k0 = -K[I];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            J.k[i] = K[I] * ((float)R.geo.n[i] + k[I][i]);
            J.G[i] = G[I][i];
            J.t[i] = t[I][i];
        }
        J.H = H[I];
        J.dH = dH[I];
        J.base = base[I];
        J.lvl = lvl[I];
    }

    // After a stage's transposed Jacobian its gradient's place takes the loss
    // cotangent of the interpolated gradient at that stage.
    template <int I>
    __device__ __forceinline__ void put_gbar(const float g[3])
    {
        G[I][0] = g[0]; G[I][1] = g[1]; G[I][2] = g[2];
    }
};

// Trilinear coefficients (component-major: c[8 q + k], gx, gy, gz) of a stencil, read
// from the dual table.  (The lane's LDS copy holds only the stencil of the
// replay's last stage; choosing between the two per lane made a wave wait
// for the table whenever any of its lanes missed, and the records of a
// step's stencils are in the caches after its replay.)
__device__ __forceinline__ void stencil_coefs(const GridDev& g, int base, float c[24])
{
    const float4* rec = g.dual + 8 * (int64_t)base;
#pragma unroll
    for (int o = 0; o < 6; ++o) {
        const float4 q = rec[o];
        c[4 * o] = q.x; c[4 * o + 1] = q.y; c[4 * o + 2] = q.z; c[4 * o + 3] = q.w;
    }
}

// Offsets of a stage position from its stencil's lowest corner, at the
// stencil level (as the forward interpolation computes them).
__device__ __forceinline__ void stage_offsets(const GridDev& g, const RayCtx& R, const GeoState& ys, int lvl,
                                              double t[3])
{
    double v[3];
    grid_coords(g, R.geo, ys.eta, ys.dx, v);
    const double sl = ldexp(1.0, lvl - g.max_level - 1);    // v sl = x 2^lvl / h0 exactly
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double q = v[d] * sl - 0.5;
        t[d] = q - floor(q);
    }
}

// Value and t-derivatives of one trilinear component
// f = c0 + tx (c1 + ty (c4 + tz c7) + tz c5) + ty (c2 + tz c6) + tz c3.
template <class T>
__device__ __forceinline__ void trilinear_jet(const T c[8], T tx, T ty, T tz, T& f, T& fx, T& fy, T& fz)
{
    f = c[0] + tx * (c[1] + ty * (c[4] + tz * c[7]) + tz * c[5]) + ty * (c[2] + tz * c[6]) + tz * c[3];
    fx = c[1] + ty * c[4] + tz * c[5] + ty * tz * c[7];
    fy = c[2] + tx * c[4] + tz * c[6] + tx * tz * c[7];
    fz = c[3] + tx * c[5] + ty * c[6] + tx * ty * c[7];
}

// Spatial derivatives of one component of the interpolated gradient (its
// coefficients k) at the stage: the t-derivatives of the trilinear
// interpolant (Eq. W_CIC) times scale = 2^lvl / h0.
__device__ __forceinline__ void gradient_row(const float k[8], const float t[3], float scale, float row[3])
{
    const float tx = t[0], ty = t[1], tz = t[2];
    row[0] = (k[1] + ty * k[4] + tz * k[5] + ty * tz * k[7]) * scale;
    row[1] = (k[2] + tx * k[4] + tz * k[6] + tx * tz * k[7]) * scale;
    row[2] = (k[3] + tx * k[5] + ty * k[6] + tx * ty * k[7]) * scale;
}

template <int I>
__device__ __forceinline__ void LdsRecord::gradient(const GridDev& g, Jet32& J) const
{
    float c[24];
    stencil_coefs(g, J.base, c);
    const float scale = (float)((double)(1 << J.lvl) * g.inv_h0);
#pragma unroll
    for (int j = 0; j < 3; ++j) gradient_row(c + 8 * j, J.t, scale, J.JG[j]);
}

// Right-hand side of the geodesic equations (Sect. 2.2) at a stage.
__device__ __forceinline__ Phys32 rhs32(const Jet32& J)
{
    Phys32 F;
    const float k0 = J.k0;
    const float psi = J.G[0] * J.k[0] + J.G[1] * J.k[1] + J.G[2] * J.k[2];
    F.eta = k0;
    F.k0 = -2.0f * J.H * k0 * k0 - 2.0f * psi * k0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        F.x[j] = J.k[j];
        F.k[j] = -2.0f * J.H * k0 * J.k[j] + 2.0f * psi * J.k[j] - 2.0f * J.G[j] * k0 * k0;
    }
    return F;
}

// Transposed Jacobian of the right-hand side at a stage applied to v:
// Yb = (dF/dY)^T v (Yb.x only with X) and the cotangent Gb of the interpolated
// grad Phi.
//   F = (k0, k, -2 H k0^2 - 2 psi k0, -2 H k0 k + 2 psi k - 2 G k0^2), psi = G.k
template <bool X = true>
__device__ __forceinline__ void rhs_vjp32(const Jet32& J, const Phys32& v, Phys32& Yb, float Gb[3])
{
    const float k0 = J.k0;
    const float a = v.k0;
    const float bk = v.k[0] * J.k[0] + v.k[1] * J.k[1] + v.k[2] * J.k[2];
    const float bG = v.k[0] * J.G[0] + v.k[1] * J.G[1] + v.k[2] * J.G[2];
    const float psi = J.G[0] * J.k[0] + J.G[1] * J.k[1] + J.G[2] * J.k[2];
#pragma unroll
    for (int j = 0; j < 3; ++j) Gb[j] = -2.0f * k0 * a * J.k[j] + 2.0f * bk * J.k[j] - 2.0f * k0 * k0 * v.k[j];
    Yb.eta = -2.0f * J.dH * k0 * (a * k0 + bk);
    Yb.k0 = v.eta + a * (-4.0f * J.H * k0 - 2.0f * psi) - 2.0f * J.H * bk - 4.0f * k0 * bG;
#pragma unroll
    for (int j = 0; j < 3; ++j)
        Yb.k[j] = v.x[j] - 2.0f * k0 * a * J.G[j] + (-2.0f * J.H * k0 + 2.0f * psi) * v.k[j] + 2.0f * J.G[j] * bk;
    if constexpr (X) {
#pragma unroll
        for (int l = 0; l < 3; ++l) Yb.x[l] = J.JG[0][l] * Gb[0] + J.JG[1][l] * Gb[1] + J.JG[2][l] * Gb[2];
    }
}

__device__ __forceinline__ void cic_weights(const float t[3], float w[8])
{
#pragma unroll
    for (int o = 0; o < 8; ++o)
        w[o] = ((o & 1) ? t[0] : 1.0f - t[0]) * ((o & 2) ? t[1] : 1.0f - t[1]) * ((o & 4) ? t[2] : 1.0f - t[2]);
}

// Cell cotangents in the adjoint workspace: component-major (phi, gx, gy,
// gz), and within a component the ids of every aligned group of 8
// consecutive cells (a Morton 2x2x2 block) spread over 8 regions, so that
// the atomics of one stencil flush land in different cache lines instead of
// serialising on one.
__device__ __forceinline__ int64_t grad_slot(int64_t id, int q, int64_t n)
{
    const int64_t m = (n + 7) >> 3;
    return (int64_t)q * (m << 3) + (id & 7) * m + (id >> 3);
}

// Per-wave table in LDS aggregating the gradient cotangents of recently
// touched cells: direct-mapped on a hash of the cell id, filled with LDS
// atomics by the lanes of one wave and evicted to the cell array with device
// atomics when a quarter full (a fuller table sends more colliding cells
// straight to the cell array, which costs more than the extra evictions).
// The 64 rays of a wave start from
// neighbouring sky pixels and cross the same cells many times, so the table
// absorbs most additions and the device atomics (which resolve beyond the
// per-XCD L2) drop by that reuse factor.
constexpr int kTab = 256;               // entries per wave (power of two)
constexpr int kTabWords = 4 * kTab + 4; // keys, 3 value planes, fill counter (padded)

struct WaveTable {
    int* keys;
    float* vals;        // [3][kTab]
    int* count;

    __device__ __forceinline__ void bind(float* base)
    {
        keys = reinterpret_cast<int*>(base);
        vals = base + kTab;
        count = reinterpret_cast<int*>(base + 4 * kTab);
    }

    // every lane of the (full) wave clears a share of the table
    __device__ __forceinline__ void clear(int lane)
    {
        for (int e = lane; e < kTab; e += 64) {
            keys[e] = -1;
            vals[e] = 0.0f;
            vals[kTab + e] = 0.0f;
            vals[2 * kTab + e] = 0.0f;
        }
        if (lane == 0) *count = 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }

    // Move every entry to the cell array; the currently active lanes share
    // the work.
    __device__ __forceinline__ void evict(const AdjointArgs& A)
    {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        const int lane = threadIdx.x & 63;
        const uint64_t act = __ballot(1);
        const int nact = __popcll(act);
        const int rank = __popcll(act & ((1ull << lane) - 1ull));
        for (int e = rank; e < kTab; e += nact) {
            const int key = keys[e];
            if (key >= 0) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float v = vals[q * kTab + e];
                    if (v != 0.0f) unsafeAtomicAdd(A.grad + grad_slot(key, 1 + q, A.n_cells), v);
                    vals[q * kTab + e] = 0.0f;
                }
                keys[e] = -1;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (rank == 0) *count = 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }

    // Add the cotangents acc[o] of the 8 stencil cells ids[o] (-1: no cell).
    // The table is direct-mapped on a hash of the cell id: a cell whose slot
    // is free or already its own is added in LDS; one whose slot holds
    // another cell goes straight to the cell array.  The 8 slot claims are
    // issued together and the LDS additions carry a zero where the slot is
    // not the cell's, so that the common path has no branches.
    __device__ __forceinline__ void add8(const AdjointArgs& A, const int ids[8], const float (&acc)[8][3])
    {
        int h[8], old[8];
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            h[o] = (int)(((uint32_t)ids[o] * 2654435761u) >> (32 - 8));
            old[o] = ids[o] >= 0 ? atomicCAS(&keys[h[o]], -1, ids[o]) : ids[o];
        }
        int claimed = 0;
        uint32_t conflict = 0;
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const bool cell = ids[o] >= 0;
            const bool mine = cell && (old[o] == -1 || old[o] == ids[o]);
            claimed += (cell && old[o] == -1) ? 1 : 0;
            conflict |= (cell && !mine) ? (1u << o) : 0u;
            const float m = mine ? 1.0f : 0.0f;
            atomicAdd(&vals[h[o]], m * acc[o][0]);
            atomicAdd(&vals[kTab + h[o]], m * acc[o][1]);
            atomicAdd(&vals[2 * kTab + h[o]], m * acc[o][2]);
        }
        if (claimed) atomicAdd(count, claimed);
        if (conflict) {
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                if (conflict & (1u << o)) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        unsafeAtomicAdd(A.grad + grad_slot(ids[o], 1 + q, A.n_cells), acc[o][q]);
                }
            }
        }
    }

    // The same for component q of the eight cells alone, by the lane of a quad
    // that holds it (`on`: not the lane that repeats another's, which goes the
    // same way and adds zeros).
    __device__ __forceinline__ void add8(const AdjointArgs& A, const int ids[8], const float acc[8], int q, bool on)
    {
        int h[8], old[8];
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            h[o] = (int)(((uint32_t)ids[o] * 2654435761u) >> (32 - 8));
            old[o] = ids[o] >= 0 ? atomicCAS(&keys[h[o]], -1, ids[o]) : ids[o];
        }
        int claimed = 0;
        uint32_t conflict = 0;
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const bool cell = ids[o] >= 0;
            const bool mine = cell && (old[o] == -1 || old[o] == ids[o]);
            claimed += (cell && old[o] == -1) ? 1 : 0;
            conflict |= (cell && !mine) ? (1u << o) : 0u;
            atomicAdd(&vals[q * kTab + h[o]], mine && on ? acc[o] : 0.0f);
        }
        if (claimed) atomicAdd(count, claimed);
        if (conflict) {
#pragma unroll
            for (int o = 0; o < 8; ++o)
                if (conflict & (1u << o))
                    unsafeAtomicAdd(A.grad + grad_slot(ids[o], 1 + q, A.n_cells), on ? acc[o] : 0.0f);
        }
    }
};
static_assert(kTab == 256, "the slot hash takes the top 8 bits");

// Per-lane accumulator of the gradient cotangents of the 8 cells of the
// current stencil: 24 words in LDS (component q of corner o is word 8 q + o;
// quad k at sum[64 k] of the wave's part), to which a step's stages are added
// once per step, and which enters the wave's table when the lane's stencil
// changes.  Only the lane itself touches its words: they are read, added to
// and written back (LDS float atomics on them cost 50 cycles each).
constexpr int kSumWords = 24;

struct Scatter {
    float4* sum;
    int cur;            // the stencil's lowest corner, -1: none

    // lds: kSumWords * kBlock floats of the block
    __device__ __forceinline__ void init(float* lds)
    {
        sum = reinterpret_cast<float4*>(lds) + (threadIdx.x >> 6) * (64 * kSumWords / 4) + (threadIdx.x & 63);
        cur = -1;
#pragma unroll
        for (int k = 0; k < kSumWords / 4; ++k) sum[64 * k] = make_float4(0.f, 0.f, 0.f, 0.f);
    }

    // the sums to the table, the accumulator empty
    __device__ __forceinline__ void flush(const AdjointArgs& A, WaveTable& T)
    {
        if (cur < 0) return;
        const int4* p = reinterpret_cast<const int4*>(A.c.grid.dual_ids + 8 * (int64_t)cur);
        const int4 a = p[0], b = p[1];
        const int ids[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        float acc[8][3];
#pragma unroll
        for (int k = 0; k < kSumWords / 4; ++k) {
            const float4 v = sum[64 * k];
            const int o = 4 * (k & 1), q = k >> 1;
            acc[o][q] = v.x; acc[o + 1][q] = v.y; acc[o + 2][q] = v.z; acc[o + 3][q] = v.w;
            sum[64 * k] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        T.add8(A, ids, acc);
        cur = -1;
    }

    // The stages' cotangents G of the interpolated gradient at offsets t in
    // the stencils base, last stage first.  A pass adds every lane's leading
    // stages that share its current stencil; the lanes with stages left
    // flush, take the next stage's stencil and go round again, which a wave
    // does once in most steps (a lane's stages rarely meet three stencils).
    __device__ __forceinline__ void add(const AdjointArgs& A, WaveTable& T, const int (&base)[4],
                                        const float (&t)[4][3], const float (&G)[4][3])
    {
        int next = 3;           // first stage not yet added
        while (next >= 0) {
            const int b = next == 3 ? base[3] : next == 2 ? base[2] : next == 1 ? base[1] : base[0];
            if (b != cur) {
                flush(A, T);
                cur = b;
            }
            float acc[3][8];
#pragma unroll
            for (int k = 0; k < kSumWords / 4; ++k) {
                const float4 v = sum[64 * k];
                float* c = acc[k >> 1] + 4 * (k & 1);
                c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
            }
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                if (next == i && base[i] == b) {
                    float w[8];
                    cic_weights(t[i], w);
#pragma unroll
                    for (int o = 0; o < 8; ++o)
#pragma unroll
                        for (int q = 0; q < 3; ++q) acc[q][o] = fmaf(w[o], G[i][q], acc[q][o]);
                    next = i - 1;
                }
            }
#pragma unroll
            for (int k = 0; k < kSumWords / 4; ++k) {
                const float* c = acc[k >> 1] + 4 * (k & 1);
                sum[64 * k] = make_float4(c[0], c[1], c[2], c[3]);
            }
        }
    }
};

// Direct atomics of a Phi cotangent onto the 8 cells of a stencil.
__device__ __forceinline__ void scatter_phi(const AdjointArgs& A, int base, const double t[3], double v)
{
    if (v == 0.0) return;
    const int32_t* ids = A.c.grid.dual_ids + 8 * (int64_t)base;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        const double w = ((o & 1) ? t[0] : 1.0 - t[0]) * ((o & 2) ? t[1] : 1.0 - t[1]) *
                         ((o & 4) ? t[2] : 1.0 - t[2]);
        const int id = ids[o];
        if (id >= 0) unsafeAtomicAdd(A.grad + grad_slot(id, 0, A.n_cells), (float)(w * v));
    }
}

// Step length and landing decision at the start of a step, exactly as the
// forward kernels take them; the field there (stage 0 of the step) into s0.
template <class FC>
__device__ __forceinline__ bool plan_step(const CastArgs& a, FC& F, const RayGeom& geo,
                                          const GeoState& y, double eta_s, double& ds, double& dl, bool& landing,
                                          Stage0& s0)
{
    const GridDev& g = a.grid;
    double v[FC::kComp];
    grid_coords<FC::kComp>(g, geo, y.eta, y.dx, v);
    int L;
    s0.bad = F.eval(g, v, s0.G, L, s0.l);
    if (L < 0) return false;
    ds = step_length(a, L);
    dl = quotient(ds, y.K);
    landing = fma(-y.K, dl, y.eta) < eta_s;
    return true;
}

// One forward step (regular or landing) from y, as in the forward kernels;
// records the stages of the final RK4 pass into rec when record is set.  Returns the
// affine length of the step taken through dl_taken.
template <class FC, class Rec, bool UNROLL>
__device__ __forceinline__ bool forward_step(const CastArgs& a, FC& F, const RayGeom& geo,
                                             const GeoState& y, double eta_s, GeoState& yn, Rec& rec, bool record,
                                             double& dl_taken, double& ds_out, bool& landing)
{
    double ds, dl;
    Stage0 s0;
    if (!plan_step(a, F, geo, y, eta_s, ds, dl, landing, s0)) return false;
    uint32_t h = 0;
    ds_out = ds;
    if (__builtin_expect(!landing, 1)) {
        // the recorder of stage 0 sees the lane's cache as plan_step left it
        if (rk4_step<FC, Rec, UNROLL>(a.grid, a.cosmo, F, geo, y, dl, yn, h, rec, record, &s0))
            return false;
        dl_taken = dl;
        return true;
    }
    // landing: two Newton passes for the step length, then the step (a
    // recorded pass evaluates its stage 0 again, since the passes before it
    // moved the lane's cache)
    double dlx = (y.eta - eta_s) / y.K;
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const bool rec_pass = record && k == 2;
        if (rk4_step<FC, Rec, UNROLL>(a.grid, a.cosmo, F, geo, y, dlx, yn, h, rec,
                                                   UNROLL ? record : rec_pass, rec_pass ? nullptr : &s0))
            return false;
        if (k < 2) dlx = dlx + (yn.eta - eta_s) / yn.K;
    }
    dl_taken = dlx;
    return true;
}

// Reverse of one RK4 step for the W cotangent columns of the Jacobian: the
// four stages are visited last to first; the jet of a stage is formed once and
// applied to every column.  For y' = y + dl/6 (F1 + 2 F2 + 2 F3 + F4) with
// Y_i = y + c_i dl F_{i-1} (c = 1/2, 1/2, 1):
//   Fbar_4 = dl/6 v,  Ybar_i = J_i^T Fbar_i,
//   Fbar_{i-1} = w_{i-1}/6 dl v + c_i dl Ybar_i,  ybar = v + sum_i Ybar_i,
//   dlbar = sum_i (w_i/6) v.F_i + sum_{i>1} c_i Ybar_i.F_{i-1}.
// Stage I (0-based) is handled with J holding its jet; the recursion moves
// to stage I - 1.
template <int I, int W, class Rec>
__device__ __forceinline__ void reverse_stage(const AdjointArgs& A, const RayCtx& R, const Rec& rec,
                                              const HubbleCubic& Hc, float dlf, Jet32& J,
                                              const Phys32 (&v)[W], Phys32 (&Fb)[W], float (&dlbar)[W],
                                              Phys32 (&dy)[W])
{
    Jet32 P;
    Phys32 FP;
    if constexpr (I > 0) {
        rec.template jet<I - 1>(A.c.cosmo, R, Hc, P);
        FP = rhs32(P);
    }
    constexpr float ci = (I == 3) ? 1.0f : 0.5f;
    constexpr float wprev = (I == 1) ? 1.0f : 2.0f;
#pragma unroll
    for (int c = 0; c < W; ++c) {
        Phys32 Yb;
        float Gb[3];
        rhs_vjp32(J, Fb[c], Yb, Gb);
        phys_axpy(dy[c], 1.0f, Yb);
        if constexpr (I > 0) {
            dlbar[c] += ci * phys_dot(Yb, FP) + (wprev * (1.0f / 6.0f)) * phys_dot(v[c], FP);
            phys_zero(Fb[c]);
            phys_axpy(Fb[c], wprev * (1.0f / 6.0f) * dlf, v[c]);
            phys_axpy(Fb[c], ci * dlf, Yb);
        }
    }
    if constexpr (I > 0) {
        J = P;
        rec.template gradient<I - 1>(A.c.grid, J);
        reverse_stage<I - 1, W>(A, R, rec, Hc, dlf, J, v, Fb, dlbar, dy);
    }
}

template <int W, class Rec>
__device__ __forceinline__ void reverse_step(const AdjointArgs& A, const RayCtx& R, const Rec& rec,
                                             const HubbleCubic& Hc, double dl,
                                             double ds_reg, double k0_step, Phys (&yb)[W])
{
    const float dlf = (float)dl;
    Phys32 v[W], Fb[W], dy[W];
    float dlbar[W];
    Jet32 J;
    rec.template jet<3>(A.c.cosmo, R, Hc, J);
    rec.template gradient<3>(A.c.grid, J);
    {
        const Phys32 F4 = rhs32(J);
#pragma unroll
        for (int c = 0; c < W; ++c) {
            v[c] = to32(yb[c]);
            dlbar[c] = phys_dot(v[c], F4) * (1.0f / 6.0f);
            phys_zero(Fb[c]);
            phys_axpy(Fb[c], dlf * (1.0f / 6.0f), v[c]);
            phys_zero(dy[c]);
        }
    }
    reverse_stage<3, W>(A, R, rec, Hc, dlf, J, v, Fb, dlbar, dy);
    // the four stage increments, summed in single precision, enter the
    // double-precision cotangent once per step
#pragma unroll
    for (int c = 0; c < W; ++c) phys_axpy(yb[c], 1.0, dy[c]);
    // a regular step has dl = ds / |k0| with ds fixed by the leaf level
    if (ds_reg > 0.0) {
        const double f = ds_reg / (k0_step * k0_step);
#pragma unroll
        for (int c = 0; c < W; ++c) yb[c].k0 += (double)dlbar[c] * f;
    }
}

// Spatial part of the transposed stage Jacobian for one column: the gradient's
// cotangent contracted with the stencil's coefficients (one trilinear scalar),
// then its derivatives, in place of the nine derivatives of the gradient.
__device__ __forceinline__ void gradient_vjp(const GridDev& g, int base, int lvl, const float t[3], const float Gb[3],
                                             float x[3])
{
    float c[24], k[8];
    stencil_coefs(g, base, c);
#pragma unroll
    for (int i = 1; i < 8; ++i) k[i] = fmaf(Gb[2], c[16 + i], fmaf(Gb[1], c[8 + i], Gb[0] * c[i]));
    const float scale = ldexpf((float)g.inv_h0, lvl);
    const float tx = t[0], ty = t[1], tz = t[2];
    x[0] = scale * fmaf(tz, fmaf(ty, k[7], k[5]), fmaf(ty, k[4], k[1]));
    x[1] = scale * fmaf(tz, fmaf(tx, k[7], k[6]), fmaf(tx, k[4], k[2]));
    x[2] = scale * fmaf(ty, fmaf(tx, k[7], k[6]), fmaf(tx, k[5], k[3]));
}

// The same for the loss's single column.  As Fbar_i = dl times the bracket of
// F_i in dlbar, dlbar = sum_i F_i.Fbar_i / dl.
template <int I>
__device__ __forceinline__ void reverse_loss_stage(const AdjointArgs& A, const RayCtx& R, RegRecord& rec, float dlf,
                                                   const Phys32& v6, Phys32& Fb, float& dlbar, Phys32& dy)
{
    Jet32 J;
    rec.template jet<I>(R, J);
    dlbar += phys_dot(Fb, rhs32(J));
    Phys32 Yb;
    float Gb[3];
    rhs_vjp32<false>(J, Fb, Yb, Gb);
    float x[3];
    gradient_vjp(A.c.grid, J.base, J.lvl, J.t, Gb, x);
#pragma unroll
    for (int l = 0; l < 3; ++l) Yb.x[l] = x[l];
    rec.template put_gbar<I>(Gb);
    phys_axpy(dy, 1.0f, Yb);
    if constexpr (I > 0) {
        constexpr float wprev = (I == 1) ? 1.0f : 2.0f;
        const float cdl = (I == 3) ? dlf : 0.5f * dlf;
        Fb.eta = fmaf(cdl, Yb.eta, wprev * v6.eta);
        Fb.k0 = fmaf(cdl, Yb.k0, wprev * v6.k0);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            Fb.x[i] = fmaf(cdl, Yb.x[i], wprev * v6.x[i]);
            Fb.k[i] = fmaf(cdl, Yb.k[i], wprev * v6.k[i]);
        }
        reverse_loss_stage<I - 1>(A, R, rec, dlf, v6, Fb, dlbar, dy);
    }
}

__device__ __forceinline__ void reverse_loss_step(const AdjointArgs& A, const RayCtx& R, RegRecord& rec, double dl,
                                                  double ds_reg, double K, Phys& yb)
{
    const float dlf = (float)dl;
    Phys32 v6, dy;
    phys_zero(v6);
    phys_axpy(v6, dlf * (1.0f / 6.0f), to32(yb));
    phys_zero(dy);
    Phys32 Fb = v6;
    float dlbar = 0.0f;
    reverse_loss_stage<3>(A, R, rec, dlf, v6, Fb, dlbar, dy);
    phys_axpy(yb, 1.0, dy);
    // a regular step has dl = ds / |k0| with ds fixed by the leaf level:
    // k0bar += dlbar ds / k0^2 = (dlbar dl) / |k0|, in double precision
    if (ds_reg > 0.0) yb.k0 += quotient((double)dlbar, K);
}

// Rays without a derivative (not stopped on the source surface, or a replay
// that did not retrace the forward path, which only happens when the cell
// values changed after the cast) get NaN in the per-ray derivative outputs.
__device__ __forceinline__ void write_nan_jacobian(const AdjointArgs& A, int64_t ray)
{
    const float q = __builtin_nanf("");
    if (A.jac) {
#pragma unroll
        for (int i = 0; i < 4; ++i) A.jac[4 * ray + i] = q;
    }
    if (A.dz_dtheta) {
        A.dz_dtheta[2 * ray] = q;
        A.dz_dtheta[2 * ray + 1] = q;
    }
}

// e1 = e_phi, e2 = -e_theta at the direction v
__device__ __forceinline__ void screen_basis(const double v[3], double e1[3], double e2[3])
{
    const double ph = atan2(v[1], v[0]);
    const double th = atan2(hypot(v[0], v[1]), v[2]);
    double sp, cp, st, ct;
    sincos(ph, &sp, &cp);
    sincos(th, &st, &ct);
    e1[0] = -sp; e1[1] = cp; e1[2] = 0.0;
    e2[0] = -cp * ct; e2[1] = -sp * ct; e2[2] = st;
}

// Double-precision interpolation jet at one point (end point and observer):
// Phi, its gradient, grad Phi and the right-hand side there.
struct PointJet {
    double phi, gphi[3], G[3], t[3];
    Phys F;
};

__device__ __forceinline__ void point_jet(const AdjointArgs& A, const RayCtx& R, const GeoState& ys, int base,
                                          int lvl, const HubbleCubic& Hc, PointJet& P)
{
    const GridDev& g = A.c.grid;
    stage_offsets(g, R, ys, lvl, P.t);
    const float4* rec = g.dual + 8 * (int64_t)base;
    double c[4][8];             // phi, gx, gy, gz
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        const float4 q = rec[o];
        double* k = c[(o / 2 + 1) & 3] + 4 * (o & 1);
        k[0] = q.x; k[1] = q.y; k[2] = q.z; k[3] = q.w;
    }
    const double scale = (double)(1 << lvl) * g.inv_h0;
    double fx, fy, fz;
    trilinear_jet<double>(c[0], P.t[0], P.t[1], P.t[2], P.phi, fx, fy, fz);
    P.gphi[0] = fx * scale; P.gphi[1] = fy * scale; P.gphi[2] = fz * scale;
#pragma unroll
    for (int j = 0; j < 3; ++j) trilinear_jet<double>(c[j + 1], P.t[0], P.t[1], P.t[2], P.G[j], fx, fy, fz);
    const double H = Hc(A.c.cosmo, ys.eta);
    const double k0 = -ys.K;
    double k[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) k[i] = ys.K * (R.geo.n[i] + (double)ys.d[i]);
    const double psi = P.G[0] * k[0] + P.G[1] * k[1] + P.G[2] * k[2];
    P.F.eta = k0;
    P.F.k0 = -2.0 * H * k0 * k0 - 2.0 * psi * k0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        P.F.x[j] = k[j];
        P.F.k[j] = -2.0 * H * k0 * k[j] + 2.0 * psi * k[j] - 2.0 * P.G[j] * k0 * k0;
    }
}

// Cotangents of the state at the end point yf (on the source surface):
// the beta_a columns, or the loss column from dL/dalpha and dL/dz5; the
// direct Phi_s term of the loss is scattered to the end point's stencil (end_base) and
// the Phi_o term returned.  The landing step has its length set by
// eta(y_f) = eta_s, so the cotangent along the flow F(y_f) is removed.
template <int W, bool SCATTER>
__device__ __forceinline__ void end_cotangents(const AdjointArgs& A, const RayCtx& R, int end_base, int end_lvl,
                                               const ObsDev& ob, int64_t ray, bool owner, const GeoState& yf, double phio,
                                               const double e1[3], const double e2[3], Phys (&yb)[W],
                                               double& phio_bar, double& phis_bar)
{
    const GridDev& g = A.c.grid;
    HubbleCubic Hf;
    Hf.init(A.c.cosmo, yf.eta);
    PointJet Jf;
    point_jet(A, R, yf, end_base, end_lvl, Hf, Jf);
    const double* n = R.geo.n;
    double r[3];
    const double sf = g.eta0 - yf.eta;
#pragma unroll
    for (int i = 0; i < 3; ++i) r[i] = sf * n[i] + (double)yf.dx[i];
    const double chi = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    const double rh[3] = {r[0] / chi, r[1] / chi, r[2] / chi};
    double f1[3], f2[3];
    screen_basis(rh, f1, f2);
    const double phis = Jf.phi;
    const double a_s = A.c.ray_stop ? A.c.ray_stop[ray].y : ob.a_s;
    const double dz_dK = a_s * (1.0 + phis) / (1.0 + phio);
    const double dz_dphis = a_s * yf.K / (1.0 + phio);
    const double dz_dphio = -a_s * yf.K * (1.0 + phis) / ((1.0 + phio) * (1.0 + phio));
#pragma unroll
    for (int c = 0; c < W; ++c) phys_zero(yb[c]);
    if constexpr (W == 2) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            yb[0].x[i] = f1[i] / chi;
            yb[1].x[i] = f2[i] / chi;
        }
    }
    phio_bar = phis_bar = 0.0;
    if (SCATTER) {
        const float ga0 = A.dL_dalpha ? A.dL_dalpha[2 * ray] : 0.0f;
        const float ga1 = A.dL_dalpha ? A.dL_dalpha[2 * ray + 1] : 0.0f;
        const double gz = A.dL_dz ? A.dL_dz[ray] : 0.0;
        // alpha = -f(sigma) t, t = r^ - (r^.n) n, sin sigma = |t|, f = sigma / sin sigma;
        // d alpha_a / d r^ . e~_b = -f e_a.e~_b + (f'/sin sigma)(e_a.t)(n.e~_b)
        const double cth = rh[0] * n[0] + rh[1] * n[1] + rh[2] * n[2];
        double t[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) t[i] = rh[i] - cth * n[i];
        const double st = sqrt(t[0] * t[0] + t[1] * t[1] + t[2] * t[2]);
        const double sig = atan2(st, cth);
        double fs, fps;           // f and f'/sin sigma (series below 1e-3 rad)
        if (sig < 1e-3) {
            fs = 1.0 + sig * sig / 6.0;
            fps = 1.0 / 3.0 + sig * sig * (2.0 / 15.0);
        } else {
            fs = sig / st;
            fps = (st - sig * cth) / (st * st * st);
        }
        const double ga[2] = {ga0, ga1};
        const double* ea[2] = {e1, e2};
        const double* fb[2] = {f1, f2};
        double cb[2] = {0.0, 0.0};
#pragma unroll
        for (int aa = 0; aa < 2; ++aa) {
            const double et = ea[aa][0] * t[0] + ea[aa][1] * t[1] + ea[aa][2] * t[2];
#pragma unroll
            for (int bb = 0; bb < 2; ++bb) {
                const double ee = ea[aa][0] * fb[bb][0] + ea[aa][1] * fb[bb][1] + ea[aa][2] * fb[bb][2];
                const double ne = n[0] * fb[bb][0] + n[1] * fb[bb][1] + n[2] * fb[bb][2];
                cb[bb] += ga[aa] * (-fs * ee + fps * et * ne);
            }
        }
        Phys& L = yb[0];
#pragma unroll
        for (int i = 0; i < 3; ++i) L.x[i] = (cb[0] * f1[i] + cb[1] * f2[i]) / chi + gz * dz_dphis * Jf.gphi[i];
        L.k0 = -gz * dz_dK;
        phis_bar = gz * dz_dphis;
        if (owner) scatter_phi(A, end_base, Jf.t, phis_bar);
        phio_bar = gz * dz_dphio;
    }
#pragma unroll
    for (int c = 0; c < W; ++c) yb[c].eta -= phys_dot(yb[c], Jf.F) / Jf.F.eta;
}

// A ray's sweep: its observer, stop surface and start.
template <class FC>
struct Sweep {
    static constexpr int C = FC::kComp;
    RayCtx R;           // the components this lane holds
    FC F;
    const ObsDev* ob;
    double eta_s, phio, kmag, e1[3], e2[3];
    int obs_base, obs_lvl, N, nseg;

    __device__ __forceinline__ void start(const AdjointArgs& A, int64_t ray, int n_steps, float* lds)
    {
        const CastArgs& a = A.c;
        int j = a.n_obs - 1;
        while (j > 0 && a.obs[j].ray_first > ray) --j;
        ob = a.obs + j;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            R.geo.vo[i] = ldexp(ob->x[FC::own_axis(i)] / a.grid.h0, a.grid.max_level + 1);
            R.geo.n[i] = a.dirs[3 * ray + FC::own_axis(i)];
        }
        eta_s = a.ray_stop ? a.ray_stop[ray].x : ob->eta_s;
        if constexpr (C == 3) F.bind(lds);
        F.reset();
        // potential at the observer and the initial |k| (as in the forward)
        int ll;
        F.locate(a.grid, R.geo.vo, ll);
        obs_base = F.base;
        obs_lvl = F.lvl;
        phio = (double)F.phi(a.grid);
        kmag = sqrt((1.0 + 2.0 * phio) / (1.0 - 2.0 * phio));
        screen_basis(a.dirs + 3 * ray, e1, e2);
        N = n_steps;
        nseg = (N + a.ckpt_every - 1) / a.ckpt_every;
    }

    // all components of the geometry
    __device__ __forceinline__ void whole(const AdjointArgs& A, int64_t ray, RayCtx& W) const
    {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            W.geo.vo[i] = ldexp(ob->x[i] / A.c.grid.h0, A.c.grid.max_level + 1);
            W.geo.n[i] = A.c.dirs[3 * ray + i];
        }
    }

    // makes the stencil at y the current one
    __device__ __forceinline__ void locate(const GridDev& g, const GeoState& y)
    {
        int ll;
        double v[C];
        grid_coords<C>(g, R.geo, y.eta, y.dx, v);
        F.locate(g, v, ll);
    }
};

// The replay must end where the forward cast ended, bit for bit.
__device__ __forceinline__ bool retraced(const RayEnd& e, const GeoState& y)
{
    return y.eta == e.eta && y.dx[0] == e.dx[0] && y.dx[1] == e.dx[1] && y.dx[2] == e.dx[2];
}

// The distortion matrix by the reverse sweep: the two columns beta_1 and
// beta_2 of the rays A.list (the finder's Newton steps; the other products take
// the tangents of cast_tangent_kernel), for more rays than adjoint_quad_kernel
// takes.
template <bool AMR>
__global__ __launch_bounds__(kBlock, 1) void adjoint_kernel(AdjointArgs A)
{
    // LDS: stencil coefficients, then the stage records
    extern __shared__ float lds[];
    const CastArgs& a = A.c;
    int64_t at;
    if (!lane_ray(a, A.n_list, at)) return;
    const int64_t ray = A.list[at];
    constexpr int W = 2;
    if (A.status[ray] != MPATH_RAY_REACHED || A.n_steps[ray] <= 0) {
        write_nan_jacobian(A, ray);
        return;
    }
    Sweep<FieldCache<AMR>> w;
    w.start(A, ray, A.n_steps[ray], lds);
    const int K = a.ckpt_every;
    Phys yb[W];
    // Segments from the source back to the observer.  Each is traversed
    // forwards from its checkpoint (storing the state before every step in
    // the tape; the last step of a segment other than the final one is not
    // needed, its result being the next checkpoint), then backwards with the
    // stages of every step re-recorded and reversed.  One loop with a single
    // step call site serves both directions.
    bool ok = true;
    // the tape entry of the next reverse step and the next segment's
    // checkpoint are loaded one iteration ahead of their use
    GeoState pre, ck = a.ckpt[(int64_t)(w.nseg - 1) * a.n_rays + ray];
    for (int seg = w.nseg - 1; seg >= 0 && ok; --seg) {
        const bool last = seg == w.nseg - 1;
        const int j0 = seg * K;
        const int len = min(w.N, j0 + K) - j0;
        const int nf = last ? len : len - 1;
        GeoState y = ck, yin = ck;
        for (int it = 0; it < nf + len; ++it) {
            const bool fwd = it < nf;
            if (it == nf) {
                // the state before the segment's last step is in registers
                pre = last ? yin : y;
                if (seg > 0) ck = a.ckpt[(int64_t)(seg - 1) * a.n_rays + ray];
                if (last) {
                    if (!retraced(a.ends[ray], y)) {
                        ok = false;
                        break;
                    }
                    double none;
                    w.locate(a.grid, y);
                    end_cotangents<W, false>(A, w.R, w.F.base, w.F.lvl, *w.ob, ray, false, y, w.phio, w.e1, w.e2, yb,
                                             none, none);
                }
            }
            const int jl = fwd ? it : len - 1 - (it - nf);
            GeoState ys;
            if (fwd) {
                A.tape[(int64_t)jl * a.n_rays + ray] = y;
                ys = y;
                yin = y;
            } else {
                ys = pre;
                if (jl > 0) pre = A.tape[(int64_t)(jl - 1) * a.n_rays + ray];
            }
            LdsRecord rec;
            rec.p = lds + FieldCache<AMR>::kFloats * kBlock + threadIdx.x;
            GeoState yn;
            double dl, ds;
            bool landing;
            if (!forward_step<FieldCache<AMR>, LdsRecord, false>(a, w.F, w.R.geo, ys, w.eta_s, yn, rec, !fwd, dl, ds, landing)) {
                ok = false;
                break;
            }
            if (fwd) {
                y = yn;
            } else {
                HubbleCubic Hc;
                Hc.init(a.cosmo, ys.eta);
                reverse_step<W>(A, w.R, rec, Hc, dl, landing ? 0.0 : ds, -ys.K, yb);
            }
        }
    }
    if (!ok) {
        write_nan_jacobian(A, ray);
        return;
    }
    // the initial state: k = kmag(Phi_o) n (theta), k0 = -1
    const double* eb[2] = {w.e1, w.e2};
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
        const double db0 = w.kmag * (yb[0].k[0] * eb[bb][0] + yb[0].k[1] * eb[bb][1] + yb[0].k[2] * eb[bb][2]);
        const double db1 = w.kmag * (yb[1].k[0] * eb[bb][0] + yb[1].k[1] * eb[bb][1] + yb[1].k[2] * eb[bb][2]);
        A.jac[4 * ray + bb] = (float)db0;          // row beta_1
        A.jac[4 * ray + 2 + bb] = (float)db1;      // row beta_2
    }
}

// The cell cotangents of the loss L by the reverse sweep of its one column.
// The stage records are not in LDS and the scatter sums take 96 bytes of it a
// lane, so that two waves fit a SIMD (one did with the records in LDS and the
// Jacobian's columns alongside), which hides most of the gather and table
// latency, and the traffic of what the 256 registers do not hold: the compiler
// spills 105 (uniform) or 120 (tree) registers, 143 and 171 with SPREAD, 396 to
// 516 bytes a lane.  131,072 rays to z = 1 on a uniform 64^3 grid (3,000 steps)
// 80.3 ms before, 34.6 now, 27 of them without the scatter; with the Jacobian
// (15 ms of tangents) 80.5 and 49.6.  Fewer rays than fill one wave per SIMD by
// four lanes each take adjoint_quad_kernel.  SPREAD: waves of fewer than 64 rays (see lane_ray).
template <bool AMR, bool SPREAD>
__global__ __launch_bounds__(kBlock, 2) void adjoint_loss_kernel(AdjointArgs A)
{
    // LDS: stencil coefficients, scatter sums, one table per wave
    extern __shared__ float lds[];
    WaveTable T;
    T.bind(lds + (FieldCache<AMR>::kFloats + kSumWords) * kBlock + (threadIdx.x >> 6) * kTabWords);
    T.clear(threadIdx.x & 63);
    const CastArgs& a = A.c;
    int64_t ray = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    bool owner = true;          // the lanes that repeat another's ray add nothing to the cells
    if constexpr (SPREAD) {
        if (!lane_ray(a, a.n_rays, ray)) return;
        owner = (int)(threadIdx.x & 63) < min((int64_t)a.lanes, a.n_rays - (ray & -(int64_t)a.lanes));
    } else {
        if (ray >= a.n_rays) return;
    }
    const int n_steps = A.n_steps[ray];
    if (A.status[ray] != MPATH_RAY_REACHED || n_steps <= 0) {
        write_nan_jacobian(A, ray);
        if (A.ray_status) A.ray_status[ray] = 1;
        return;
    }
    const GridDev& g = a.grid;
    Sweep<FieldCache<AMR>> w;
    w.start(A, ray, n_steps, lds);
    const int K = a.ckpt_every;
    Phys yb[1];
    double phio_bar = 0.0;
    Scatter S;
    S.init(lds + FieldCache<AMR>::kFloats * kBlock);
    NoRecord none;
    bool ok = true;
    // segments from the source back to the observer: forwards from the
    // checkpoint into the tape (the last step of a segment other than the
    // final one is not needed), then backwards, re-recording every step
    GeoState ck = a.ckpt[(int64_t)(w.nseg - 1) * a.n_rays + ray];
    for (int seg = w.nseg - 1; seg >= 0 && ok; --seg) {
        const bool last = seg == w.nseg - 1;
        const int j0 = seg * K;
        const int len = min(w.N, j0 + K) - j0;
        GeoState y = ck, pre = ck;
        double dl, ds;
        bool landing;
        for (int it = 0; it < len; ++it) {
            pre = y;                      // the state before the segment's last step, in the end
            if (it == len - 1 && !last) break;
            A.tape[(int64_t)it * a.n_rays + ray] = y;
            GeoState yn;
            if (!forward_step<FieldCache<AMR>, NoRecord, true>(a, w.F, w.R.geo, y, w.eta_s, yn, none, false, dl, ds, landing)) {
                ok = false;
                break;
            }
            y = yn;
        }
        if (!ok) break;
        if (seg > 0) ck = a.ckpt[(int64_t)(seg - 1) * a.n_rays + ray];
        if (last) {
            if (!retraced(a.ends[ray], y)) {
                ok = false;
                break;
            }
            w.locate(a.grid, y);
            double phis_bar;
            end_cotangents<1, true>(A, w.R, w.F.base, w.F.lvl, *w.ob, ray, owner, y, w.phio, w.e1, w.e2, yb, phio_bar,
                                    phis_bar);
        }
        for (int jl = len - 1; jl >= 0; --jl) {
            // the lanes still iterating empty the table when it is a quarter full
            if (*T.count > kTab / 4) T.evict(A);
            const GeoState ys = pre;
            // the tape entry of the next step is loaded one step ahead of its use
            if (jl > 0) pre = A.tape[(int64_t)(jl - 1) * a.n_rays + ray];
            RegRecord rec;
            GeoState yn;
            if (!forward_step<FieldCache<AMR>, RegRecord, true>(a, w.F, w.R.geo, ys, w.eta_s, yn, rec, true, dl, ds, landing)) {
                ok = false;
                break;
            }
            reverse_loss_step(A, w.R, rec, dl, landing ? 0.0 : ds, ys.K, yb[0]);
            if (owner) S.add(A, T, rec.base, rec.t, rec.G);
        }
    }
    if (!ok) write_nan_jacobian(A, ray);
    if (A.ray_status && !(ok && A.checked)) A.ray_status[ray] = ok ? 0 : 2;
    if (ok && owner) {
        S.flush(A, T);
        // the initial state: k = kmag(Phi_o) n (theta), k0 = -1
        const double* n = w.R.geo.n;
        const double dkmag = w.kmag * 2.0 / (1.0 - 4.0 * w.phio * w.phio);
        phio_bar += (yb[0].k[0] * n[0] + yb[0].k[1] * n[1] + yb[0].k[2] * n[2]) * dkmag;
        GeoState y0;
        y0.eta = g.eta0;
        y0.K = 1.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) { y0.d[i] = 0.0f; y0.dx[i] = 0.0f; }
        double t0[3];
        stage_offsets(g, w.R, y0, w.obs_lvl, t0);
        scatter_phi(A, w.obs_base, t0, phio_bar);
    }
    // every lane that took a ray arrives here together: empty the table
    T.evict(A);
}

// ---------------------------------------------------------------------------
// The loss's column with four lanes per ray (QuadRay), for few rays: a SIMD
// then holds one wave whichever way, and the length of a step's instruction
// sequence decides.  Every lane replays and reverses its own component, with
// the stages' coefficients kept from the replay and the scatter sums of its
// component in registers, and shares the scalars.  The start and the end of a
// ray run on whole vectors in all four lanes alike.  Without LOSS, the
// matrix's columns of the rays A.list: the replay likewise, then each lane
// reverses one column (the first lane beta_1, the others beta_2) on whole
// vectors, with the operations of adjoint_kernel.
// ---------------------------------------------------------------------------
struct QuadRecord {
    float K[4], H[4], dH[4], d[4], G[4], t[4];
    float4 p[4], q[4];
    int base[4], lvl[4];

    template <class FC>
    __device__ __forceinline__ void stage(int i, const GeoState&, const GeoState& yi, const FC& F, const float* g,
                                          const HubbleCubic& Hc, const CosmoDev& cz)
    {
        K[i] = (float)yi.K;
        H[i] = (float)Hc(cz, yi.eta);
        dH[i] = (float)Hc.deriv(cz, yi.eta);
        d[i] = yi.d[0];
        G[i] = g[0];
        t[i] = F.t;
        p[i] = F.p;
        q[i] = F.q;
        base[i] = F.base;
        lvl[i] = FC::kUniform ? 0 : F.lvl;
    }

    // the stage's jet on whole vectors, each lane giving its component (R: own)
    template <int I>
    __device__ __forceinline__ void jet(const CosmoDev&, const RayCtx& R, const HubbleCubic&, Jet32& J) const
    {
        J.k0 = -K[I];
        const float k = K[I] * ((float)R.geo.n[0] + d[I]);
        QuadRay::whole_vector(&k, J.k);
        QuadRay::whole_vector(&G[I], J.G);
        QuadRay::whole_vector(&t[I], J.t);
        J.H = H[I];
        J.dH = dH[I];
        J.base = base[I];
        J.lvl = lvl[I];
    }

    template <int I>
    __device__ __forceinline__ void gradient(const GridDev& g, Jet32& J) const
    {
        const float4 a = p[I], b = q[I];
        const float c[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        float row[3];
        gradient_row(c, J.t, (float)((double)(1 << J.lvl) * g.inv_h0), row);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            float col[3];
            QuadRay::whole_vector(&row[l], col);
            J.JG[0][l] = col[0]; J.JG[1][l] = col[1]; J.JG[2][l] = col[2];
        }
    }
};

// A state or cotangent: the scalars and one component.
struct QuadPhys {
    float eta, x, k0, k;
};

// Stage I and those before it (reverse_loss_stage); the sums over the axes are
//   psi = G.k, bk = Fb.k.k, bG = Fb.k.G, bx = Fb.x.k.
template <int I>
__device__ __forceinline__ void quad_loss_stage(float nf, float inv_h0, QuadRecord& rec, float dlf, const QuadPhys& v6,
                                                QuadPhys Fb, float& dlbar, QuadPhys& dy)
{
    const float k0 = -rec.K[I], k = rec.K[I] * (nf + rec.d[I]), G = rec.G[I], H = rec.H[I];
    const float a = Fb.k0;
    auto sum = [](float v) { return QuadRay::sum(&v); };
    const float psi = sum(G * k), bk = sum(Fb.k * k), bG = sum(Fb.k * G), bx = sum(Fb.x * k);
    const float f = -2.0f * H * k0 + 2.0f * psi;            // F_k = f k - 2 G k0^2
    dlbar += Fb.eta * k0 + a * (-2.0f * H * k0 * k0 - 2.0f * psi * k0) + bx + f * bk - 2.0f * k0 * k0 * bG;
    const float u = 2.0f * (bk - k0 * a);
    const float Gb = u * k - 2.0f * k0 * k0 * Fb.k;
    QuadPhys Yb;
    Yb.eta = -2.0f * rec.dH[I] * k0 * (a * k0 + bk);
    Yb.k0 = Fb.eta + a * (-4.0f * H * k0 - 2.0f * psi) - 2.0f * H * bk - 4.0f * k0 * bG;
    Yb.k = Fb.x + u * G + f * Fb.k;
    // the derivatives of this lane's component along the three axes times its
    // cotangent, summed over the components; each lane takes its own axis
    const float tx = QuadRay::of<0>(rec.t[I]), ty = QuadRay::of<1>(rec.t[I]), tz = QuadRay::of<2>(rec.t[I]);
    const float4 p = rec.p[I], q = rec.q[I];
    const float e = fmaf(tz, q.w, q.x);
    const float gs = Gb * ldexpf(inv_h0, rec.lvl[I]);
    const float x0 = sum(gs * fmaf(tz, q.y, fmaf(ty, e, p.y)));
    const float x1 = sum(gs * fmaf(tz, q.z, fmaf(tx, e, p.z)));
    const float x2 = sum(gs * fmaf(ty, q.z, fmaf(tx, fmaf(ty, q.w, q.y), p.w)));
    const int ax = QuadRay::own_axis(0);
    Yb.x = ax == 0 ? x0 : ax == 1 ? x1 : x2;
    rec.G[I] = Gb;              // its place takes the gradient's cotangent
    dy.eta += Yb.eta; dy.k0 += Yb.k0; dy.x += Yb.x; dy.k += Yb.k;
    if constexpr (I > 0) {
        constexpr float wprev = (I == 1) ? 1.0f : 2.0f;
        const float cdl = (I == 3) ? dlf : 0.5f * dlf;
        Fb.eta = fmaf(cdl, Yb.eta, wprev * v6.eta);
        Fb.k0 = fmaf(cdl, Yb.k0, wprev * v6.k0);
        Fb.x = fmaf(cdl, Yb.x, wprev * v6.x);
        Fb.k = fmaf(cdl, Yb.k, wprev * v6.k);
        quad_loss_stage<I - 1>(nf, inv_h0, rec, dlf, v6, Fb, dlbar, dy);
    }
}

// Scatter's accumulator of one component.
struct QuadScatter {
    float sum[8];
    int cur;

    __device__ __forceinline__ void flush(const AdjointArgs& A, WaveTable& T)
    {
        if (cur >= 0) {
            const int4* p = reinterpret_cast<const int4*>(A.c.grid.dual_ids + 8 * (int64_t)cur);
            const int4 a = p[0], b = p[1];
            const int ids[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            T.add8(A, ids, sum, QuadRay::own_axis(0), (threadIdx.x & 3) != 3);
        }
#pragma unroll
        for (int o = 0; o < 8; ++o) sum[o] = 0.0f;
    }

    __device__ __forceinline__ void add(const AdjointArgs& A, WaveTable& T, const QuadRecord& rec)
    {
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            float t[3], w[8];
            QuadRay::whole_vector(&rec.t[i], t);
            cic_weights(t, w);
            if (rec.base[i] != cur) {
                flush(A, T);
                cur = rec.base[i];
            }
#pragma unroll
            for (int o = 0; o < 8; ++o) sum[o] = fmaf(w[o], rec.G[i], sum[o]);
        }
    }
};

// a quad's part of a stored state
__device__ __forceinline__ GeoState own_state(const GeoState& s)
{
    const int ax = QuadRay::own_axis(0);
    GeoState y;
    y.eta = s.eta;
    y.K = s.K;
    y.d[0] = s.d[ax];
    y.dx[0] = s.dx[ax];
    return y;
}

template <bool AMR, bool LOSS>
__global__ __launch_bounds__(kBlock, 1) void adjoint_quad_kernel(AdjointArgs A)
{
    extern __shared__ float lds[];
    using FC = QuadCache<AMR>;
    const CastArgs& a = A.c;
    const int64_t n = LOSS ? a.n_rays : A.n_list;
    WaveTable T;
    if constexpr (LOSS) {
        T.bind(lds + (threadIdx.x >> 6) * kTabWords);
        T.clear(threadIdx.x & 63);
    }
    int64_t at;
    if (!lane_ray<4>(a, n, at)) return;
    const int64_t ray = LOSS ? at : A.list[at];
    const int n_steps = A.n_steps[ray];
    if (A.status[ray] != MPATH_RAY_REACHED || n_steps <= 0) {
        write_nan_jacobian(A, ray);
        if (LOSS && A.ray_status) A.ray_status[ray] = 1;
        return;
    }
    // the quads that repeat another's ray add nothing to the cells
    const bool owner = (int)(threadIdx.x & 63) / 4 < min((int64_t)a.lanes, n - (at & -(int64_t)a.lanes));
    const int ax = FC::own_axis(0);
    const GridDev& g = a.grid;
    Sweep<FC> w;
    w.start(A, ray, n_steps, nullptr);
    const float nf = (float)w.R.geo.n[0], inv_h0 = (float)g.inv_h0;
    const int K = a.ckpt_every;
    double yb_eta = 0.0, yb_k0 = 0.0, yb_x = 0.0, yb_k = 0.0;     // LOSS: this component
    Phys yb[1];                                                  // else this column
    double phio_bar = 0.0, phis_bar = 0.0;
    QuadScatter S;
    S.cur = -1;
    if constexpr (LOSS) S.flush(A, T);
    NoRecord none;
    bool ok = true;
    GeoState ck = own_state(a.ckpt[(int64_t)(w.nseg - 1) * a.n_rays + ray]);
    for (int seg = w.nseg - 1; seg >= 0 && ok; --seg) {
        const bool last = seg == w.nseg - 1;
        const int j0 = seg * K;
        const int len = min(w.N, j0 + K) - j0;
        GeoState y = ck, pre = ck;
        double dl, ds;
        bool landing;
        for (int it = 0; it < len; ++it) {
            pre = y;                      // the state before the segment's last step, in the end
            if (it == len - 1 && !last) break;
            GeoState& e = A.tape[(int64_t)it * a.n_rays + ray];
            e.eta = y.eta;
            e.K = y.K;
            e.d[ax] = y.d[0];
            e.dx[ax] = y.dx[0];
            GeoState yn;
            if (!forward_step<FC, NoRecord, true>(a, w.F, w.R.geo, y, w.eta_s, yn, none, false, dl, ds, landing)) {
                ok = false;
                break;
            }
            y = yn;
        }
        if (!ok) break;
        if (seg > 0) ck = own_state(a.ckpt[(int64_t)(seg - 1) * a.n_rays + ray]);
        if (last) {
            GeoState ye;
            ye.eta = y.eta;
            ye.K = y.K;
            FC::whole_vector(y.d, ye.d);
            FC::whole_vector(y.dx, ye.dx);
            if (!retraced(a.ends[ray], ye)) {
                ok = false;
                break;
            }
            w.locate(g, y);
            RayCtx R;
            w.whole(A, ray, R);
            if constexpr (LOSS) {
                end_cotangents<1, true>(A, R, w.F.base, w.F.lvl, *w.ob, ray, false, ye, w.phio, w.e1, w.e2, yb,
                                        phio_bar, phis_bar);
                yb_eta = yb[0].eta;
                yb_k0 = yb[0].k0;
                yb_x = ax == 0 ? yb[0].x[0] : ax == 1 ? yb[0].x[1] : yb[0].x[2];
                yb_k = ax == 0 ? yb[0].k[0] : ax == 1 ? yb[0].k[1] : yb[0].k[2];
            } else {
                Phys c[2];
                end_cotangents<2, false>(A, R, w.F.base, w.F.lvl, *w.ob, ray, false, ye, w.phio, w.e1, w.e2, c,
                                         phio_bar, phis_bar);
                yb[0] = ax == 0 ? c[0] : c[1];
            }
        }
        for (int jl = len - 1; jl >= 0; --jl) {
            if constexpr (LOSS) {
                if (*T.count > kTab / 4) T.evict(A);
            }
            const GeoState ys = pre;
            // the tape entry of the next step is loaded one step ahead of its use
            if (jl > 0) pre = own_state(A.tape[(int64_t)(jl - 1) * a.n_rays + ray]);
            QuadRecord rec;
            GeoState yn;
            if (!forward_step<FC, QuadRecord, true>(a, w.F, w.R.geo, ys, w.eta_s, yn, rec, true, dl, ds, landing)) {
                ok = false;
                break;
            }
            if constexpr (!LOSS) {
                HubbleCubic Hc;
                reverse_step<1>(A, w.R, rec, Hc, dl, landing ? 0.0 : ds, -ys.K, yb);
                continue;
            }
            const float dlf = (float)dl, s6 = dlf * (1.0f / 6.0f);
            const QuadPhys v6 = {s6 * (float)yb_eta, s6 * (float)yb_x, s6 * (float)yb_k0, s6 * (float)yb_k};
            QuadPhys dy = {0.0f, 0.0f, 0.0f, 0.0f};
            float dlbar = 0.0f;
            quad_loss_stage<3>(nf, inv_h0, rec, dlf, v6, v6, dlbar, dy);
            yb_eta += (double)dy.eta;
            yb_k0 += (double)dy.k0;
            yb_x += (double)dy.x;
            yb_k += (double)dy.k;
            if (!landing) yb_k0 += quotient((double)dlbar, ys.K);
            if (owner) S.add(A, T, rec);
        }
    }
    if (!ok) write_nan_jacobian(A, ray);
    if constexpr (!LOSS) {
        if (!ok) return;
        // the initial state: k = kmag(Phi_o) n (theta), k0 = -1
        const double* eb[2] = {w.e1, w.e2};
#pragma unroll
        for (int bb = 0; bb < 2; ++bb) {
            const double v = w.kmag * (yb[0].k[0] * eb[bb][0] + yb[0].k[1] * eb[bb][1] + yb[0].k[2] * eb[bb][2]);
            A.jac[4 * ray + (ax == 0 ? 0 : 2) + bb] = (float)v;         // row beta_1 or beta_2
        }
        return;
    }
    if (A.ray_status && !(ok && A.checked)) A.ray_status[ray] = ok ? 0 : 2;
    if (ok && owner) {
        S.flush(A, T);
        // the initial state: k = kmag(Phi_o) n (theta), k0 = -1
        const double dkmag = w.kmag * 2.0 / (1.0 - 4.0 * w.phio * w.phio);
        const double kn = yb_k * w.R.geo.n[0];
        const int q0 = threadIdx.x & 60;
        phio_bar += (__shfl(kn, q0) + __shfl(kn, q0 + 1) + __shfl(kn, q0 + 2)) * dkmag;
        RayCtx R;
        w.whole(A, ray, R);
        GeoState y0;
        y0.eta = g.eta0;
        y0.K = 1.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) { y0.d[i] = 0.0f; y0.dx[i] = 0.0f; }
        double t0[3];
        stage_offsets(g, R, y0, w.obs_lvl, t0);
        // Phi at the end point: after the loops, since with one lane of a quad
        // branching off inside them the compiler (ROCm 7.2) once spilled a pointer
        // before the other lanes were switched on again, and those then read
        // from wherever their register pointed.  Any branch of some lanes can
        // meet that; build.py searches every build's assembly for it.
        GeoState ye;
        const RayEnd e = a.ends[ray];
        ye.eta = e.eta;
        double te[3];
        GeoState yo = ye;
        yo.dx[0] = e.dx[ax];
        w.locate(g, yo);
#pragma unroll
        for (int i = 0; i < 3; ++i) ye.dx[i] = e.dx[i];
        stage_offsets(g, R, ye, w.F.lvl, te);
        if ((threadIdx.x & 3) == 0) {
            scatter_phi(A, w.obs_base, t0, phio_bar);
            scatter_phi(A, w.F.base, te, phis_bar);
        }
    }
    T.evict(A);
}

// The check of a Jacobian: `ends` are the end states of the cast that carried
// the tangents.  A ray that did not reach the source has no derivative; one that
// ended elsewhere than the forward cast is reported.  A loss sweep after it
// (AdjointArgs::checked) leaves that report: its own replay starts from the
// stored checkpoints and misses values that changed before the last one.
__global__ __launch_bounds__(256) void retrace_kernel(AdjointArgs A, const RayEnd* __restrict__ ends)
{
    const int64_t ray = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (ray >= A.c.n_rays) return;
    int st = 1;
    if (A.status[ray] == MPATH_RAY_REACHED && A.n_steps[ray] > 0) {
        GeoState y;
        const RayEnd e = ends[ray];
        y.eta = e.eta;
        y.dx[0] = e.dx[0]; y.dx[1] = e.dx[1]; y.dx[2] = e.dx[2];
        st = retraced(A.c.ends[ray], y) ? 0 : 2;
    }
    if (st) write_nan_jacobian(A, ray);
    if (A.ray_status) A.ray_status[ray] = st;
}

__global__ void fill_zero_kernel(float* __restrict__ p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// Cell cotangents from the workspace layout to the caller's order and
// layout [n][4] (overwrites).
__global__ void scatter_grad_kernel(const float* __restrict__ g_lib, const int64_t* __restrict__ perm,
                                    float4* __restrict__ out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[perm[i]] = make_float4(g_lib[grad_slot(i, 0, n)], g_lib[grad_slot(i, 1, n)], g_lib[grad_slot(i, 2, n)],
                               g_lib[grad_slot(i, 3, n)]);
}

// On a uniform periodic grid whose gradient is the central difference of the
// potential, g_d[c] = (Phi[c + e_d] - Phi[c - e_d]) / (2 h0), the total
// cotangent of Phi is the direct one plus the transposed difference operator
// applied to the cotangents of g:
//   dL/dPhi[c] += sum_d (gbar_d[c - e_d] - gbar_d[c + e_d]) / (2 h0).
__global__ void central_transpose_kernel(const float* __restrict__ g_lib, const int64_t* __restrict__ perm,
                                         float* __restrict__ out, int n0, double inv_2h, int64_t n)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    // the id of a coarse cell is its Morton index
    const int3 p = make_int3((int)compact1by2((uint32_t)c), (int)compact1by2((uint32_t)c >> 1),
                             (int)compact1by2((uint32_t)c >> 2));
    const uint32_t m = (uint32_t)n0 - 1u;
    auto id = [m](int i, int j, int k) { return (int64_t)morton3((uint32_t)i & m, (uint32_t)j & m, (uint32_t)k & m); };
    auto gq = [&](int64_t cell, int q) { return (double)g_lib[grad_slot(cell, q, n)]; };
    double acc = gq(c, 0);
    acc += (gq(id(p.x - 1, p.y, p.z), 1) - gq(id(p.x + 1, p.y, p.z), 1)) * inv_2h;
    acc += (gq(id(p.x, p.y - 1, p.z), 2) - gq(id(p.x, p.y + 1, p.z), 2)) * inv_2h;
    acc += (gq(id(p.x, p.y, p.z - 1), 3) - gq(id(p.x, p.y, p.z + 1), 3)) * inv_2h;
    out[perm[c]] = (float)acc;
}

}  // namespace

hipError_t launch_adjoint(const AdjointArgs& args, hipStream_t s)
{
    if (args.n_list == 0) return hipSuccess;
    AdjointArgs A = args;
    // four lanes a ray while that leaves a SIMD one wave: the matrix step of
    // a finder of 4,096 sources (uniform 64^3) 13.8 ms with one lane, 5.6 with four
    if (by_quads(args.c, args.n_list, 1)) {
        A.c = spread_rays(args.c, args.n_list, 1, 16);
        const dim3 quads = ray_grid(A.c, A.n_list);
        if (A.c.grid.max_level > 0) hipLaunchKernelGGL((adjoint_quad_kernel<true, false>), quads, dim3(kBlock), 0, s, A);
        else hipLaunchKernelGGL((adjoint_quad_kernel<false, false>), quads, dim3(kBlock), 0, s, A);
        return hipGetLastError();
    }
    A.c = spread_rays(args.c, args.n_list, 1);
    const dim3 grid = ray_grid(A.c, A.n_list), block(kBlock);
    const size_t lds = (size_t)(FieldCache<true>::kFloats + 4 * LdsRecord::kWords) * kBlock * sizeof(float);
    if (A.c.grid.max_level > 0) hipLaunchKernelGGL(adjoint_kernel<true>, grid, block, lds, s, A);
    else hipLaunchKernelGGL(adjoint_kernel<false>, grid, block, lds, s, A);
    return hipGetLastError();
}

hipError_t launch_adjoint_loss(const AdjointArgs& args, hipStream_t s)
{
    const int64_t n = args.c.n_rays;
    if (n == 0) return hipSuccess;
    AdjointArgs A = args;
    // Four lanes a ray while that leaves a SIMD one wave (the kernel takes all
    // its registers): 3,072 rays to z = 0.3 on a uniform 64^3 grid 7.6 ms with one
    // lane, 3.9 with four, 16,384 9.1 and 5.0, 24,576 10.1 and 10.0; 64^3 + 5
    // levels 6.0 and 3.6, 8.2 and 5.4, 8.7 and 7.8.
    if (by_quads(args.c, n, 1)) {
        A.c = spread_rays(args.c, n, 1, 16);
        const size_t tab = (size_t)(kBlock / 64) * kTabWords * sizeof(float);
        if (A.c.grid.max_level > 0)
            hipLaunchKernelGGL((adjoint_quad_kernel<true, true>), ray_grid(A.c, n), dim3(kBlock), tab, s, A);
        else hipLaunchKernelGGL((adjoint_quad_kernel<false, true>), ray_grid(A.c, n), dim3(kBlock), tab, s, A);
        return hipGetLastError();
    }
    A.c = spread_rays(args.c, n, 1);
    const dim3 grid = ray_grid(A.c, n), block(kBlock);
    const size_t lds = ((size_t)(FieldCache<true>::kFloats + kSumWords) * kBlock +
                        (size_t)(kBlock / 64) * kTabWords) * sizeof(float);
    const bool amr = A.c.grid.max_level > 0;
    if (A.c.lanes < 64) {
        if (amr) hipLaunchKernelGGL((adjoint_loss_kernel<true, true>), grid, block, lds, s, A);
        else hipLaunchKernelGGL((adjoint_loss_kernel<false, true>), grid, block, lds, s, A);
    } else {
        if (amr) hipLaunchKernelGGL((adjoint_loss_kernel<true, false>), grid, block, lds, s, A);
        else hipLaunchKernelGGL((adjoint_loss_kernel<false, false>), grid, block, lds, s, A);
    }
    return hipGetLastError();
}

hipError_t launch_retrace(const AdjointArgs& A, const RayEnd* ends, hipStream_t s)
{
    const int64_t n = A.c.n_rays;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(retrace_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, A, ends);
    return hipGetLastError();
}

hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_scatter_grad(const float* grad_lib, const int64_t* perm, float4* out_user, int64_t n,
                               hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_grad_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, grad_lib, perm,
                       out_user, n);
    return hipGetLastError();
}

hipError_t launch_central_transpose(const float* g_lib, const int64_t* perm, float* out, int n0, double h0,
                                    int64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(central_transpose_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g_lib, perm,
                       out, n0, 0.5 / h0, n);
    return hipGetLastError();
}

}  // namespace mpath
