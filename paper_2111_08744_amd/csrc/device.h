// device.h -- device-side building blocks of the ray tracer: HEALPix
// directions, the tabulated conformal Hubble rate, octree lookups with the
// AMR level fallback and a lane-resident stencil cache, and one RK4 step of
// the null geodesic equations in the split FP64/FP32 representation.
#pragma once

#include <type_traits>

#include "internal.h"

namespace mpath {

constexpr uint32_t kFnvOffset = 2166136261u;
constexpr int kBlock = 256;       // threads per block of the integration kernels
constexpr uint32_t kFnvPrime = 16777619u;

__device__ __forceinline__ uint32_t fnv(uint32_t h, uint32_t v) { return (h ^ v) * kFnvPrime; }

// The GPU hands consecutive workgroups to its 8 XCDs in turn, and each XCD
// has its own L2.  Renumber workgroups so that each XCD runs a contiguous
// range of them (consecutive rays are neighbouring sky pixels whose paths
// share cells): XCD x = b mod 8 takes logical blocks
// [start(x), start(x) + count(x)) in the order it receives them.
constexpr int kNumXcd = 8;

__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nblocks)
{
    const int64_t q = nblocks / kNumXcd, r = nblocks % kNumXcd;
    const int64_t x = b % kNumXcd, idx = b / kNumXcd;
    return x < r ? x * (q + 1) + idx : r * (q + 1) + (x - r) * q + idx;
}

// Rays per wave of a launch of n rays: `most` (64 lanes' worth), or fewer where that leaves SIMDs without a
// wave: the smallest power of two that needs at most `waves` waves per SIMD.
// A stage stalls the wave when any of its rays enters a new stencil, so waves
// of fewer rays run a step sooner; beyond one wave per SIMD the additional
// instructions cost more than that saves, except where the stalls are long (a
// tree's walk, the 27 cells of TSC), which two waves per SIMD hide better.
// Uniform 64^3, 3,072 rays to z = 0.3: 64 rays a wave 2.01 ms, 8 1.70, 4 (768
// waves) 1.65, 2 (1,536) 2.01; 6,144 rays on 64^3 + 5 levels: 1.97, 1.73, 4
// (1,536 waves) 1.57; TSC there 5.14, 4.19, 3.34.
inline CastArgs spread_rays(const CastArgs& a, int64_t n, int waves, int most = 64)
{
    CastArgs c = a;
    c.lanes = most;
    while (c.lanes > 1 && (n + c.lanes / 2 - 1) / (c.lanes / 2) <= (int64_t)waves * a.simds) c.lanes /= 2;
    return c;
}

// Whether n rays of four lanes each (QuadRay) need at most `waves` waves per
// SIMD; the launchers say how many are worth it.
inline bool by_quads(const CastArgs& a, int64_t n, int waves) { return n <= (int64_t)16 * a.simds * waves; }

inline dim3 ray_grid(const CastArgs& a, int64_t n)
{
    const int64_t per = (int64_t)(kBlock / 64) * a.lanes;
    return dim3((unsigned)((n + per - 1) / per));
}

// Ray (of n) of this lane in the one-ray-per-lane launches: every wave takes a.lanes
// (a power of two) consecutive rays; its other lanes, and those past the last
// ray, run copies of them, which write the same values to the same places.
// (A wave that masks them off instead, with 8 lanes or fewer active and the
// SIMD to itself, was measured to run at half the speed.)  False for a wave
// without rays.
template <int LANES = 1>
__device__ __forceinline__ bool lane_ray(const CastArgs& a, int64_t n, int64_t& r)
{
    const int64_t wave = xcd_block(blockIdx.x, gridDim.x) * (kBlock / 64) + (threadIdx.x >> 6);
    r = wave * a.lanes;
    if (r >= n) return false;
    r += threadIdx.x / LANES & (a.lanes - 1);
    if (r >= n) r = n - 1;
    return true;
}

// ---------------------------------------------------------------------------
// HEALPix NESTED pixel centre (Gorski et al. 2005; Sect. 2.4 starts one photon
// at every pixel centre).  Within base face f the nested index interleaves
// the face coordinates (x in the even bits, y in the odd bits); the ring
// counted from the north pole is jr = (2 + f/4) nside - x - y - 1; the
// azimuth is pi/4 (jpll + (x - y)/nr) with jpll = 2 (f mod 4) + 1 on the
// polar faces and 2 (f mod 4) on the equatorial ones.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t compact1by1(uint32_t x)
{
    x &= 0x55555555u;
    x = (x ^ (x >> 1)) & 0x33333333u;
    x = (x ^ (x >> 2)) & 0x0f0f0f0fu;
    x = (x ^ (x >> 4)) & 0x00ff00ffu;
    x = (x ^ (x >> 8)) & 0x0000ffffu;
    return x;
}

__device__ inline void healpix_nest_dir(int64_t nside, int64_t pix, double v[3])
{
    const int64_t npface = nside * nside;
    const int face = (int)(pix / npface);
    const uint32_t ip = (uint32_t)(pix - (int64_t)face * npface);
    const int64_t x = compact1by1(ip), y = compact1by1(ip >> 1);
    const int64_t jr = (int64_t)(2 + face / 4) * nside - x - y - 1;
    const int jpll = 2 * (face & 3) + ((face >> 2) != 1 ? 1 : 0);
    const double three_ns2 = 3.0 * (double)nside * (double)nside;
    int64_t nr;
    double z, st;
    if (jr < nside) {
        nr = jr;
        const double one_minus_z = (double)(nr * nr) / three_ns2;
        z = 1.0 - one_minus_z;
        st = sqrt(one_minus_z * (2.0 - one_minus_z));
    } else if (jr > 3 * nside) {
        nr = 4 * nside - jr;
        const double one_plus_z = (double)(nr * nr) / three_ns2;
        z = one_plus_z - 1.0;
        st = sqrt(one_plus_z * (2.0 - one_plus_z));
    } else {
        nr = nside;
        z = (double)(2 * nside - jr) * 2.0 / (3.0 * (double)nside);
        st = sqrt((1.0 - z) * (1.0 + z));
    }
    const double ph = 0.25 * M_PI * ((double)jpll + (double)(x - y) / (double)nr);
    double sp, cp;
    sincos(ph, &sp, &cp);
    v[0] = st * cp;
    v[1] = st * sp;
    v[2] = z;
}

// Conformal Hubble rate a'/a over one RK4 step: the cubic of the table
// interval holding the step's start (coefficients in tau = the position in
// the interval, tabulated per interval), which the sub-steps (|eta - eta_n| <=
// one step, less than the table spacing) evaluate with four FMAs.  Outside
// its interval the cubic deviates from the interpolant of the neighbouring
// interval by O(h^4 d4H/deta4) ~ 1e-18.
struct HubbleCubic {
    double c0, c1, c2, c3;   // H = c0 + tau (c1 + tau (c2 + tau c3))
    double off;              // tau = eta inv_deta + off

    __device__ __forceinline__ void init(const CosmoDev& c, double eta)
    {
        #pragma clang fp contract(off)
        // a static background has inv_deta = 0 and zeros in interval 0
        int i = (int)fma(eta, c.inv_deta, c.eta_off);
        i = i < 0 ? 0 : (i > c.n - 2 ? c.n - 2 : i);
        off = c.eta_off - (double)i;
        const double2 lo = c.cubic[2 * i], hi = c.cubic[2 * i + 1];
        c0 = lo.x; c1 = lo.y; c2 = hi.x; c3 = hi.y;
    }

    __device__ __forceinline__ double operator()(const CosmoDev& c, double eta) const
    {
        #pragma clang fp contract(off)
        const double tau = fma(eta, c.inv_deta, off);
        return fma(tau, fma(tau, fma(tau, c3, c2), c1), c0);
    }

    // d(a'/a)/d eta of the same cubic
    __device__ __forceinline__ double deriv(const CosmoDev& c, double eta) const
    {
        const double tau = fma(eta, c.inv_deta, off);
        return (c1 + tau * (2.0 * c2 + 3.0 * tau * c3)) * c.inv_deta;
    }
};

// Scale factor a(eta): cubic Hermite interpolation of the (a, da/deta) table
// on the nodes of the a'/a table (1 on a static background).
__device__ inline double scale_factor(const CosmoDev& c, double eta)
{
    if (c.is_static) return 1.0;
    const double u = (eta - c.eta_lo) * c.inv_deta;
    int i = (int)floor(u);
    i = i < 0 ? 0 : (i > c.n - 2 ? c.n - 2 : i);
    const double t = u - (double)i;
    const double2 p0 = c.atable[i];
    const double2 p1 = c.atable[i + 1];
    const double a0 = p0.x, a1 = c.deta * p0.y;
    const double a2 = fma(-c.deta, fma(2.0, p0.y, p1.y), 3.0 * (p1.x - p0.x));
    const double a3 = fma(c.deta, p0.y + p1.y, 2.0 * (p0.x - p1.x));
    return fma(t, fma(t, fma(t, a3, a2), a1), a0);
}

// ---------------------------------------------------------------------------
// Octree lookups.  Integer cell coordinates are kept unwrapped (a periodic
// ray may leave the box) and wrapped only to address memory.
// ---------------------------------------------------------------------------

// Interleaved coordinates m with `one` (0 or the axis's lowest bit) added to
// the axis whose bits are `lanes`, wrapping.
__host__ __device__ __forceinline__ uint32_t step_up(uint32_t m, uint32_t lanes, uint32_t one)
{
    return (m & ~lanes) | (((m | ~lanes) + one) & lanes);
}

// Id of cell (l, J) or -1 if it does not exist: coarse ancestor by Morton
// index, then one child link per level.
__host__ __device__ __forceinline__ int lookup_cell(const GridDev& g, int l, int J0, int J1, int J2)
{
    const int M = g.n0 << l;
    if (g.periodic) {
        J0 &= M - 1; J1 &= M - 1; J2 &= M - 1;
    } else if ((unsigned)J0 >= (unsigned)M || (unsigned)J1 >= (unsigned)M || (unsigned)J2 >= (unsigned)M) {
        return -1;
    }
    int id = (int)morton3((uint32_t)(J0 >> l), (uint32_t)(J1 >> l), (uint32_t)(J2 >> l));
    for (int m = l - 1; m >= 0; --m) {
        const int ch = g.child[id];
        if (ch < 0) return -1;
        id = ch + (((J0 >> m) & 1) | (((J1 >> m) & 1) << 1) | (((J2 >> m) & 1) << 2));
    }
    return id;
}

// Level of a cell id (ids are level-major; the levels past the deepest start
// past every id).  Unrolled in two parts, the second behind a uniform branch,
// so that a part's comparisons wait once for the level table in scalar
// registers.
__device__ __forceinline__ int level_of(const GridDev& g, int id)
{
    int l = 0;
#pragma unroll
    for (int k = 1; k <= 4; ++k) l += id >= g.level_start[k] ? 1 : 0;
    if (g.max_level > 4) {
#pragma unroll
        for (int k = 5; k < kMaxLevels; ++k) l += id >= g.level_start[k] ? 1 : 0;
    }
    return l;
}

// Stencil record of the 8 corner payloads v[o] (o = ox + 2 oy + 4 oz): per
// component (gx, gy, gz, phi) two float4 of trilinear coefficients,
// f(t) = c0 + c1 tx + c2 ty + c3 tz + c4 tx ty + c5 tx tz + c6 ty tz + c7 tx ty tz,
// which equals sum_o prod_d W_CIC(t_d - o_d) v[o] for t in [0, 1]^3.  A stage
// needs the gradient only: its 96 bytes come first.
__device__ __forceinline__ void stencil_record(const float4 v[8], float4 rec[8])
{
#define MPATH_TRI(f, k)                                                                       \
    {                                                                                         \
        const float c1 = v[1].f - v[0].f, c2 = v[2].f - v[0].f;                               \
        const float c4 = v[3].f - v[2].f - c1;                                                \
        rec[2 * k] = make_float4(v[0].f, c1, c2, v[4].f - v[0].f);                            \
        rec[2 * k + 1] = make_float4(c4, v[5].f - v[4].f - c1, v[6].f - v[4].f - c2,          \
                                     v[7].f - v[6].f - v[5].f + v[4].f - c4);                 \
    }
    MPATH_TRI(y, 0) MPATH_TRI(z, 1) MPATH_TRI(w, 2) MPATH_TRI(x, 3)
#undef MPATH_TRI
}

__device__ __forceinline__ float trilinear_eval(float c0, float c1, float c2, float c3, float c4, float c5,
                                                float c6, float c7, float tx, float ty, float tz)
{
    #pragma clang fp contract(off)
    const float a = fmaf(tz, c5, fmaf(ty, fmaf(tz, c7, c4), c1));
    const float b = fmaf(tz, c6, c2);
    return fmaf(tz, c3, fmaf(ty, b, fmaf(tx, a, c0)));
}

// How the lanes carry a ray's vectors.  WholeRay: one lane, all three
// components.  QuadRay: four lanes, one component each (the fourth repeats the
// third), everything that is no vector in all four; the lanes of a quad take
// every branch together, and a component reaches the others by a lane
// permutation within the quad.
struct WholeRay {
    static constexpr int kComp = 3;     // components a lane holds
    static __device__ __forceinline__ int own_axis(int i) { return i; }     // axis of its component i
    static __device__ __forceinline__ float dot(const float m[3], const float G[3])
    {
        return fmaf(m[2], G[2], fmaf(m[1], G[1], m[0] * G[0]));
    }
    static __device__ __forceinline__ float sum(const float v[3])
    {
        #pragma clang fp contract(off)
        return v[0] + v[1] + v[2];
    }
    template <class T>
    static __device__ __forceinline__ void whole_vector(const T v[3], T all[3])
    {
        all[0] = v[0]; all[1] = v[1]; all[2] = v[2];
    }
};

struct QuadRay {
    static constexpr int kComp = 1;
    template <int P0, int P1, int P2, int P3>
    static __device__ __forceinline__ uint32_t perm(uint32_t x)
    {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, P0 | P1 << 2 | P2 << 4 | P3 << 6, 0xf, 0xf, true);
    }
    // the value of component K, of the next one and of the one after
    template <int K>
    static __device__ __forceinline__ uint32_t of(uint32_t x) { return perm<K, K, K, K>(x); }
    template <int K>
    static __device__ __forceinline__ float of(float x) { return __uint_as_float(of<K>(__float_as_uint(x))); }
    template <int K>
    static __device__ __forceinline__ double of(double x)
    {
        return __hiloint2double((int)of<K>((uint32_t)__double2hiint(x)), (int)of<K>((uint32_t)__double2loint(x)));
    }
    static __device__ __forceinline__ uint32_t next(uint32_t x) { return perm<1, 2, 0, 0>(x); }
    static __device__ __forceinline__ uint32_t after(uint32_t x) { return perm<2, 0, 1, 1>(x); }
    static __device__ __forceinline__ uint32_t all_or(uint32_t x) { return x | next(x) | after(x); }

    static __device__ __forceinline__ int own_axis(int)
    {
        const int c = threadIdx.x & 3;
        return c < 2 ? c : 2;
    }
    static __device__ __forceinline__ float dot(const float m[1], const float G[1])
    {
        return fmaf(of<2>(m[0]), of<2>(G[0]), fmaf(of<1>(m[0]), of<1>(G[0]), of<0>(m[0]) * of<0>(G[0])));
    }
    static __device__ __forceinline__ float sum(const float v[1])
    {
        #pragma clang fp contract(off)
        return of<0>(v[0]) + of<1>(v[0]) + of<2>(v[0]);
    }
    template <class T>
    static __device__ __forceinline__ void whole_vector(const T v[1], T all[3])
    {
        all[0] = of<0>(v[0]); all[1] = of<1>(v[0]); all[2] = of<2>(v[0]);
    }
};

// Child link of a leaf whose stencil record (the 8 cells from it) consists of
// leaves of its own level only; every other leaf has -1.  A point inside such
// a dual cell is in a leaf of that level and takes that stencil, whichever of
// the 8 cells holds it.
constexpr int kWholeLeaf = -2;

// A cached region that is the stencil's dual cell (FieldCache::off).
constexpr uint32_t kDual = ~0u;

// Field value interpolated at one point, with the lane's cache of the last
// resolved 8-cell stencil (as trilinear coefficients) and of the region of
// points that resolve to it.
//
// Reuse is exact.  The leaf level of x only changes when x leaves its leaf
// cell, and for x inside a leaf cell of level L the CIC base at every level
// l <= L is a function of floor(x / h_{L+1}) alone (the half of the leaf cell
// x lies in per axis), so the resolved stencil is a function of the half-cell;
// the build precomputes it per half-cell.  Where all 8 cells of the stencil
// are leaves of its own level (kWholeLeaf; always so on a uniform grid), the
// whole dual cell between their centres shares it, and the region is that
// dual cell.  The region is a cube: u = v sc - kd is in [0, 1)^3 inside it.
// v is in double precision and v sc - kd rounds monotonically, so u < 0 means
// outside exactly; u is compared after its conversion to float, where a value
// just below 1 may become 1, which costs a second look-up and changes nothing.
// With a whole dual cell u is also the offset t in the stencil.
//
// The check takes 5 instructions a stage beyond the conversions of t that
// the weights need anyway (3 FMAs, a maximum of the bit patterns, one
// comparison: negative values and NaN compare above 1), in place of three
// floors, conversions, shifts and comparisons and the offsets' integer
// arithmetic, which were 40 of a stage's 145 VALU instructions.
//
// The coefficients live in LDS, quad o (four coefficients) of the wave's 64
// lanes in 64 consecutive float4, which is the layout that loads straight to
// LDS write (16 bytes a lane at consecutive places) and that 16-byte LDS reads
// take without bank conflicts.  A record thus passes through no registers,
// which leaves its loads all in flight at once; by way of registers they came
// in two batches, two memory latencies, for want of 24 free registers.
//
// TIME: the grid also carries dPhi/deta (Sect. 2.2, from a double-layer
// light cone); eval leaves the interpolated value in tv.  PHI: the
// coefficients of Phi are kept too (for a field evaluation whose Phi is
// needed at every step; else phi() reads them from the record).
template <bool AMR, bool TIME = false, bool PHI = false>
struct FieldCache : WholeRay {
    static constexpr bool kTime = TIME;
    static constexpr bool kUniform = !AMR;
    static constexpr int kComps = PHI ? 4 : 3;
    static constexpr int kQuads = 2 * kComps + (TIME ? 2 : 0);
    static constexpr int kFloats = 4 * kQuads;          // LDS words per lane
    int leafL;          // leaf level of the points of the cached region
    int lvl;            // level of the resolved stencil
    int base;           // id of its lowest corner cell
    uint32_t off, offz; // AMR, region a half-cell: its place in the stencil (see locate), x and y in
                        // 16 bits each; kDual: the region is the stencil's dual cell
    double kd[3], sc;   // the region
    float t[3];         // offsets of the last evaluated point in that stencil
    float4* c;          // quad o of this lane at c[64 o]: per component (gx, gy, gz[, phi]
                        // [, dphi/deta]) the coefficients c0..c3, then c4..c7
    float tv;           // TIME: dPhi/deta at the last evaluated point
    float isw_step;     // TIME: ISW increment of the last RK4 step (set by rk4_step)

    using LdsQuad = __attribute__((address_space(3))) float4;
    LdsQuad* wave;      // the wave's first float4 (uniform)

    // lds: kFloats * kBlock floats of the block
    __device__ __forceinline__ void bind(float* lds)
    {
        wave = (LdsQuad*)lds + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (64 * kQuads);
        c = reinterpret_cast<float4*>(lds) + (threadIdx.x >> 6) * (64 * kQuads) + (threadIdx.x & 63);
    }

    __device__ __forceinline__ void reset()
    {
        leafL = -1;
        lvl = 0;
        base = 0;
        off = kDual;
        sc = 0.0;
        kd[0] = kd[1] = kd[2] = __builtin_nan("");      // no point is inside
    }

    // coefficient quad o (0: c0..c3, 1: c4..c7) of component f
    __device__ __forceinline__ float4 quad(int f, int o) const { return c[64 * (2 * f + o)]; }

    // component i's coefficients, and the offsets along the three axes
    __device__ __forceinline__ void coefs(int i, float4& p, float4& q) const
    {
        p = quad(i, 0);
        q = quad(i, 1);
    }
    __device__ __forceinline__ void offsets(float o[3]) const { o[0] = t[0]; o[1] = t[1]; o[2] = t[2]; }

    __device__ __forceinline__ float tri(int f) const
    {
        const float4 p = quad(f, 0), q = quad(f, 1);
        return trilinear_eval(p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w, t[0], t[1], t[2]);
    }

    // N quads from src to this lane's quads O, O + 1, ... (asynchronous; see
    // wait).  The instruction's offset (16 k) moves source and destination
    // alike, lane l's 16 bytes going to the destination + 16 l.
    template <int O, int N, int K = 0>
    __device__ __forceinline__ void fetch(const float4* src)
    {
        using Src = const __attribute__((address_space(1))) void;
        using Dst = __attribute__((address_space(3))) void;
        __builtin_amdgcn_global_load_lds((Src*)src, (Dst*)(wave + 64 * (O + K) - K), 16, 16 * K, 0);
        if constexpr (K + 1 < N) fetch<O, N, K + 1>(src);
    }
    __device__ __forceinline__ void wait() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

    // u of the point in the cached region (w before its conversion); true when
    // it lies inside
    __device__ __forceinline__ bool inside(const double v[3], double w[3], float u[3]) const
    {
        #pragma clang fp contract(off)
        uint32_t m = 0u;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            w[d] = AMR ? fma(v[d], sc, -kd[d]) : fma(v[d], 0.5, -kd[d]);
            u[d] = (float)w[d];
            const uint32_t b = __float_as_uint(u[d]);
            m = b > m ? b : m;
        }
        return m < 0x3f800000u;
    }

    // Resolve the stencil of the point with fine-grid coordinates v: its
    // region, base and coefficients.  leaf receives the level of the deepest
    // cell containing the point (-1 outside a non-periodic box).  False when
    // no complete stencil exists even at level 0; the coefficients are then
    // zeros and nothing is cached.
    __device__ __forceinline__ bool find(const GridDev& g, const double v[3], int& leaf)
    {
        #pragma clang fp contract(off)
        const int Lm = AMR ? g.max_level : 0;
        int I[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) I[d] = (int)floor(v[d]);    // at level max_level + 1
        const int M = g.n0;
        // the coarse dual cell holding the point
        int bc[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) bc[d] = ((AMR ? I[d] >> Lm : I[d]) - 1) >> 1;
        bool ok = true;
        int L = 0, l = 0;
        if (!g.periodic) {
            ok = (unsigned)bc[0] < (unsigned)(M - 1) && (unsigned)bc[1] < (unsigned)(M - 1) &&
                 (unsigned)bc[2] < (unsigned)(M - 1);              // b + 1 must exist too
            const int Mh = 2 * (M << Lm);
            if ((unsigned)I[0] >= (unsigned)Mh || (unsigned)I[1] >= (unsigned)Mh || (unsigned)I[2] >= (unsigned)Mh)
                L = -1;
        }
        int b = (int)morton3((uint32_t)(bc[0] & (M - 1)), (uint32_t)(bc[1] & (M - 1)), (uint32_t)(bc[2] & (M - 1)));
        // Its record is requested together with its mark: most points of most
        // trees are in unrefined surroundings, and the record is then there
        // after one memory latency.  Otherwise the leaf is looked up and the
        // stencil of the half-cell taken from the table.
        fetch<0, 2 * kComps>(g.dual + 8 * (int64_t)b);
        bool w = true;
        if constexpr (AMR) w = ok && g.child[b] == kWholeLeaf;
        if (AMR && !w && L >= 0) {
            // the coarse cell: b, or the next one along the axes where the point is
            // in its lower half
            const uint32_t bits = (1u << (3 * __builtin_ctz((unsigned)M))) - 1u;
            uint32_t id = (uint32_t)b;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const uint32_t lanes = (0x49249249u << d) & bits;
                id = step_up(id, lanes, (uint32_t)(~(I[d] >> Lm) & 1) << d);
            }
            for (int m = Lm; m > 0; --m) {
                const int ch = g.child[id];
                if (ch < 0) break;
                id = ch + (((I[0] >> m) & 1) | (((I[1] >> m) & 1) << 1) | (((I[2] >> m) & 1) << 2));
                ++L;
            }
            // a point in a leaf of level 0 takes the level-0 stencil (or none at
            // the edge of a non-periodic box)
            if (L > 0) {
                const int sh = Lm - L;
                b = g.leafinfo[8 * (int64_t)((int)id - g.level_start[1]) +
                               (((I[0] >> sh) & 1) | (((I[1] >> sh) & 1) << 1) | (((I[2] >> sh) & 1) << 2))];
                ok = b >= 0;
                if (ok) {
                    l = level_of(g, b);
                    w = l > 0 && g.child[b] == kWholeLeaf;
                    wait();
                    fetch<0, 2 * kComps>(g.dual + 8 * (int64_t)b);
                }
            }
        }
        leaf = L;
        if (!ok) {
            wait();
#pragma unroll
            for (int o = 0; o < kQuads; ++o) c[64 * o] = make_float4(0.f, 0.f, 0.f, 0.f);
            t[0] = t[1] = t[2] = 0.0f;
            reset();
            return false;
        }
        if constexpr (AMR) {
            const int sh = w ? Lm - l : Lm - L;
            // u = v 2^-sh - k in the half-cell k, u = v 2^-(sh + 1) - (b + 1/2)
            // in the dual cell, b + 1/2 = ((k - 1) | 1) / 2
            sc = ldexp(1.0, w ? -sh - 1 : -sh);
            int k[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) k[d] = I[d] >> sh;
            off = kDual;
            if (w) {
#pragma unroll
                for (int d = 0; d < 3; ++d) kd[d] = 0.5 * (double)((k[d] - 1) | 1);
            } else {
                // half-cell k of the leaf's level L; the stencil's lowest centre is
                // half-cell boundary 2^(s + 1) b + 2^s, b = ((k >> s) - 1) >> 1
                const int s = L - l;
                uint32_t o[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    kd[d] = (double)k[d];
                    o[d] = (uint32_t)(k[d] - ((((k[d] >> s) - 1) | 1) << s));
                }
                off = o[0] | o[1] << 16;
                offz = o[2];
            }
        } else {
#pragma unroll
            for (int d = 0; d < 3; ++d) kd[d] = (double)bc[d] + 0.5;
        }
        leafL = L;
        lvl = l;
        base = b;
        if constexpr (TIME) fetch<2 * kComps, 2>(g.tdual + 2 * (int64_t)b);
        wait();
        return true;
    }

    // Make the stencil of the point with fine-grid coordinates v = x / h_f,
    // h_f = h0 / 2^(max_level + 1), the current one and set its offsets t.
    // Returns false when no complete stencil exists.
    __device__ __forceinline__ bool locate(const GridDev& g, const double v[3], int& leaf_level)
    {
        #pragma clang fp contract(off)
        double w[3];
        float u[3];
        bool ok = true;
        leaf_level = leafL;
        if (!inside(v, w, u)) {
            ok = find(g, v, leaf_level);
            if (ok) (void)inside(v, w, u);
            else u[0] = u[1] = u[2] = 0.0f;
        }
        t[0] = u[0]; t[1] = u[1]; t[2] = u[2];
        if constexpr (AMR) {
            if (off != kDual) {
                // the half-cell's place counted from the stencil's lowest centre
                // in half-cells, and the point's in it, in units of 2^(s + 1)
                // half-cells (the sum in double precision: one rounding, to t)
                const int e = lvl - leafL - 1;
                t[0] = ldexpf((float)(w[0] + (double)(off & 0xffffu)), e);
                t[1] = ldexpf((float)(w[1] + (double)(off >> 16)), e);
                t[2] = ldexpf((float)(w[2] + (double)offz), e);
            }
        }
        return ok;
    }

    // Leaf level at the point with fine-grid coordinates v, -1 outside a
    // non-periodic box.
    __device__ __forceinline__ int leaf(const GridDev& g, const double v[3])
    {
        int L;
        (void)locate(g, v, L);
        return L;
    }

    // grad Phi at the point with fine-grid coordinates v (CIC, Eq. W_CIC,
    // with the level fallback).  Returns 0, or 1 when no complete stencil
    // exists (G is then zero).  leaf_level and stencil_level receive the
    // levels of the deepest cell containing the point and of the stencil.
    __device__ __forceinline__ int eval(const GridDev& g, const double v[3], float G[3], int& leaf_level,
                                        int& stencil_level)
    {
        const bool ok = locate(g, v, leaf_level);
        stencil_level = AMR ? lvl : 0;
        // the coefficients are read from LDS at every stage: without this the
        // compiler carries all of them in registers from one stage to the next
        asm volatile("" ::: "memory");
        // f = c0 + tx (c1 + ty (c4 + tz c7) + tz c5) + ty (c2 + tz c6) + tz c3
        G[0] = tri(0);
        G[1] = tri(1);
        G[2] = tri(2);
        if constexpr (TIME) tv = tri(kComps);
        return ok ? 0 : 1;
    }

    // Phi at the last evaluated point
    __device__ __forceinline__ float phi(const GridDev& g) const
    {
        if constexpr (PHI) return tri(3);
        const float4 p = g.dual[8 * (int64_t)base + 6], q = g.dual[8 * (int64_t)base + 7];
        return trilinear_eval(p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w, t[0], t[1], t[2]);
    }
};

// FieldCache for a ray carried by four lanes: the same regions, look-ups and
// arithmetic, component by component.  A lane evaluates one component of the
// gradient, whose eight coefficients it keeps in registers.
template <bool AMR>
struct QuadCache : QuadRay {
    static constexpr bool kTime = false;
    static constexpr bool kUniform = !AMR;
    int leafL, lvl, base;   // as in FieldCache
    uint32_t off;           // this axis's
    double kd, sc;
    float t;                // this axis
    float4 p, q;            // coefficients c0..c3, c4..c7 of this axis's component

    __device__ __forceinline__ void reset()
    {
        leafL = -1;
        lvl = 0;
        base = 0;
        off = kDual;
        sc = 0.0;
        kd = __builtin_nan("");
    }

    __device__ __forceinline__ void coefs(int, float4& a, float4& b) const
    {
        a = p;
        b = q;
    }
    __device__ __forceinline__ void offsets(float o[3]) const { o[0] = of<0>(t); o[1] = of<1>(t); o[2] = of<2>(t); }

    __device__ __forceinline__ bool inside(double v, double& w, float& u) const
    {
        #pragma clang fp contract(off)
        w = AMR ? fma(v, sc, -kd) : fma(v, 0.5, -kd);
        u = (float)w;
        uint32_t m = __float_as_uint(u);
        const uint32_t n = next(m);
        const uint32_t a = after(m);
        m = n > m ? n : m;
        m = a > m ? a : m;
        return m < 0x3f800000u;
    }

    // Bit k of x at bit 3 k + axis, over the axes.
    static __device__ __forceinline__ uint32_t interleave(uint32_t x)
    {
        return all_or((uint32_t)morton3(x, 0u, 0u) << own_axis(0));
    }

    __device__ __forceinline__ void load(const GridDev& g, int b)
    {
        const float4* src = g.dual + 8 * (int64_t)b + 2 * own_axis(0);
        p = src[0];
        q = src[1];
    }

    __device__ __forceinline__ bool find(const GridDev& g, double v, int& leaf)
    {
        #pragma clang fp contract(off)
        const int Lm = AMR ? g.max_level : 0;
        const int I = (int)floor(v);
        const int M = g.n0;
        const int bc = ((AMR ? I >> Lm : I) - 1) >> 1;
        bool ok = true;
        int L = 0, l = 0;
        if (!g.periodic) {
            ok = all_or((unsigned)bc < (unsigned)(M - 1) ? 0u : 1u) == 0u;
            const int Mh = 2 * (M << Lm);
            if (all_or((unsigned)I < (unsigned)Mh ? 0u : 1u)) L = -1;
        }
        int b = (int)interleave((uint32_t)(bc & (M - 1)));
        load(g, b);
        bool w = true;
        if constexpr (AMR) w = ok && g.child[b] == kWholeLeaf;
        if (AMR && !w && L >= 0) {
            int id = (int)interleave((uint32_t)((I >> (Lm + 1)) & (M - 1)));
            for (int m = Lm; m > 0; --m) {
                const int ch = g.child[id];
                if (ch < 0) break;
                id = ch + (int)all_or((uint32_t)((I >> m) & 1) << own_axis(0));
                ++L;
            }
            if (L > 0) {
                b = g.leafinfo[8 * (int64_t)(id - g.level_start[1]) +
                               all_or((uint32_t)((I >> (Lm - L)) & 1) << own_axis(0))];
                ok = b >= 0;
                if (ok) {
                    l = level_of(g, b);
                    w = l > 0 && g.child[b] == kWholeLeaf;
                    load(g, b);
                }
            }
        }
        leaf = L;
        if (!ok) {
            p = q = make_float4(0.f, 0.f, 0.f, 0.f);
            t = 0.0f;
            reset();
            return false;
        }
        if constexpr (AMR) {
            const int sh = w ? Lm - l : Lm - L;
            sc = ldexp(1.0, w ? -sh - 1 : -sh);
            const int k = I >> sh;
            const int s = L - l;
            kd = w ? 0.5 * (double)((k - 1) | 1) : (double)k;
            off = w ? kDual : (uint32_t)(k - ((((k >> s) - 1) | 1) << s));
        } else {
            kd = (double)bc + 0.5;
        }
        leafL = L;
        lvl = l;
        base = b;
        return true;
    }

    __device__ __forceinline__ bool locate(const GridDev& g, const double v[1], int& leaf_level)
    {
        #pragma clang fp contract(off)
        bool ok = true;
        double w;
        leaf_level = leafL;
        if (!inside(v[0], w, t)) {
            ok = find(g, v[0], leaf_level);
            if (ok) (void)inside(v[0], w, t);
            else t = 0.0f;
        }
        if constexpr (AMR) {
            if (off != kDual) t = ldexpf((float)(w + (double)off), lvl - leafL - 1);
        }
        return ok;
    }

    __device__ __forceinline__ int eval(const GridDev& g, const double v[1], float G[1], int& leaf_level,
                                        int& stencil_level)
    {
        const bool ok = locate(g, v, leaf_level);
        stencil_level = AMR ? lvl : 0;
        G[0] = trilinear_eval(p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w, of<0>(t), of<1>(t), of<2>(t));
        return ok ? 0 : 1;
    }

    __device__ __forceinline__ float phi(const GridDev& g) const
    {
        const float4 u = g.dual[8 * (int64_t)base + 6], w = g.dual[8 * (int64_t)base + 7];
        return trilinear_eval(u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w, of<0>(t), of<1>(t), of<2>(t));
    }
};

// Leaf containing the point with unwrapped coordinates I at level
// max_level + 1 (a walk from its coarse cell); its id in id.  Returns its
// level, or -1 outside a non-periodic box.
template <bool AMR>
__device__ __forceinline__ int walk_to_leaf(const GridDev& g, const int I[3], int& id)
{
    const int Lm = AMR ? g.max_level : 0;
    int J0 = I[0] >> 1, J1 = I[1] >> 1, J2 = I[2] >> 1;   // level max_level
    const int M = g.n0 << Lm;
    if (g.periodic) {
        J0 &= M - 1; J1 &= M - 1; J2 &= M - 1;
    } else if ((unsigned)J0 >= (unsigned)M || (unsigned)J1 >= (unsigned)M || (unsigned)J2 >= (unsigned)M) {
        return -1;
    }
    id = (int)morton3((uint32_t)(J0 >> Lm), (uint32_t)(J1 >> Lm), (uint32_t)(J2 >> Lm));
    int L = 0;
    if (AMR) {
        for (int m = Lm - 1; m >= 0; --m) {
            const int ch = g.child[id];
            if (ch < 0) break;
            id = ch + (((J0 >> m) & 1) | (((J1 >> m) & 1) << 1) | (((J2 >> m) & 1) << 2));
            ++L;
        }
    }
    return L;
}

// Field by nearest grid point (Sect. 2.2, W_NGP): the values of the deepest
// cell containing the point.  The lane keeps the last leaf and its values.
template <bool AMR>
struct NgpCache : WholeRay {
    static constexpr bool kTime = false;
    static constexpr bool kUniform = !AMR;
    static constexpr int kFloats = 0;
    static constexpr int kNoKey = 0x40000000;
    int keyL;           // level of the cached leaf
    int key[3];         // its unwrapped coordinates at that level
    float val[4];       // its (phi, gx, gy, gz)

    __device__ __forceinline__ void bind(float*) {}
    __device__ __forceinline__ void reset()
    {
        keyL = 0;
        key[0] = key[1] = key[2] = kNoKey;
    }

    // Leaf level at the point with fine coordinates I (-1 outside a
    // non-periodic box); loads the leaf's values when it changes.
    __device__ __forceinline__ int leaf(const GridDev& g, const int I[3])
    {
        const int Lm = AMR ? g.max_level : 0;
        const int sh = Lm + 1 - keyL;
        if ((I[0] >> sh) == key[0] && (I[1] >> sh) == key[1] && (I[2] >> sh) == key[2]) return keyL;
        int id;
        const int L = walk_to_leaf<AMR>(g, I, id);
        if (L < 0) return -1;
        const float4 q = g.payload[id];
        val[0] = q.x; val[1] = q.y; val[2] = q.z; val[3] = q.w;
        const int s2 = Lm + 1 - L;
        keyL = L;
        key[0] = I[0] >> s2; key[1] = I[1] >> s2; key[2] = I[2] >> s2;
        return L;
    }

    __device__ __forceinline__ int eval(const GridDev& g, const double v[3], float G[3], int& leaf_level,
                                        int& stencil_level)
    {
        int I[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) I[d] = (int)floor(v[d]);
        const int L = leaf(g, I);
        leaf_level = L;
        stencil_level = 0;
        G[0] = G[1] = G[2] = 0.0f;
        if (L < 0) return 1;
        stencil_level = L;
        G[0] = val[1]; G[1] = val[2]; G[2] = val[3];
        return 0;
    }

    // Phi at the last evaluated point
    __device__ __forceinline__ float phi(const GridDev&) const { return val[0]; }
};

// Field by triangular-shaped cloud (Sect. 2.2, W_TSC): the 27 cells around
// the cell containing the point at the leaf level, falling back one level at
// a time while any of them is missing.  The stencil depends only on the leaf
// cell (the cell containing the point at every coarser level is its
// ancestor), so the lane resolves it only when the leaf changes and keeps
// the 27 payloads in registers: a stage then costs its region check,
// weights and 108 multiply-adds, with no memory access.  It is bound by
// instruction issue; the check by the leaf's region, which also gives f where
// the stencil is at the leaf's level, in place of integer coordinates and
// keys: 49,152 rays to z = 1 on a uniform 64^3 grid 10.8 -> 9.8 ms.  On a tree
// the resolution's walks and the payloads do not fit the 256 registers: 112 are
// spilled.  Per axis, with f the position in the centre cell (in [0, 1)), the weights of the cells at
// -1, 0, +1 are (1 - f)^2 / 2, 3/4 - (f - 1/2)^2 and f^2 / 2.
template <bool AMR>
struct TscCache : WholeRay {
    static constexpr bool kTime = false;
    static constexpr bool kUniform = !AMR;
    static constexpr int kFloats = 0;
    int keyL;           // level of the leaf whose stencil is cached
    int lvl;            // level of the stencil
    // the leaf: u = v sc - kd in [0, 1)^3, as FieldCache's regions (on a tree, where
    // registers are short, kd as integers)
    typename std::conditional<AMR, int, double>::type kd[3];
    double sc;
    float4 p[27];       // payloads of stencil cell q = (x + 1) + 3 (y + 1) + 9 (z + 1)
    float w[3][3];      // weights of the last evaluated point per axis

    __device__ __forceinline__ void bind(float*) {}
    __device__ __forceinline__ void reset()
    {
        keyL = 0;
        lvl = 0;
        sc = 0.0;
        kd[0] = kd[1] = kd[2] = 1;      // no point is inside
    }

    // Load the payloads of the 27 cells cc + {-1, 0, 1}^3 at level l when
    // all of them exist; false otherwise (nothing is loaded).  Level 0: the
    // Morton id is the OR of one bit spread per axis, so 3 spreads, each with
    // one added and one taken away on its bits, give the 27 ids (nine spreads
    // were a third of the gather's instructions).  Refined level: the 27 cells have 2 x 2 x 2 parents (two per
    // axis, the parents of cc - 1 and cc + 1); each cell is its parent's
    // first child plus its octant, so 8 walks to level l - 1 replace 27
    // walks to level l.
    __host__ __device__ __forceinline__ bool gather(const GridDev& g, int l, const int cc[3])
    {
        if (!AMR || l == 0) {
            const int M = g.n0;
            const uint32_t bits = (1u << (3 * __builtin_ctz((unsigned)M))) - 1u;
            uint32_t sp[3][3];
            bool all = true;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                all &= g.periodic || (cc[d] >= 1 && cc[d] + 1 < M);
                const uint32_t lanes = (0x49249249u << d) & bits;
                sp[d][1] = part1by2((uint32_t)(cc[d] & (M - 1))) << d;
                sp[d][0] = (sp[d][1] - (1u << d)) & lanes;
                sp[d][2] = step_up(sp[d][1], lanes, 1u << d) & lanes;
            }
            if (!all) return false;
#pragma unroll
            for (int q = 0; q < 27; ++q) p[q] = g.payload[sp[0][q % 3] | sp[1][(q / 3) % 3] | sp[2][q / 9]];
            return true;
        }
        // per axis: the two parents, which of them holds the middle cell, and
        // the octant bit of the outer cells (cc -+ 1) and of the middle one
        int P[3][2], mid[3], bo[3], bm[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            P[d][0] = (cc[d] - 1) >> 1;
            P[d][1] = (cc[d] + 1) >> 1;
            mid[d] = (cc[d] >> 1) - P[d][0];
            bo[d] = (cc[d] + 1) & 1;
            bm[d] = cc[d] & 1;
        }
        int ch[8];
        bool all = true;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int par = lookup_cell(g, l - 1, P[0][s & 1], P[1][(s >> 1) & 1], P[2][s >> 2]);
            const int k = g.child[par >= 0 ? par : 0];
            ch[s] = par >= 0 ? k : -1;
            all &= ch[s] >= 0;
        }
        if (!all) return false;
        // first child of the parent of every cell, selected along z, y, x
        int t[2][2][3], u[2][3][3];
#pragma unroll
        for (int sx = 0; sx < 2; ++sx)
#pragma unroll
            for (int sy = 0; sy < 2; ++sy) {
                t[sx][sy][0] = ch[sx + 2 * sy];
                t[sx][sy][2] = ch[sx + 2 * sy + 4];
                t[sx][sy][1] = mid[2] ? t[sx][sy][2] : t[sx][sy][0];
            }
#pragma unroll
        for (int sx = 0; sx < 2; ++sx)
#pragma unroll
            for (int z = 0; z < 3; ++z) {
                u[sx][0][z] = t[sx][0][z];
                u[sx][2][z] = t[sx][1][z];
                u[sx][1][z] = mid[1] ? u[sx][2][z] : u[sx][0][z];
            }
#pragma unroll
        for (int q = 0; q < 27; ++q) {
            const int x = q % 3, y = (q / 3) % 3, z = q / 9;
            const int first = x == 0 ? u[0][y][z] : x == 2 ? u[1][y][z] : (mid[0] ? u[1][y][z] : u[0][y][z]);
            const int oct = (x == 1 ? bm[0] : bo[0]) | ((y == 1 ? bm[1] : bo[1]) << 1) | ((z == 1 ? bm[2] : bo[2]) << 2);
            p[q] = g.payload[first + oct];
        }
        return true;
    }

    __device__ __forceinline__ bool resolve(const GridDev& g, int L, const int I[3])
    {
        const int Lm = AMR ? g.max_level : 0;
        for (int l = L; l >= 0; --l) {
            const int s = Lm + 1 - l;
            const int cc[3] = {I[0] >> s, I[1] >> s, I[2] >> s};
            if (gather(g, l, cc)) {
                lvl = l;
                return true;
            }
        }
        // no stencil (the ray stops): the payloads are cleared so that every
        // path writes them, and the old ones need no registers during the search
#pragma unroll
        for (int q = 0; q < 27; ++q) p[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        return false;
    }

    // u of the point in the cached leaf; true when it lies inside
    __device__ __forceinline__ bool inside(const double v[3], float u[3]) const
    {
        #pragma clang fp contract(off)
        uint32_t m = 0u;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            u[d] = (float)fma(v[d], sc, -(double)kd[d]);
            const uint32_t b = __float_as_uint(u[d]);
            m = b > m ? b : m;
        }
        return m < 0x3f800000u;
    }

    __device__ __forceinline__ int eval(const GridDev& g, const double v[3], float G[3], int& leaf_level,
                                        int& stencil_level)
    {
        const int Lm = AMR ? g.max_level : 0;
        float f[3];
        G[0] = G[1] = G[2] = 0.0f;
        stencil_level = 0;
        if (!inside(v, f)) {
            int I[3], id;
#pragma unroll
            for (int d = 0; d < 3; ++d) I[d] = (int)floor(v[d]);
            leaf_level = walk_to_leaf<AMR>(g, I, id);
            if (leaf_level < 0) return 1;
            if (!resolve(g, leaf_level, I)) {
                reset();
                return 1;
            }
            keyL = leaf_level;
            const int s = Lm + 1 - keyL;
            sc = ldexp(1.0, -s);
#pragma unroll
            for (int d = 0; d < 3; ++d) kd[d] = I[d] >> s;
            (void)inside(v, f);
        }
        leaf_level = keyL;
        stencil_level = lvl;
        if (AMR && lvl != keyL) {
            // position in the centre cell, the leaf's ancestor at the stencil's
            // level: v 2^(lvl - Lm - 1) less its coordinate, exact in FP64
            const double sl = ldexp(1.0, lvl - Lm - 1);
#pragma unroll
            for (int d = 0; d < 3; ++d) f[d] = (float)(v[d] * sl - (double)((int)kd[d] >> (keyL - lvl)));
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float h = f[d] - 0.5f;
            w[d][0] = 0.5f * (1.0f - f[d]) * (1.0f - f[d]);
            w[d][1] = 0.75f - h * h;
            w[d][2] = 0.5f * f[d] * f[d];
        }
#pragma unroll
        for (int z = 0; z < 3; ++z)
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                const float wyz = w[1][y] * w[2][z];
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    const float wq = w[0][x] * wyz;
                    const float4 q = p[x + 3 * y + 9 * z];
                    G[0] = fmaf(wq, q.y, G[0]);
                    G[1] = fmaf(wq, q.z, G[1]);
                    G[2] = fmaf(wq, q.w, G[2]);
                }
            }
        return 0;
    }

    // Phi at the last evaluated point (the same weights)
    __device__ __forceinline__ float phi(const GridDev&) const
    {
        float acc = 0.0f;
#pragma unroll
        for (int z = 0; z < 3; ++z)
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                const float wyz = w[1][y] * w[2][z];
#pragma unroll
                for (int x = 0; x < 3; ++x) acc = fmaf(w[0][x] * wyz, p[x + 3 * y + 9 * z].x, acc);
            }
        return acc;
    }
};

// ---------------------------------------------------------------------------
// Geodesic state in the split representation.  With K = -k0 > 0,
// k = K (n + d) and x = x_obs + s n + dx, the null geodesic equations of
// Sect. 2.2 (dPhi/dlambda = grad Phi . k, dPhi/deta = 0) become
//   d eta/dl = -K,  ds/dl = K,  d dx/dl = K d,
//   dK/dl = 2 H K^2 - 2 K^2 (m.G),                          m = n + d, G = grad Phi
//   d(K d)/dl - n dK/dl = K^2 [4 (m.G) m - 2 G + 2 (H - m.G) d]   (=: P)
// RK4 is applied to (eta, K, dx, K d): d at a stage or at the step end is
// (K_n d_n + c dl P)/K.  This is the same RK4 as on (eta, x, k0, k), since
// the map between the two is linear given K, and it keeps only small
// quantities (d ~ deflection, dx ~ transverse displacement) in FP32.  The
// path coordinate s has the same increments as -eta, so s = eta_0 - eta
// exactly and is not carried.
// ---------------------------------------------------------------------------
struct RayGeom {
    double vo[3];       // observer in fine-grid coordinates (x_obs / h_f)
    double n[3];        // initial direction (unit)
};

// Comoving step length in a leaf of level L: h_L / N = ds_level[L], which
// equals ds_level[0] 2^-L exactly (h0 / 2^L / N rounds like h0 / N, and the
// power of two scales exactly); computed so, since indexing the argument
// array by a per-lane level would be a memory load at every step.
__device__ __forceinline__ double step_length(const CastArgs& a, int L)
{
    return a.adaptive ? ldexp(a.ds_level[0], -L) : a.ds_level[0];
}

// Fine-grid coordinates v = x / h_f, h_f = h0 / 2^(max_level + 1), of
// x = x_obs + s n + dx, s = eta0 - eta.  The observer term is the exact
// quotient; the displacement is scaled by 1/h_f (at the observer both agree
// exactly with x / h_f, elsewhere to one rounding).  Scaling by the power of
// two is exact, so v is 2^(max_level + 1) times the coarse-grid coordinates
// computed the same way.
// C: components the lane holds.
template <int C = 3>
__device__ __forceinline__ void grid_coords(const GridDev& g, const RayGeom& r, double eta, const float dx[C],
                                            double v[C])
{
    #pragma clang fp contract(off)
    const double s = g.eta0 - eta;
#pragma unroll
    for (int i = 0; i < C; ++i) v[i] = fma(fma(s, r.n[i], (double)dx[i]), g.inv_hf, r.vo[i]);
}

// dPhi/dl in the spatial geodesic equation.  ChainRule: grad Phi . k
// (+ dPhi/deta k0 on a time-dependent grid) at every RK4 stage (Eq. dPhi/dl,
// first form).  StepDifference: the equations written with dPhi/dl only
// (dPhi/deta eliminated, so the time equation takes grad Phi . k) and
// dPhi/dl estimated once per step as the difference of Phi between the last
// two step starts over the affine length between them (Eq. dPhi/dl, second
// form; the first step takes grad Phi . k at the observer).
struct ChainRule {
    static constexpr bool kDiff = false;
};

struct StepDifference {
    static constexpr bool kDiff = true;
    float phi_prev;     // Phi at the previous step start
    double dl_prev;     // affine length of the previous step (0: no step yet)
    float phi0;         // Phi at the start of the step being taken
    float D;            // its dPhi/dl
};

// No-op stage recorder of the forward kernels.  A recorder's stage hook
// sees the stage index, the step-start state y, the stage state yi, the
// field evaluator (its stencil and offsets at the stage), the interpolated
// gradient and the background cubic of the step.
struct NoRecord {
    template <class FC>
    __device__ __forceinline__ void stage(int, const GeoState&, const GeoState&, const FC&, const float*,
                                          const HubbleCubic&, const CosmoDev&)
    {
    }
};

// The field at a step's start point, evaluated by the caller (which needs
// the leaf level there for the step length): stage 0 of the step takes it
// instead of evaluating the same point again.
struct Stage0 {
    float phi, G[3], tv;   // phi: step-difference form only; tv: dPhi/deta (time-dependent potential)
    int l;                 // stencil level
    int bad;               // no complete stencil
};

// a / b for b of order one, as the hardware's reciprocal estimate in single
// precision, two Newton steps and a residual correction in double precision:
// the IEEE quotient without the scaling that the general division needs.
__device__ __forceinline__ double quotient(double a, double b)
{
    #pragma clang fp contract(off)
    double r = (double)__builtin_amdgcn_rcpf((float)b);
    r = fma(r, fma(-b, r, 1.0), r);
    r = fma(r, fma(-b, r, 1.0), r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

// One RK4 step of affine length dl from y into out (F: the lane's field
// evaluator, any interpolation order).  With a time-dependent potential
// (FC::kTime) the spatial equation takes dPhi/dl = grad Phi . k + T k0 with
// T = dPhi/deta (in the time equation the two T terms cancel: 2 T k0^2 -
// 2 T k0 k0), and the step's ISW increment int T K dl (= int T |d eta|) is
// left in F.isw_step.  The four stencil levels
// are appended to hash only when all four stages succeed (return 0).  When
// record is set, the recorder receives every stage's state and stencil (base
// id, level); the reverse sweep uses it to replay the forward stages exactly.
//
// The integration kernels issue vector instructions nearly all the time, so
// the instructions of a stage decide their speed.  The right-hand sides are
// kept as halves, fK = K^2 (H - m.G) and fP = K^2 ((H - m.G) d + 2 (m.G) m - G)
// (the factors 2 are exact and go into the step lengths they are multiplied
// with), and the four stages are unrolled (UNROLL) so that weights and step
// fractions are constants: about 105 instructions a stage where the general
// form took 145.  With the region check and the records' way through LDS (see
// FieldCache): 725 -> 582 instructions per wave-step and 13.26 -> 9.34 ms for
// 196,608 rays to z = 1 on a uniform 64^3 grid, 71.3 -> 61.6 ms for 786,432 rays
// on a 128^3 + 3 level tree (989 -> 843 instructions and 56.7 ms with the later
// savings in its look-ups).
template <class FC, class Rec, class DP, bool UNROLL>
__device__ __forceinline__ int rk4_core(const GridDev& g, const CosmoDev& cz, FC& F,
                                        const RayGeom& r, const GeoState& y, double dl, GeoState& out,
                                        uint32_t& hash, Rec& rec, bool record, DP& dp,
                                        const Stage0* s0 = nullptr)
{
    #pragma clang fp contract(off)
    constexpr int C = FC::kComp;
    float nf[C];
#pragma unroll
    for (int i = 0; i < C; ++i) nf[i] = (float)r.n[i];
    const double half = 0.5 * dl;
    double acc_eta = 0.0, acc_K = 0.0;
    float acc_dx[C] = {}, acc_P[C] = {};
    double f_K = 0.0, Kprev = y.K;
    float f_dx[C] = {}, f_P[C] = {};
    float acc_I = 0.f;
    uint32_t h = hash;
    HubbleCubic Hc;
    Hc.init(cz, y.eta);
    // one stage; true when no complete stencil exists at its position (the
    // remaining stages then run on meaningless values, every lookup staying
    // in bounds, and the step is rejected after the last one, so that there
    // is a single exit)
    auto stage = [&](const int st, const Stage0* z) -> bool {
        #pragma clang fp contract(off)
        GeoState yi;
        if (st == 0) {
            yi = y;
        } else {
            const double c = st == 3 ? dl : half;
            const double c2 = st == 3 ? dl + dl : dl;
            yi.eta = fma(-c, Kprev, y.eta);        // f_eta = -K of the previous stage
            yi.K = fma(c2, f_K, y.K);
            // d_stage = (K d + c P) / K_stage = d + (K / K_stage - 1) d + (c / K_stage) P:
            // d is carried exactly and only the small corrections are rounded
            const float cf = (float)c;
            const float inv = __builtin_amdgcn_rcpf((float)yi.K);   // 1 ulp
            const float rm1 = (float)(y.K - yi.K) * inv;
            const float cK = (cf + cf) * inv;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                yi.dx[i] = fmaf(cf, f_dx[i], y.dx[i]);
                yi.d[i] = fmaf(cK, f_P[i], fmaf(rm1, y.d[i], y.d[i]));
            }
        }
        float G[C];
        float phi = 0.0f;
        int l = 0;
        bool bad;
        if (z) {
            // stage 0 at the step start, evaluated by the caller
            phi = z->phi;
#pragma unroll
            for (int i = 0; i < C; ++i) G[i] = z->G[i];
            l = z->l;
            bad = z->bad != 0;
            if constexpr (FC::kTime) F.tv = z->tv;
        } else {
            double u[C];
            grid_coords<C>(g, r, yi.eta, yi.dx, u);
            int leafl;
            bad = F.eval(g, u, G, leafl, l) != 0;
            if constexpr (DP::kDiff) {
                if (st == 0) phi = F.phi(g);
            }
        }
        h = fnv(h, (uint32_t)l);
        if (record) rec.stage(st, y, yi, F, G, Hc, cz);
        const double H = Hc(cz, yi.eta);
        float m[C];
#pragma unroll
        for (int i = 0; i < C; ++i) m[i] = nf[i] + yi.d[i];
        const float mG = FC::dot(m, G);
        Kprev = yi.K;
        f_K = yi.K * yi.K * (H - (double)mG);
        const float Kf = (float)yi.K;
        const float K2 = Kf * Kf;
        const float hm = (float)H - mG;
        // dk/dl with k = K m: K^2 (2 H m + 2 (m.G - T) m - 2 G); the P form
        // subtracts n dK/dl, dK/dl = K^2 (2 H - 2 m.G)
        float cm = mG + mG;
        if constexpr (FC::kTime) cm = cm - F.tv;
        if constexpr (DP::kDiff) {
            // m.G (from -n dK/dl) + D / K (the spatial equation's dPhi/dl)
            if (st == 0) {
                dp.phi0 = phi;
                dp.D = dp.dl_prev > 0.0 ? (float)(((double)phi - (double)dp.phi_prev) / dp.dl_prev) : Kf * mG;
            }
            cm = dp.D / Kf + mG;
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
            f_dx[i] = Kf * yi.d[i];
            f_P[i] = K2 * fmaf(hm, yi.d[i], fmaf(cm, m[i], -G[i]));
        }
        if (st == 0) {
            if constexpr (FC::kTime) acc_I = F.tv * Kf;
            acc_eta = yi.K;
            acc_K = f_K;
#pragma unroll
            for (int i = 0; i < C; ++i) { acc_dx[i] = f_dx[i]; acc_P[i] = f_P[i]; }
        } else {
            const double w = st == 3 ? 1.0 : 2.0;
            const float wf = st == 3 ? 1.0f : 2.0f;
            if constexpr (FC::kTime) acc_I = fmaf(wf, F.tv * Kf, acc_I);
            acc_eta = fma(w, yi.K, acc_eta);
            acc_K = fma(w, f_K, acc_K);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                acc_dx[i] = fmaf(wf, f_dx[i], acc_dx[i]);
                acc_P[i] = fmaf(wf, f_P[i], acc_P[i]);
            }
            // the sums are taken here: the compiler would otherwise move them past
            // the test of the last stage and keep every stage's terms until then
            asm volatile("" : "+v"(acc_eta), "+v"(acc_K));
#pragma unroll
            for (int i = 0; i < C; ++i) asm volatile("" : "+v"(acc_dx[i]), "+v"(acc_P[i]));
        }
        return bad;
    };
    bool failed = stage(0, s0);
    if constexpr (UNROLL) {
        failed |= stage(1, nullptr);
        failed |= stage(2, nullptr);
        failed |= stage(3, nullptr);
    } else {
#pragma unroll 1
        for (int st = 1; st < 4; ++st) failed |= stage(st, nullptr);
    }
    if (failed) return 1;
    const double h6 = dl * (1.0 / 6.0);
    out.eta = fma(-h6, acc_eta, y.eta);
    out.K = fma(h6 + h6, acc_K, y.K);
    const float h6f = (float)h6;
    const float inv = __builtin_amdgcn_rcpf((float)out.K);
    const float rm1 = (float)(y.K - out.K) * inv;
    const float cK = (h6f + h6f) * inv;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        out.dx[i] = fmaf(h6f, acc_dx[i], y.dx[i]);
        out.d[i] = fmaf(cK, acc_P[i], fmaf(rm1, y.d[i], y.d[i]));
    }
    if constexpr (FC::kTime) F.isw_step = h6f * acc_I;
    hash = h;
    return 0;
}

// The step by the chain rule, with a recorder.
template <class FC, class Rec, bool UNROLL = true>
__device__ __forceinline__ int rk4_step(const GridDev& g, const CosmoDev& cz, FC& F,
                                        const RayGeom& r, const GeoState& y, double dl, GeoState& out,
                                        uint32_t& hash, Rec& rec, bool record, const Stage0* s0 = nullptr)
{
    ChainRule cr;
    return rk4_core<FC, Rec, ChainRule, UNROLL>(g, cz, F, r, y, dl, out, hash, rec, record, cr, s0);
}

template <class FC>
__device__ __forceinline__ int rk4_step(const GridDev& g, const CosmoDev& cz, FC& F,
                                        const RayGeom& r, const GeoState& y, double dl, GeoState& out,
                                        uint32_t& hash)
{
    NoRecord none;
    return rk4_step<FC, NoRecord, false>(g, cz, F, r, y, dl, out, hash, none, false);
}

// The forward step with a choice of dPhi/dl (ChainRule or StepDifference).
template <class FC, class DP, bool UNROLL = true>
__device__ __forceinline__ int rk4_step_dp(const GridDev& g, const CosmoDev& cz, FC& F,
                                           const RayGeom& r, const GeoState& y, double dl, GeoState& out,
                                           uint32_t& hash, DP& dp, const Stage0* s0 = nullptr)
{
    NoRecord none;
    return rk4_core<FC, NoRecord, DP, UNROLL>(g, cz, F, r, y, dl, out, hash, none, false, dp, s0);
}

// NaN or infinity anywhere in the state (a sum of the small FP32 parts is
// non-finite exactly when one of them is; they cannot overflow together).
// eta needs no test of its own: it is the start's minus a sum of the stages'
// K, and a stage's K that is not finite makes its fK and with it the end's K
// not finite.
template <class Form = WholeRay>
__device__ __forceinline__ bool finite_state(const GeoState& y)
{
    if constexpr (Form::kComp == 1) {
        const float s = y.d[0] + y.dx[0];
        return isfinite(y.K) && Form::all_or(isfinite(s) ? 0u : 1u) == 0u;
    } else {
        const float s = ((y.d[0] + y.d[1]) + (y.d[2] + y.dx[0])) + (y.dx[1] + y.dx[2]);
        return isfinite(y.K) && isfinite(s);
    }
}

}  // namespace mpath
