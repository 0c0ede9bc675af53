// VDI generation on the GPU (paper Section 3: supersegments by Eq. 1 along
// each generating ray of V_O; supplement Alg. S1: per-ray bisection of the
// sensitivity gamma so that a ray yields at most N_S supersegments).
//
// One thread per generating ray, FP64 throughout, every expression in the
// order written and without contraction into fused multiply-adds, so that the
// comparisons deciding supersegment boundaries come out as the same arithmetic
// does on a CPU (only where an FP32 distance settles a comparison by more than
// its error bound is the FP64 one left out).  The first pass over a ray, direct
// volume rendering to find where early termination ends it, takes the samples
// (trilinear interpolation of cell-centred voxels, transfer function, opacity
// corrected to the sample length) and caches them in device memory; the
// counting passes of the bisection and the final capped split read them back.
//
// The 720p volume (512^3 u16, 1280 x 720, N_S 20, 30 deg) takes 7.2 ms, bound by
// the waits of its dependent FP64 chains at 3 wavefronts per SIMD and lanes
// idle while the longest ray of their wavefront finishes; it took 29 ms with
// FP64 powers, divisions and roots at every step.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stddef.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "vdi_trace.h"

namespace vdi {
namespace {

constexpr double kGenTTerm = 1e-5;  // early ray termination of the generating rays

struct GenCam {
    double eye[3], F[3], R[3], U[3], tanh_, aspect, near_;
    int W, H;
};

struct GenVol {
    int nx, ny, nz, is_u16;
    const void *data;
    double bmin[3], bmax[3];
    double ext[3], inv[3];  // bmax - bmin; 1 / ext where div_by may use it, else 0
    __host__ __device__ int n(int a) const { return a == 0 ? nx : (a == 1 ? ny : nz); }
};

// Tables of pow_tab and of the 4-knot transfer function (fill_gen_tab).
// Kernels copy them to LDS: kept as constants they took registers from the
// start of the kernel on.
struct GenTab {
    double4 tf[3][3];  // interval s: colour at its knot and opacity; their rise over it; knot, length, 1 / length

    double4 lg[65];  // x near (64 + j) / 128: c = 1 / that in 24 bits, -log c as hi + lo
    double2 ex[24];  // exp(-k / 64) as hi + lo
};

struct GenParams {
    GenCam cam;
    GenVol vol;
    int NS, tf, maxs, delta, far_eye;
    double ds, gamma;  // gamma > 0: fixed
    GenTab tab;
};

// A constant of a polynomial, set where it is used: left to itself the
// compiler keeps every FP64 constant of the passes' loops in registers from the
// start of the kernel on (over 128 of them spilled), although a scalar move
// beside the vector instructions costs nothing.
__host__ __device__ __forceinline__ double here(double c)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(c));
#endif
    return c;
}

// x^y for opacities: (1 - a)^(len / ds) of a sample (0.5 <= x <= 1) and, WIDE,
// (1 - A)^(len / lenS) of an open supersegment (0 < x <= 1).  Both transfer
// functions keep a <= 0.2 and a sample is no longer than ds (its ray no
// longer than maxs ds), and the second is a mean of the first over the
// supersegment's samples: the result is at least 0.7 (or not a number, and
// then so is x).  Table-driven in the manner of Tang (1989, 1990): x c_j - 1 =
// f with |f| < 0.008 gives log x = -log c_j + log1p(f) as an unevaluated sum,
// its product with y as another, exp by a table in steps of 1/64 and a
// series, and one rounding at the end: at most 0.514 ulp off for the opacities
// (2,000,000 arguments against 113-bit arithmetic; 0.23% not correctly
// rounded), which is as close as pow() itself.  About 45 instructions where
// pow() takes about 200, and a sample takes one.
template <bool WIDE>
__host__ __device__ inline double pow_tab(const GenTab &W, double x, double y)
{
#pragma clang fp contract(off)
    int e = 0;
    if constexpr (WIDE) {
#ifdef __HIP_DEVICE_COMPILE__
        e = __builtin_amdgcn_frexp_exp(x);
        x = __builtin_amdgcn_frexp_mant(x);
#else
        x = frexp(x, &e);
#endif
    }
    const double4 t = W.lg[min(max((int)(x * 128.0 + 0.5) - 64, 0), 64)];
    const double f = fma(x, t.x, -1.0);
    double r = fma(f, here(-1.0 / 8), here(1.0 / 7));
    r = fma(f, r, here(-1.0 / 6));
    r = fma(f, r, here(1.0 / 5));
    r = fma(f, r, -0.25);
    r = fma(f, r, here(1.0 / 3));
    r = (f * f) * fma(f, r, -0.5);
    double sh = t.y + f, sl = (f - (sh - t.y)) + (t.z + r);
    if constexpr (WIDE) {
        // e log 2, its first part exact in 24 bits.
        constexpr long double kLn2 = 0.6931471805599453094172321214581765680755L;
        const double a = e * here((double)(float)kLn2), h = a + sh;
        const double z = h - a;
        sl += (a - (h - z)) + (sh - z) + e * here((double)(kLn2 - (float)kLn2));
        sh = h;
    }
    const double zh = y * sh, zl = fma(y, sh, -zh) + y * sl;
    const int k = min(max((int)(0.5 - zh * 64.0), 0), 23);
    const double u = fma((double)k, 1.0 / 64, zh) + zl;
    double q = fma(u, here(1.0 / 5040), here(1.0 / 720));
    q = fma(u, q, here(1.0 / 120));
    q = fma(u, q, here(1.0 / 24));
    q = fma(u, q, here(1.0 / 6));
    const double em1 = fma(u * u, fma(u, q, 0.5), u);
    const double2 x2 = W.ex[k];
    return x2.x + fma(x2.x, em1, x2.y);
}

// x / b, correctly rounded, from the correctly rounded reciprocal y = 1 / b
// (Markstein 1990: a quotient within an ulp, corrected by its exact
// remainder, rounds correctly): 5 instructions for the 11 of a division.  For
// x far from the ends of the exponent range, as coordinates and scalars are.
__host__ __device__ inline double div_by(double x, double b, double y)
{
    double q = x * y;
    q = fma(fma(-b, q, x), y, q);
    return fma(fma(-b, q, x), y, q);
}

struct Sample {
    double c[3], a;  // straight colour, opacity corrected to the sample length
    double v;        // interpolated scalar
};

// A lane's cache of its ray's first K samples, (v, a) of sample q at
// p[q * stride]: the passes after the first read them back instead of
// sampling the volume again.  K = 0: no cache.
struct SampleCache {
    double2 *p;
    int K, stride;
};

// An open supersegment: samples [qs, qe) of its ray (qs < 0: none is open),
// premultiplied colour and opacity.  While none is open C and A are zero, so
// that the first sample is taken by the same expressions as the later ones
// (0 + (1 - 0) a c is a c).
struct Open {
    double C[3], A;
    int qs, qe;
};

__host__ __device__ inline double clamp01(double v)
{
#pragma clang fp contract(off)
    return v < 0.0 ? 0.0 : (v > 1.0 ? 1.0 : v);
}

__host__ __device__ inline int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// How a kernel reads voxels.  kF32, kU16: x-neighbours in one load of 8 or 4
// bytes, aligned to a voxel only (global loads allow that); the volume is at
// least two voxels wide.  kAny: any format and width, one voxel a load.  kFar:
// as kAny, for far eyes (eye_far): there the length of a sample or of a
// supersegment is mostly the rounding of its ends, so that a power's exponent
// may be anything and Eq. 1 is decided in FP64 alone.
enum VoxelKind { kF32, kU16, kAny, kFar };
// f(kind of G's volume and eye, as a type).
template <typename F>
auto by_kind(const GenParams &G, F f)
{
    if (G.far_eye) return f(std::integral_constant<VoxelKind, kFar>());
    if (G.vol.nx < 2) return f(std::integral_constant<VoxelKind, kAny>());
    return G.vol.is_u16 ? f(std::integral_constant<VoxelKind, kU16>()) : f(std::integral_constant<VoxelKind, kF32>());
}

// x^y by pow_tab, or for far eyes by pow.
template <VoxelKind K, bool WIDE>
__host__ __device__ inline double power(const GenTab &W, double x, double y)
{
    if constexpr (K == kFar) return pow(x, y);
    else return pow_tab<WIDE>(W, x, y);
}

typedef uint32_t PairU16 __attribute__((aligned(2), may_alias));
typedef uint64_t PairF32 __attribute__((aligned(4), may_alias));

// The eight voxels around cell (floor) coordinates f, clamped to the edge.
// Element offsets need 64 bits (a row index does not: ny nz <= 2^28).
// put(2 dz + dy, voxel at x, voxel at x + 1), as stored; kAny converts and
// scales to [0, 1].
template <VoxelKind K, typename F>
__host__ __device__ __forceinline__ void load_corners(const GenVol &v, const int *f, F put)
{
    const int x0 = clampi(f[0], 0, v.nx - 1), x1 = clampi(f[0] + 1, 0, v.nx - 1);
    const int y0 = clampi(f[1], 0, v.ny - 1), y1 = clampi(f[1] + 1, 0, v.ny - 1);
    const int z0 = clampi(f[2], 0, v.nz - 1), z1 = clampi(f[2] + 1, 0, v.nz - 1);
    const int xb = K == kAny || K == kFar ? 0 : clampi(f[0], 0, v.nx - 2);
    const size_t at = (size_t)(uint32_t)(z0 * v.ny + y0) * (uint32_t)v.nx + (uint32_t)xb;
    const size_t dy = y1 != y0 ? (size_t)v.nx : 0, dz = z1 != z0 ? (size_t)v.nx * v.ny : 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const size_t o = at + (m & 1 ? dy : 0) + (m & 2 ? dz : 0);
        if constexpr (K == kF32) {
            const uint64_t u = *reinterpret_cast<const PairF32 *>(static_cast<const float *>(v.data) + o);
            const float a = __builtin_bit_cast(float, (uint32_t)u), b = __builtin_bit_cast(float, (uint32_t)(u >> 32));
            put(m, x0 != xb ? b : a, x1 != xb ? b : a);
        } else if constexpr (K == kU16) {
            const uint32_t u = *reinterpret_cast<const PairU16 *>(static_cast<const uint16_t *>(v.data) + o);
            put(m, (uint16_t)(x0 != xb ? u >> 16 : u), (uint16_t)(x1 != xb ? u >> 16 : u));
        } else if (v.is_u16) {
            const uint16_t *p = static_cast<const uint16_t *>(v.data) + o;
            put(m, (double)p[x0] * (1.0 / 65535.0), (double)p[x1] * (1.0 / 65535.0));
        } else {
            const float *p = static_cast<const float *>(v.data) + o;
            put(m, (double)p[x0], (double)p[x1]);
        }
    }
}

// Trilinear interpolation of cell-centred voxels, clamped to the edge.
template <VoxelKind K>
__host__ __device__ inline double sample_tri(const GenVol &v, const double *P)
{
#pragma clang fp contract(off)
    double w[3];
    int f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double x = P[a] - v.bmin[a];
        const double u = (v.inv[a] != 0.0 ? div_by(x, v.ext[a], v.inv[a]) : x / v.ext[a]) * v.n(a) - 0.5;
        const double fl = floor(u);
        w[a] = u - fl;
        f[a] = (int)fl;
    }
    double c[4];
    load_corners<K>(v, f, [&](int m, auto lo, auto hi) {
        const double l = K == kU16 ? (double)lo * (1.0 / 65535.0) : (double)lo;
        const double h = K == kU16 ? (double)hi * (1.0 / 65535.0) : (double)hi;
        c[m] = l * (1 - w[0]) + h * w[0];
    });
    const double c0 = c[0] * (1 - w[1]) + c[1] * w[1], c1 = c[2] * (1 - w[1]) + c[3] * w[1];
    return c0 * (1 - w[2]) + c1 * w[2];
}

// The two transfer functions of the synthetic workloads (VDI_TF_*): colour,
// and opacity if asked for.
template <bool OPACITY>
__host__ __device__ inline void tf_eval(const GenTab &W, int tf, double v, double *c, double &a)
{
#pragma clang fp contract(off)
    if (tf == VDI_TF_RAMP) {
        c[0] = v;
        c[1] = 0.25 + 0.5 * v;
        c[2] = 1.0 - v;
        if constexpr (OPACITY) a = 0.2 * clamp01((v - 0.05) / 0.95);
        return;
    }
    v = clamp01(v);
    const double4 *k = W.tf[v < 0.25 ? 0 : (v < 0.55 ? 1 : 2)];
    const double u = div_by(v - k[2].x, k[2].y, k[2].z);
    c[0] = k[0].x + u * k[1].x;
    c[1] = k[0].y + u * k[1].y;
    c[2] = k[0].z + u * k[1].z;
    if constexpr (OPACITY) a = k[0].w + u * k[1].w;
}

// Sample q of a ray (midpoint of [t0 + q len, t0 + (q + 1) len]).
template <VoxelKind K>
__host__ __device__ inline Sample take_sample(const GenParams &G, const GenTab &W, const double *d, double t0,
                                                  double len, int q)
{
#pragma clang fp contract(off)
    const double tm = t0 + (q + 0.5) * len;
    double P[3];
    for (int a = 0; a < 3; ++a) P[a] = G.cam.eye[a] + tm * d[a];
    const double v = sample_tri<K>(G.vol, P);
    Sample s;
    double atf;
    tf_eval<true>(W, G.tf, v, s.c, atf);
    s.a = atf > 0.0 ? 1.0 - power<K, false>(W, 1.0 - atf, len / G.ds) : 0.0;
    s.v = v;
    return s;
}

// The samples of a ray again, in order: from the cache where it holds them (the
// same doubles: the colour is the transfer function of the same v), else from
// the volume.  FITS: the cache holds every ray's samples.  An entry is loaded
// one sample ahead of its use.
template <bool FITS, VoxelKind K>
struct Samples {
    double2 ahead;

    __host__ __device__ inline double2 entry(const SampleCache &C, int q) const
    {
        return C.p[(size_t)(FITS ? q : min(q, C.K - 1)) * C.stride];
    }
    __host__ __device__ inline Samples(const SampleCache &C) : ahead(make_double2(0.0, 0.0))
    {
        if (FITS || C.K > 0) ahead = entry(C, 0);
    }
    // Sample q of ns; called for q = 0, 1, 2, ...
    __host__ __device__ inline Sample next(const GenParams &G, const GenTab &W, const SampleCache &C, const double *d,
                                           double t0, double len, int q, int ns)
    {
        if (!FITS && q >= C.K) return take_sample<K>(G, W, d, t0, len, q);
        const double2 e = ahead;
        ahead = entry(C, min(q + 1, ns - 1));
        Sample s;
        double unused;
        s.a = e.y;
        s.v = e.x;
        s.c[0] = s.c[1] = s.c[2] = 0.0;
        if (s.a != 0.0) tf_eval<false>(W, G.tf, e.x, s.c, unused);  // nothing takes a transparent sample
        return s;
    }
};

__host__ __device__ inline void reset(Open &o)
{
    o.C[0] = o.C[1] = o.C[2] = o.A = 0.0;
    o.qs = -1;
}

__host__ __device__ inline void take(Open &o, const Sample &s, int q)
{
#pragma clang fp contract(off)
    if (o.qs < 0) o.qs = q;
    for (int m = 0; m < 3; ++m) o.C[m] += (1.0 - o.A) * s.a * s.c[m];
    o.A += (1.0 - o.A) * s.a;
    o.qe = q + 1;
}

// Eq. 1's distance between the open supersegment, its opacity normalised to
// one sample length, and the next sample, in FP64, against gamma.
template <VoxelKind K>
__host__ __device__ inline bool far_exact(const GenTab &W, const Open &o, const Sample &s, double t0, double len, double gamma)
{
#pragma clang fp contract(off)
    const double lenS = (t0 + o.qe * len) - (t0 + o.qs * len);
    const double abar = 1.0 - power<K, true>(W, 1.0 - o.A, len / lenS);
    double d2 = 0.0;
    for (int m = 0; m < 3; ++m) {
        const double e = o.C[m] / o.A * abar - s.c[m] * s.a;
        d2 += e * e;
    }
    return sqrt(d2) >= gamma;
}

// The same decision with most of the FP64 left out.  The squared distance is
// computed in FP32 (hardware base-2 exponential, logarithm and
// reciprocal); only when it lies within kFarErr of gamma is far_exact asked,
// so the outcome is always far_exact's.  The bound, for a ray whose opacities
// are at most 0.25 and whose colours lie in [0, 1] (Passes::err is NaN
// for others and for far eyes, and every decision exact): with m = qe - qs samples the
// normalised opacity is 1 - 2^(log2(1 - A) / m), where |log2(1 - A) / m| <=
// 0.42 since it is the mean of the samples' logarithms.  Rounding 1 - A to
// FP32 moves the exponent by at most 1e-7, the logarithm's, reciprocal's and
// product's errors (1 ulp each) by 2e-7; with the exponential's ulp the
// opacity is off by at most 4e-7, and the quotient C / A, its product and the
// sample's colour add 2e-7 per channel: 1.1e-6 over three channels.  len /
// lenS differs from 1 / m by 1e-12 at most.  kFarErr is three times that.
// far_exact takes about 250 instructions and was two thirds of the kernel;
// the filter takes about 30, and asks for it in less than 1% of the steps.
constexpr float kFarErr = 3.5e-6f;

#ifdef __HIP_DEVICE_COMPILE__
__device__ inline float gen_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float gen_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ inline float gen_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
#else
__host__ inline float gen_exp2(float x) { return exp2f(x); }
__host__ inline float gen_log2(float x) { return log2f(x); }
__host__ inline float gen_rcp(float x) { return 1.0f / x; }
#endif

// gamma with the squares of the FP32 distances at which far_exact's outcome
// is certain (below lo2: false, from hi2 on: true).
struct Sensitivity {
    double gamma;
    float lo2, hi2;
};

__host__ __device__ inline Sensitivity sensitivity(double gamma, float err)
{
    const float g = (float)gamma, lo = fmaxf(g - err, 0.0f), hi = g + err;
    return {gamma, lo * lo, hi * hi};
}

// 1: far, 0: not, -1: too close to call, or not a number.
__host__ __device__ inline int far_filter(const Open &o, const Sample &s, const Sensitivity &g)
{
    const float a = (float)s.a;
    const float ab = 1.0f - gen_exp2(gen_log2((float)(1.0 - o.A)) * gen_rcp((float)(o.qe - o.qs)));
    const float k = ab * gen_rcp((float)o.A);
    float d2 = 0.0f;
    for (int m = 0; m < 3; ++m) {
        const float e = (float)o.C[m] * k - (float)s.c[m] * a;
        d2 += e * e;
    }
    return d2 >= g.hi2 ? 1 : (d2 < g.lo2 ? 0 : -1);
}

// What the passes over a ray's samples share: its parameters, the ns samples
// before early termination, and the filter's error bound.
struct Passes {
    double t0, len;
    int ns;
    float err;
};

// Count the supersegments of a ray at three sensitivities in one pass (Eq. 1):
// a sample joins the open supersegment unless it is far from it, a
// transparent sample closes it.  The pass ends once every count exceeds `most`
// (nothing asks by how much).  Three cover two steps of the bisection,
// whichever way the first one goes: the samples are then read from the cache,
// and their colours computed, half as often, and the three chains of dependent
// FP64 operations overlap.
template <bool FITS, VoxelKind K>
__host__ __device__ inline void count_segments(const GenParams &G, const GenTab &W, const SampleCache &C,
                                               const double *d, const Passes &P, const Sensitivity *g, int most, int *out)
{
    Open o[3];
    int n[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        reset(o[k]);
        n[k] = 0;
    }
    Samples<FITS, K> samples(C);
    for (int q = 0; q < P.ns; ++q) {
        const Sample s = samples.next(G, W, C, d, P.t0, P.len, q, P.ns);
        int far[3];
        bool asked = false, more = false;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            far[k] = o[k].qs < 0 ? 0 : (s.a == 0.0 ? 1 : far_filter(o[k], s, g[k]));
            asked = asked || far[k] < 0;
        }
        if (asked) {
            // One copy of far_exact, whichever sensitivity asks for it.
#pragma nounroll
            for (int k = 0; k < 3; ++k) {
                if ((k == 0 ? far[0] : (k == 1 ? far[1] : far[2])) >= 0) continue;
                auto of = [&](auto a, auto b, auto c) { return k == 0 ? a : (k == 1 ? b : c); };
                const Open x = {{of(o[0].C[0], o[1].C[0], o[2].C[0]), of(o[0].C[1], o[1].C[1], o[2].C[1]),
                                 of(o[0].C[2], o[1].C[2], o[2].C[2])},
                                of(o[0].A, o[1].A, o[2].A), of(o[0].qs, o[1].qs, o[2].qs), of(o[0].qe, o[1].qe, o[2].qe)};
                const int f = far_exact<K>(W, x, s, P.t0, P.len, of(g[0].gamma, g[1].gamma, g[2].gamma));
                if (k == 0) far[0] = f;
                else if (k == 1) far[1] = f;
                else far[2] = f;
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (far[k]) {
                ++n[k];
                reset(o[k]);
            }
            more = more || n[k] <= most;
            if (s.a != 0.0) take(o[k], s, q);
        }
        if (!more) break;
    }
    for (int k = 0; k < 3; ++k) out[k] = n[k] + (o[k].qs >= 0 ? 1 : 0);
}

// Split the samples of a ray into at most cap supersegments with sensitivity
// g (Eq. 1) and write supersegment j to slot j of list li (depths as V_O view
// depth f = t cos(theta), b likewise).  Once cap - 1 are closed the last one
// takes every remaining non-transparent sample, across gaps.
template <bool FITS, VoxelKind K>
__host__ __device__ inline int split_ray(const GenParams &G, const GenTab &W, const SampleCache &C, const double *d, double cth,
                                         const Passes &P, const Sensitivity &g, int cap, size_t li, size_t plane,
                                         float2 *depth, float4 *rgba)
{
#pragma clang fp contract(off)
    int n = 0;
    Open o;
    reset(o);
    auto close = [&]() {
        const double ts = P.t0 + o.qs * P.len, te = P.t0 + o.qe * P.len;
        float f = (float)(ts * cth), b = (float)(te * cth);
        if (!(b > f)) b = nextafterf(f, INFINITY);
        const size_t at = (size_t)n * plane + li;
        depth[at] = make_float2(f, b);
        const double A = o.A;
        rgba[at] = make_float4((float)(o.C[0] / A), (float)(o.C[1] / A), (float)(o.C[2] / A), (float)A);
        ++n;
        reset(o);
    };
    Samples<FITS, K> samples(C);
    for (int q = 0; q < P.ns; ++q) {
        const Sample s = samples.next(G, W, C, d, P.t0, P.len, q, P.ns);
        if (o.qs >= 0 && n != cap - 1) {
            int far = s.a == 0.0 ? 1 : far_filter(o, s, g);
            if (far < 0) far = far_exact<K>(W, o, s, P.t0, P.len, g.gamma);
            if (far) close();
        }
        if (s.a != 0.0) take(o, s, q);
    }
    if (o.qs >= 0) close();
    return n;
}

// Ray through the centre of pixel (px, py) of the camera, clipped to the
// AABB and the camera's near plane: unit direction d, cos(theta) = F.d and
// the parameter range [t0, t1] along d (false when empty).
__host__ __device__ inline bool ray_clip(const GenParams &G, int px, int py, double *d, double &cth, double &t0,
                                         double &t1)
{
#pragma clang fp contract(off)
    const int W = G.cam.W, H = G.cam.H;
    const double xc = -1.0 + (2.0 * px + 1.0) / W, yc = -1.0 + (2.0 * py + 1.0) / H;
    for (int a = 0; a < 3; ++a)
        d[a] = G.cam.F[a] + xc * G.cam.tanh_ * G.cam.aspect * G.cam.R[a] + yc * G.cam.tanh_ * G.cam.U[a];
    const double nrm = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    for (int a = 0; a < 3; ++a) d[a] /= nrm;
    cth = G.cam.F[0] * d[0] + G.cam.F[1] * d[1] + G.cam.F[2] * d[2];
    double lo = G.cam.near_ / cth, hi = INFINITY;
    bool in = true;
    // Unrolled: the parameters of a kernel, indexed by a loop counter, are
    // copied to scratch memory and kept in vector registers.
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (fabs(d[a]) < 1e-300) {
            in = in && !(G.cam.eye[a] < G.vol.bmin[a] || G.cam.eye[a] > G.vol.bmax[a]);
            continue;
        }
        double ta = (G.vol.bmin[a] - G.cam.eye[a]) / d[a], tb = (G.vol.bmax[a] - G.cam.eye[a]) / d[a];
        if (ta > tb) {
            const double t = ta;
            ta = tb;
            tb = t;
        }
        if (ta > lo) lo = ta;
        if (tb < hi) hi = tb;
    }
    if (!in) return false;
    t0 = lo;
    t1 = hi;
    return hi > lo;
}

// Number of equal samples over [t0, t1]: about one per ds, at least 1.
__host__ __device__ inline int sample_count(const GenParams &G, double t0, double t1)
{
#pragma clang fp contract(off)
    int N = (int)ceil((t1 - t0) / G.ds - 1e-9);
    if (N < 1) N = 1;
    if (N > G.maxs) N = G.maxs;
    return N;
}

// Sensitivity of one ray (supplement Alg. S1; bracket updates as read in
// the design notes).  The ray's supersegments at sensitivity g do not grow
// with g; the search wants N_S - delta <= count(g) <= N_S.
// A first trial at 1e-5 stands if it gives at most N_S.  Otherwise the
// bracket (lo, hi) always has count(lo) > N_S, and hi is sqrt 3 or gives
// fewer than N_S - delta; each further trial halves it.  A bracket narrower
// than 1e-6 ends the search at hi, or at lo if the trial in hand gives no
// supersegment; so does the 25th trial.
// Counts come three at a time: a trial and the two that may follow it
// (count3 fills a pass's counts, each right up to N_S and above it only known
// to be above).  Sensitivities over `reach` (at least 2e-5, so that halving
// towards the first trial ends), which no distance of the ray exceeds, give
// `runs`, the ray's runs of non-transparent samples, without a pass; the first
// pass holds the first trial and the first two that need one.
// The lanes of a wavefront take their passes together: each first settles
// what its counts in hand decide.
template <typename Count3>
__host__ __device__ inline double search_gamma(int NS, int delta, int runs, double reach, Count3 count3)
{
#pragma clang fp contract(off)
    double lo = 1e-5, hi = sqrt(3.0), g = lo;
    double held[3];
    int counts[3];
    held[0] = lo;
    double top = hi;
    do {
        held[1] = 0.5 * (lo + top);
        top = held[1];
    } while (held[1] > reach);
    held[2] = 0.5 * (lo + held[1]);
    int trials = 0;
    for (;;) {
        count3(held, counts);
        for (;;) {
            int c;
            if (g > reach)
                c = runs;
            else if (g == held[0])
                c = counts[0];
            else if (g == held[1])
                c = counts[1];
            else if (g == held[2])
                c = counts[2];
            else
                break;
            ++trials;
            if (trials == 1) {
                if (c <= NS) return lo;
            } else {
                if (hi - lo < 1e-6) return c == 0 ? lo : hi;
                if (c > NS)
                    lo = g;
                else if (c < NS - delta)
                    hi = g;
                else
                    return g;
                if (trials == 25) return hi;
            }
            g = 0.5 * (lo + hi);
        }
        held[0] = g;
        held[1] = 0.5 * (lo + g);
        held[2] = 0.5 * (g + hi);
    }
}

// The whole generation of list (px, py): ray, samples, gamma, supersegments.
// pw: G.tab or a nearer copy of it (a choice by pointer would keep the whole of
// G in scratch memory, see copy_gen_tab).
template <bool FITS, VoxelKind K>
__host__ __device__ inline void gen_ray(const GenParams &G, const GenTab &pw, const SampleCache &C, int px, int py,
                                        uint8_t *count, float2 *depth, float4 *rgba, double *gamma_out)
{
#pragma clang fp contract(off)
    const int W = G.cam.W, H = G.cam.H;
    const size_t li = (size_t)py * W + px, plane = (size_t)W * H;
    double d[3], cth, t0, t1;
    const bool hit = ray_clip(G, px, py, d, cth, t0, t1);
    int n = 0;
    double gamma = 0.0;
    if (hit) {
        const int N = sample_count(G, t0, t1);
        const double len = (t1 - t0) / N;
        // Direct volume rendering front to back: where early termination ends
        // the ray; and what bounds its distances (colours in [0, 1], and
        // each normalised opacity, a mean, no more than the largest).
        double T = 1.0, most = 0.0;
        int ns = 0, runs = 0;
        bool plain = K != kFar, gap = true;
        for (int q = 0; q < N; ++q) {
            const Sample s = take_sample<K>(G, pw, d, t0, len, q);
            if (FITS || q < C.K) C.p[(size_t)q * C.stride] = make_double2(s.v, s.a);
            plain = plain && s.a <= 0.25 && (G.tf != VDI_TF_RAMP || (s.v >= 0.0 && s.v <= 1.0));
            most = fmax(most, s.a);
            runs += gap && s.a != 0.0 ? 1 : 0;
            gap = s.a == 0.0;
            ++ns;
            T *= 1.0 - s.a;
            if (T <= kGenTTerm) break;
        }
        const Passes P = {t0, len, ns, plain ? kFarErr : NAN};
        if (G.gamma > 0.0) {
            gamma = G.gamma;
        } else {
            const double reach = plain ? fmax(1.7322 * most, 2e-5) : INFINITY;
            gamma = search_gamma(G.NS, G.delta, runs, reach, [&](const double *g, int *out) {
                const Sensitivity s[3] = {sensitivity(g[0], P.err), sensitivity(g[1], P.err), sensitivity(g[2], P.err)};
                count_segments<FITS, K>(G, pw, C, d, P, s, G.NS, out);
            });
        }
        n = split_ray<FITS, K>(G, pw, C, d, cth, P, sensitivity(gamma, P.err), G.NS, li, plane, depth, rgba);
    }
    count[li] = (uint8_t)n;
    if (gamma_out) gamma_out[li] = gamma;
    for (int j = n; j < G.NS; ++j) {
        depth[(size_t)j * plane + li] = make_float2(0.0f, 0.0f);
        rgba[(size_t)j * plane + li] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}

__host__ inline void gen_ray(const GenParams &G, const SampleCache &C, int px, int py, uint8_t *count, float2 *depth,
                             float4 *rgba, double *gamma_out)
{
    gen_ray<false, kAny>(G, G.tab, C, px, py, count, depth, rgba, gamma_out);
}

// Persistent wavefronts: each takes the next tile of 64 rays from `counter`
// (zero at launch) until none is left, and keeps the samples of its rays in
// its own cache region: [K][64 lanes] of (v, a), so that the 64 lanes, which
// step through a pass in lockstep, touch 1 KiB of consecutive memory per
// sample.  Samples beyond K are taken from the volume again.
constexpr size_t kGenCacheBytes = (size_t)4 << 30;  // at most this much cache in all
// A wavefront generates a tile of kGenTileW x kGenTileH rays: neighbouring
// rays in both directions see similar data, so their work differs less.
#ifndef VDI_GEN_TILE_W
#define VDI_GEN_TILE_W 8
#endif
constexpr int kGenTileW = VDI_GEN_TILE_W, kGenTileH = 64 / VDI_GEN_TILE_W;
#ifndef VDI_GEN_WAVES
#define VDI_GEN_WAVES 3  // wavefronts per SIMD the kernel is compiled for
#endif

// A kernel's GenParams, its first parameter, read from the kernel arguments
// where they are used.  Through the parameter all of them are loaded at the
// kernel's start and spilled from the scalar registers, and indexing any part
// of it copies the whole to scratch memory.
__device__ __forceinline__ const GenParams &gen_args(const GenParams &param)
{
#ifdef __HIP_DEVICE_COMPILE__
    using Args = const __attribute__((address_space(4))) GenParams;
    auto *p = (Args *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const GenParams *)p;
#else
    return param;
#endif
}

// G.tab into LDS, by one wavefront.
__device__ inline void copy_gen_tab(const GenParams &G, GenTab *to)
{
    static_assert(sizeof(GenTab) % sizeof(double) == 0, "copied by doubles");
    const double *from = reinterpret_cast<const double *>(&G.tab);
    for (int i = (int)threadIdx.x; i < (int)(sizeof(GenTab) / sizeof(double)); i += 64)
        reinterpret_cast<double *>(to)[i] = from[i];
    __syncthreads();
}

template <bool FITS, VoxelKind K_>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(VDI_GEN_WAVES))) void k_generate(GenParams args, unsigned *__restrict__ counter, int ntiles,
                                                 double2 *__restrict__ cache, int K, uint8_t *__restrict__ count,
                                                 float2 *__restrict__ depth, float4 *__restrict__ rgba,
                                                 double *__restrict__ gamma_out)
{
    const GenParams &G = gen_args(args);
    __shared__ GenTab s_tab;
    copy_gen_tab(G, &s_tab);
    const int tiles_x = (G.cam.W + kGenTileW - 1) / kGenTileW;
    const SampleCache C = {cache + (size_t)blockIdx.x * K * 64 + threadIdx.x, K, 64};
    for (;;) {
        int tile = 0;
        if (threadIdx.x == 0) tile = (int)atomicAdd(counter, 1u);
        tile = __shfl(tile, 0);
        if (tile >= ntiles) break;
        const int px = (tile % tiles_x) * kGenTileW + (int)threadIdx.x % kGenTileW;
        const int py = (tile / tiles_x) * kGenTileH + (int)threadIdx.x / kGenTileW;
        if (px < G.cam.W && py < G.cam.H) gen_ray<FITS, K_>(G, s_tab, C, px, py, count, depth, rgba, gamma_out);
    }
}

// ---------------------------------------------------------------------------
// Direct volume rendering (the image a VDI approximates; Section 6 compares
// VDI renderings against it): one lane per pixel of the camera, the samples
// and transfer function of generation, front-to-back emission-absorption with
// early termination at transmittance <= 1e-5.
// ---------------------------------------------------------------------------

// FP32 shading: the voxel coordinates u (FP64, cell-centred: voxel i at
// u = i) give the trilinear cell and weights; interpolation, transfer
// function, opacity and compositing run in FP32.  u16 voxels are interpolated
// as stored and scaled once.
template <VoxelKind K>
struct Gather {
    using V = std::conditional_t<K == kU16, uint16_t, float>;
    float w[3];
    V lo[4], hi[4];
};
template <VoxelKind K>
__device__ __forceinline__ void gather_f32(const GenVol &v, const double *u, Gather<K> &g)
{
    int f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double fl = floor(u[a]);
        g.w[a] = (float)(u[a] - fl);
        f[a] = (int)fl;
    }
    load_corners<K>(v, f, [&](int m, auto lo, auto hi) {
        g.lo[m] = (typename Gather<K>::V)lo;
        g.hi[m] = (typename Gather<K>::V)hi;
    });
}
// a (1 - w) + b w; as a + w (b - a), one instruction less, where voxels are
// whole numbers: float voxels may be infinite, or far enough apart that b - a
// is.
template <VoxelKind K>
__device__ __forceinline__ float lerp_f32(float a, float b, float w)
{
    return K == kU16 ? fmaf(w, b - a, a) : fmaf(b, w, a * (1.0f - w));
}
template <VoxelKind K>
__device__ __forceinline__ float value_f32(const Gather<K> &g)
{
    float c[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) c[m] = lerp_f32<K>((float)g.lo[m], (float)g.hi[m], g.w[0]);
    const float c0 = lerp_f32<K>(c[0], c[1], g.w[1]), c1 = lerp_f32<K>(c[2], c[3], g.w[1]);
    const float r = lerp_f32<K>(c0, c1, g.w[2]);
    return K == kU16 ? r * (1.0f / 65535.0f) : r;
}

// Opacity of the transfer functions in FP32, and the colour it goes with (only
// asked for where a sample is not transparent, or its colour not finite).
__device__ __forceinline__ float tf_opacity_f32(int tf, float v)
{
    if (tf == VDI_TF_RAMP) return 0.2f * fminf(fmaxf((v - 0.05f) * (1.0f / 0.95f), 0.0f), 1.0f);
    v = fminf(fmaxf(v, 0.0f), 1.0f);
    return v < 0.55f ? fmaxf(v - 0.25f, 0.0f) * (0.04f / 0.3f) : fmaf(v - 0.55f, 0.08f / 0.45f, 0.04f);
}
__device__ __forceinline__ void tf_colour_f32(int tf, float v, float *c)
{
    if (tf == VDI_TF_RAMP) {
        c[0] = v;
        c[1] = fmaf(0.5f, v, 0.25f);
        c[2] = 1.0f - v;
        return;
    }
    v = fminf(fmaxf(v, 0.0f), 1.0f);
    const bool low = v < 0.55f;  // opaque from the second knot on
    const float u = low ? (v - 0.25f) * (1.0f / 0.3f) : (v - 0.55f) * (1.0f / 0.45f);
    c[0] = low ? fmaf(u, 0.85f, 0.1f) : fmaf(u, -0.05f, 0.95f);
    c[1] = low ? fmaf(u, 0.2f, 0.7f) : fmaf(u, -0.75f, 0.9f);
    c[2] = low ? fmaf(u, -0.6f, 0.9f) : fmaf(u, -0.2f, 0.3f);
}

// Pixel of this lane: workgroups (one wavefront) render tiles of 16 x 4 pixels,
// whose rays run close together through the volume, dealt to the XCDs in
// bands of 8 pixel rows (xcd_tile).  1024 x 1024 x 512 f32, 1920 x 1080, 25 deg,
// and 512^3 u16, 1280 x 720, FP64: 8 x 8 2.15 / 1.34 ms, 16 x 4 2.10 / 1.34,
// 32 x 2 2.32 / 1.39, 64 x 1 2.27 / 1.44.
constexpr int kDvrBandRows = 8, kDvrTileW = 16, kDvrTileH = 64 / kDvrTileW;
__device__ __forceinline__ void dvr_pixel(const GenCam &cam, int &px, int &py)
{
    const int tiles_x = (cam.W + kDvrTileW - 1) / kDvrTileW, tiles_y = (cam.H + kDvrTileH - 1) / kDvrTileH;
    const int tile = xcd_tile((int)blockIdx.x, tiles_x, tiles_y, kDvrBandRows / kDvrTileH);
    px = (tile % tiles_x) * kDvrTileW + (int)threadIdx.x % kDvrTileW;
    py = (tile / tiles_x) * kDvrTileH + (int)threadIdx.x / kDvrTileW;
}

template <VoxelKind K>
__global__ __launch_bounds__(64) void k_dvr_f64(GenParams args, float4 *__restrict__ out)
{
#pragma clang fp contract(off)
    const GenParams &G = gen_args(args);
    __shared__ GenTab s_tab;
    copy_gen_tab(G, &s_tab);
    int px, py;
    dvr_pixel(G.cam, px, py);
    if (px >= G.cam.W || py >= G.cam.H) return;
    double d[3], cth, t0, t1;
    float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (ray_clip(G, px, py, d, cth, t0, t1)) {
        const int N = sample_count(G, t0, t1);
        const double len = (t1 - t0) / N;
        double T = 1.0, acc[3] = {0.0, 0.0, 0.0};
        for (int q = 0; q < N; ++q) {
            const Sample s = take_sample<K>(G, s_tab, d, t0, len, q);
            for (int m = 0; m < 3; ++m) acc[m] += T * s.a * s.c[m];
            T *= 1.0 - s.a;
            if (T <= kGenTTerm) break;
        }
        o = make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)(1.0 - T));
    }
    out[(size_t)py * G.cam.W + px] = o;
}

// Samples whose voxels are fetched together: a sample's chain is its loads,
// then interpolation to transmittance, and only the last depends on the sample
// before it.  The same frame at 16 x 4: 1 sample 2.7 ms, 2 2.2, 4 2.1.  The
// kernel is bound by the L1's rate of gather accesses, about one a lane: x
// neighbours in one load took it from 4.05 to 2.1 ms.
constexpr int kDvrAhead = 4;

template <VoxelKind K>
__global__ __launch_bounds__(64) void k_dvr_f32(GenParams args, float4 *__restrict__ out)
{
#pragma clang fp contract(off)
    const GenParams &G = gen_args(args);
    int px, py;
    dvr_pixel(G.cam, px, py);
    if (px >= G.cam.W || py >= G.cam.H) return;
    double d[3], cth, t0, t1;
    float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (ray_clip(G, px, py, d, cth, t0, t1)) {
        const int N = sample_count(G, t0, t1);
        const double len = (t1 - t0) / N;
        // Opacity 1 - (1 - a)^r as 1 - 2^(r log2(1 - a)) with the hardware
        // base-2 exponential and logarithm.
        const float r = (float)(len / G.ds);
        // Voxel coordinate of sample q along each axis: u0 + q du (FP64, rounded
        // as written: the only sample of a thin volume lies on its voxels'
        // centres, where the last bit says which neighbour has weight 0).
        double u0[3], du[3];
        for (int a = 0; a < 3; ++a) {
            const double sc = G.vol.n(a) / (G.vol.bmax[a] - G.vol.bmin[a]);
            u0[a] = (G.cam.eye[a] + (t0 + 0.5 * len) * d[a] - G.vol.bmin[a]) * sc - 0.5;
            du[a] = len * d[a] * sc;
        }
        float T = 1.0f, acc[3] = {0.0f, 0.0f, 0.0f};
        for (int q = 0; q < N && T > (float)kGenTTerm; q += kDvrAhead) {
            Gather<K> g[kDvrAhead];
#pragma unroll
            for (int k = 0; k < kDvrAhead; ++k) {
                // Past the last sample: the last one again, left out below.
                const double qk = (double)min(q + k, N - 1);
                const double u[3] = {u0[0] + qk * du[0], u0[1] + qk * du[1], u0[2] + qk * du[2]};
                gather_f32<K>(G.vol, u, g[k]);
            }
#pragma unroll
            for (int k = 0; k < kDvrAhead; ++k) {
                const float v = value_f32(g[k]), atf = tf_opacity_f32(G.tf, v);
                // The ramp's colour is v itself: not a number after 0 times it.
                const bool counts = atf > 0.0f || (K != kU16 && G.tf == VDI_TF_RAMP && !(fabsf(v) < INFINITY));
                if (counts && q + k < N && T > (float)kGenTTerm) {
                    const float at = 1.0f - __builtin_amdgcn_exp2f(r * __builtin_amdgcn_logf(1.0f - atf)), w = T * at;
                    float c[3];
                    tf_colour_f32(G.tf, v, c);
                    for (int m = 0; m < 3; ++m) acc[m] = fmaf(w, c[m], acc[m]);
                    T *= 1.0f - at;
                }
            }
        }
        o = make_float4(acc[0], acc[1], acc[2], 1.0f - T);
    }
    out[(size_t)py * G.cam.W + px] = o;
}

// ---------------------------------------------------------------------------
// Image quality of a rendering against a reference (Section 6: SSIM and
// PSNR of VDI renderings against DVR).  RGB of RGBA float32 images, data
// range 1.  SSIM (Wang et al. 2004): 11 x 11 Gaussian window, sigma 1.5,
// K1 = 0.01, K2 = 0.03, population moments, averaged over the pixels whose
// window lies inside the image and over the three channels.  PSNR from the
// mean squared error over all pixels and channels.
// ---------------------------------------------------------------------------
constexpr int kSsimR = 5;                 // window radius
constexpr int kQualityBlock = 256;        // threads per block of the partial-sum kernel

struct SsimWeights {
    double w[2 * kSsimR + 1];             // 1-d Gaussian, normalised to sum 1
};

// A block scores a tile of kQualityTW x kQualityTH pixels.  The window is
// separable: per channel, the five moments (x, y, xx, yy, xy) are summed along
// the rows of the tile and of the 5 rows above and below it, from the pixels in
// LDS into LDS, then along the columns: 11 + 11 weights a pixel instead of
// 121, at 26 / 16 of the rows.  1280 x 720: 147 -> 57 us.
constexpr int kQualityTW = 32, kQualityTH = 16;
constexpr int kQualityLW = kQualityTW + 2 * kSsimR, kQualityLH = kQualityTH + 2 * kSsimR;

// Per block: the sum of the SSIM (3 channels summed) of its valid pixels and
// the sum of squared RGB differences of all its pixels, in a fixed order.
__global__ __launch_bounds__(kQualityBlock) void k_quality_partials(const float4 *__restrict__ a,
                                                                    const float4 *__restrict__ b, int W, int H,
                                                                    SsimWeights g, double2 *__restrict__ part)
{
    __shared__ float pa[3][kQualityLH][kQualityLW], pb[3][kQualityLH][kQualityLW];
    __shared__ double mom[5][kQualityLH][kQualityTW];
    __shared__ double sh[2][kQualityBlock];
    const int tiles_x = (W + kQualityTW - 1) / kQualityTW;
    const int x0 = (int)(blockIdx.x % (unsigned)tiles_x) * kQualityTW, y0 = (int)(blockIdx.x / (unsigned)tiles_x) * kQualityTH;
    for (int i = threadIdx.x; i < kQualityLW * kQualityLH; i += kQualityBlock) {
        // Pixels outside the image are in no window that counts.
        const int lx = i % kQualityLW, ly = i / kQualityLW;
        const int x = min(max(x0 + lx - kSsimR, 0), W - 1), y = min(max(y0 + ly - kSsimR, 0), H - 1);
        const float4 u = a[(size_t)y * W + x], v = b[(size_t)y * W + x];
        pa[0][ly][lx] = u.x, pa[1][ly][lx] = u.y, pa[2][ly][lx] = u.z;
        pb[0][ly][lx] = v.x, pb[1][ly][lx] = v.y, pb[2][ly][lx] = v.z;
    }
    __syncthreads();
    double ssim = 0.0, se = 0.0;
    for (int c = 0; c < 3; ++c) {
        for (int i = threadIdx.x; i < kQualityTW * kQualityLH; i += kQualityBlock) {
            const int lx = i % kQualityTW, ly = i / kQualityTW;
            double m[5] = {0, 0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k <= 2 * kSsimR; ++k) {
                const double u = pa[c][ly][lx + k], v = pb[c][ly][lx + k], wu = g.w[k] * u, wv = g.w[k] * v;
                m[0] += wu;
                m[1] += wv;
                m[2] = fma(wu, u, m[2]);
                m[3] = fma(wv, v, m[3]);
                m[4] = fma(wu, v, m[4]);
            }
            for (int k = 0; k < 5; ++k) mom[k][ly][lx] = m[k];
        }
        __syncthreads();
        for (int i = threadIdx.x; i < kQualityTW * kQualityTH; i += kQualityBlock) {
            const int lx = i % kQualityTW, ly = i / kQualityTW, x = x0 + lx, y = y0 + ly;
            if (x >= W || y >= H) continue;
            const double d = (double)pa[c][ly + kSsimR][lx + kSsimR] - pb[c][ly + kSsimR][lx + kSsimR];
            se = fma(d, d, se);
            if (x < kSsimR || x >= W - kSsimR || y < kSsimR || y >= H - kSsimR) continue;
            double m[5] = {0, 0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k <= 2 * kSsimR; ++k)
                for (int j = 0; j < 5; ++j) m[j] = fma(g.w[k], mom[j][ly + k][lx], m[j]);
            const double C1 = 0.01 * 0.01, C2 = 0.03 * 0.03;
            const double vx = m[2] - m[0] * m[0], vy = m[3] - m[1] * m[1], cxy = m[4] - m[0] * m[1];
            ssim += ((2 * m[0] * m[1] + C1) * (2 * cxy + C2)) / ((m[0] * m[0] + m[1] * m[1] + C1) * (vx + vy + C2));
        }
        __syncthreads();
    }
    sh[0][threadIdx.x] = ssim;
    sh[1][threadIdx.x] = se;
    __syncthreads();
    for (int s = kQualityBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + s];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(sh[0][0], sh[1][0]);
}

// One block sums the partials in a fixed order.
__global__ __launch_bounds__(kQualityBlock) void k_quality_sum(const double2 *__restrict__ part, int nparts,
                                                               double2 *__restrict__ total)
{
    __shared__ double sh[2][kQualityBlock];
    double s0 = 0.0, s1 = 0.0;
    for (int k = threadIdx.x; k < nparts; k += kQualityBlock) {
        s0 += part[k].x;
        s1 += part[k].y;
    }
    sh[0][threadIdx.x] = s0;
    sh[1][threadIdx.x] = s1;
    __syncthreads();
    for (int s = kQualityBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + s];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = make_double2(sh[0][0], sh[1][0]);
}

// Table entries in 64-bit long double, kept as a double and the rest of it.
void fill_gen_tab(GenTab &W)
{
    static const GenTab tab = [] {
        GenTab t;
        for (int j = 0; j < 65; ++j) {
            const double c = (double)(float)(128.0 / (64 + j));
            const long double l = -logl((long double)c);
            t.lg[j] = make_double4(c, (double)l, (double)(l - (long double)(double)l), 0.0);
        }
        const double kv[4] = {0.0, 0.25, 0.55, 1.0}, ka[4] = {0.0, 0.0, 0.04, 0.12};
        const double kc[4][3] = {{0.1, 0.2, 0.8}, {0.1, 0.7, 0.9}, {0.95, 0.9, 0.3}, {0.9, 0.15, 0.1}};
        for (int s = 0; s < 3; ++s) {
            t.tf[s][0] = make_double4(kc[s][0], kc[s][1], kc[s][2], ka[s]);
            t.tf[s][1] = make_double4(kc[s + 1][0] - kc[s][0], kc[s + 1][1] - kc[s][1], kc[s + 1][2] - kc[s][2],
                                      ka[s + 1] - ka[s]);
            t.tf[s][2] = make_double4(kv[s], kv[s + 1] - kv[s], 1.0 / (kv[s + 1] - kv[s]), 0.0);
        }
        for (int k = 0; k < 24; ++k) {
            const long double e = expl(-(long double)k / 64.0L);
            t.ex[k] = make_double2((double)e, (double)(e - (long double)(double)e));
        }
        return t;
    }();
    W = tab;
}

void gnorm(double *v)
{
    const double n = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    v[0] /= n;
    v[1] /= n;
    v[2] /= n;
}

void gcross(const double *a, const double *b, double *o)
{
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
}

}  // namespace
}  // namespace vdi

namespace vdi {
namespace {

// Whether a ray's parameters t may exceed 1e8 ds.  Up to there a rounding of t
// (2^-53 of it) is about 1e-8 of a sample.
bool eye_far(const GenParams &G)
{
    double d2 = 0.0;  // to the AABB's farthest corner
    for (int a = 0; a < 3; ++a) {
        const double d = std::max(fabs(G.vol.bmin[a] - G.cam.eye[a]), fabs(G.vol.bmax[a] - G.cam.eye[a]));
        d2 += d * d;
    }
    return !(sqrt(d2) <= 1e8 * G.ds);
}

// Samples that each of `lanes` lanes caches: all that a ray can have, G.maxs
// (sample_count), while the cache fits the budget.
int cache_entries(const GenParams &G, size_t lanes)
{
    return (int)std::min<size_t>((size_t)G.maxs, kGenCacheBytes / (lanes * sizeof(double2)));
}

// Check the arguments and fill the per-call constants of the kernel.
int make_gen_params(const vdi_volume *vol, const vdi_gen_params *p, GenParams &G)
{
    if (!vol || !p || !vol->data) return set_error(VDI_ERR_ARG, "null argument");
    if (vol->nx < 1 || vol->ny < 1 || vol->nz < 1 || vol->nx > 16384 || vol->ny > 16384 || vol->nz > 16384)
        return set_error(VDI_ERR_ARG, "volume size out of range");
    if (vol->voxel_fmt != VDI_VOXEL_F32 && vol->voxel_fmt != VDI_VOXEL_U16)
        return set_error(VDI_ERR_ARG, "unknown voxel format");
    for (int a = 0; a < 3; ++a)
        if (!isfinite(vol->aabb_min[a]) || !isfinite(vol->aabb_max[a]) || !(vol->aabb_max[a] > vol->aabb_min[a]))
            return set_error(VDI_ERR_ARG, "the AABB must be finite and non-empty");
    if (p->width < 1 || p->height < 1 || p->width > 32768 || p->height > 32768)
        return set_error(VDI_ERR_ARG, "VDI size out of range");
    if (p->max_supersegments < 1 || p->max_supersegments > VDI_MAX_SUPERSEGMENTS)
        return set_error(VDI_ERR_ARG, "max_supersegments must be in [1, 255]");
    if (p->tf != VDI_TF_RAMP && p->tf != VDI_TF_KNOTS4) return set_error(VDI_ERR_ARG, "unknown transfer function");
    if (!isfinite(p->gamma) || p->gamma < 0.0) return set_error(VDI_ERR_ARG, "gamma must be finite and >= 0");
    const vdi_camera &c = p->camera_VO;
    const float cv[11] = {c.eye[0], c.eye[1], c.eye[2], c.target[0], c.target[1], c.target[2],
                          c.up[0],  c.up[1],  c.up[2],  c.fov_y_deg, c.near_plane};
    for (float x : cv)
        if (!isfinite(x)) return set_error(VDI_ERR_ARG, "camera has a non-finite value");
    if (!(c.fov_y_deg > 0.0f && c.fov_y_deg < 180.0f) || !(c.near_plane > 0.0f))
        return set_error(VDI_ERR_ARG, "camera fov or near plane out of range");

    memset(&G, 0, sizeof G);
    // V_O basis: F = normalize(target - eye), R = normalize(F x up), U = R x F.
    double up[3];
    for (int a = 0; a < 3; ++a) {
        G.cam.eye[a] = c.eye[a];
        G.cam.F[a] = (double)c.target[a] - (double)c.eye[a];
        up[a] = c.up[a];
    }
    gnorm(G.cam.F);
    gcross(G.cam.F, up, G.cam.R);
    gnorm(G.cam.R);
    gcross(G.cam.R, G.cam.F, G.cam.U);
    for (int a = 0; a < 3; ++a)
        if (!isfinite(G.cam.F[a]) || !isfinite(G.cam.R[a]))
            return set_error(VDI_ERR_ARG, "degenerate camera (target equals eye, or up parallel to the view)");
    G.cam.tanh_ = tan((double)c.fov_y_deg * M_PI / 360.0);
    G.cam.aspect = (double)p->width / (double)p->height;
    G.cam.near_ = c.near_plane;
    G.cam.W = p->width;
    G.cam.H = p->height;
    G.vol.nx = vol->nx;
    G.vol.ny = vol->ny;
    G.vol.nz = vol->nz;
    G.vol.is_u16 = vol->voxel_fmt == VDI_VOXEL_U16;
    G.vol.data = vol->data;
    double ext = 0.0;
    for (int a = 0; a < 3; ++a) {
        G.vol.bmin[a] = vol->aabb_min[a];
        G.vol.bmax[a] = vol->aabb_max[a];
        G.vol.ext[a] = vol->aabb_max[a] - vol->aabb_min[a];
        G.vol.inv[a] = G.vol.ext[a] > 1e-100 && G.vol.ext[a] < 1e100 ? 1.0 / G.vol.ext[a] : 0.0;
        ext = std::max(ext, G.vol.ext[a]);
    }
    const int nmax = std::max(vol->nx, std::max(vol->ny, vol->nz));
    G.ds = ext / nmax;  // one voxel of the longest axis
    G.maxs = 2 * nmax + 8;
    // A ray has at most one sample per ds of the AABB's diagonal and one more
    // (its last): less than maxs, as long as the eye is not so far away that
    // t1 - t0 is a rounding error of t1.
    const double diag = sqrt(G.vol.ext[0] * G.vol.ext[0] + G.vol.ext[1] * G.vol.ext[1] + G.vol.ext[2] * G.vol.ext[2]);
    G.far_eye = eye_far(G);
    if (!G.far_eye) G.maxs = (int)std::min((double)G.maxs, ceil(diag / G.ds) + 2.0);
    G.NS = p->max_supersegments;
    G.delta = (int)floor(0.15 * G.NS);
    G.tf = p->tf;
    G.gamma = p->gamma;
    fill_gen_tab(G.tab);
    return VDI_OK;
}

}  // namespace
}  // namespace vdi

extern "C" int vdi_generate(const vdi_volume *vol, const vdi_gen_params *p, uint8_t *count, float *depth, float *rgba,
                            double *gamma_out, void *stream)
{
    if (!count || !depth || !rgba) return vdi::set_error(VDI_ERR_ARG, "null output");
    vdi::GenParams G;
    const int rc = vdi::make_gen_params(vol, p, G);
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Persistent grid: as many single-wavefront workgroups as fit on the device at once.
    int device = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, vdi::k_generate<true, vdi::kU16>, 64, 0);
    if (e != hipSuccess) return vdi::hip_error(e, "device query");
    const long long ntiles = (long long)((p->width + vdi::kGenTileW - 1) / vdi::kGenTileW) *
                             ((p->height + vdi::kGenTileH - 1) / vdi::kGenTileH);
    const int blocks = (int)std::max<long long>(1, std::min<long long>(ntiles, (long long)std::max(1, cus * per_cu)));
    const int K = vdi::cache_entries(G, (size_t)blocks * 64);
    const bool fits = K == G.maxs;
    const size_t cache_bytes = (size_t)blocks * K * 64 * sizeof(double2);
    size_t bytes = (size_t)1 << 20;
    while (bytes < 256 + cache_bytes) bytes <<= 1;
    hipMemPool_t pool = nullptr;
    e = vdi::library_pool(device, &pool);
    if (e != hipSuccess) return vdi::hip_error(e, "scratch pool");
    char *scratch = nullptr;
    e = hipMallocFromPoolAsync((void **)&scratch, bytes, pool, st);
    if (e != hipSuccess) return vdi::set_error(VDI_ERR_OOM, "generation scratch (%zu bytes)", bytes);
    e = hipMemsetAsync(scratch, 0, sizeof(unsigned), st);
    if (e == hipSuccess) {
        auto kernel = vdi::by_kind(G, [&](auto k) {
            return fits ? vdi::k_generate<true, decltype(k)::value> : vdi::k_generate<false, decltype(k)::value>;
        });
        kernel<<<blocks, 64, 0, st>>>(G, reinterpret_cast<unsigned *>(scratch), (int)ntiles,
                                               reinterpret_cast<double2 *>(scratch + 256), K, count,
                                               reinterpret_cast<float2 *>(depth), reinterpret_cast<float4 *>(rgba),
                                               gamma_out);
        e = hipGetLastError();
    }
    const hipError_t e2 = hipFreeAsync(scratch, st);
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess) return vdi::hip_error(e, "generation launch");
    return VDI_OK;
}

extern "C" int vdi_dvr(const vdi_volume *vol, const vdi_dvr_params *p, float *out_rgba, void *stream)
{
    if (!p || !out_rgba) return vdi::set_error(VDI_ERR_ARG, "null argument");
    if (p->precision != VDI_DVR_F64 && p->precision != VDI_DVR_F32)
        return vdi::set_error(VDI_ERR_ARG, "unknown DVR precision");
    if (p->width > 16384 || p->height > 16384) return vdi::set_error(VDI_ERR_ARG, "image size out of range");
    vdi_gen_params gp;
    memset(&gp, 0, sizeof gp);
    gp.camera_VO = p->camera;
    gp.width = p->width;
    gp.height = p->height;
    gp.max_supersegments = 1;
    gp.tf = p->tf;
    vdi::GenParams G;
    const int rc = vdi::make_gen_params(vol, &gp, G);
    if (rc) return rc;
    const dim3 grid((unsigned)((p->width + vdi::kDvrTileW - 1) / vdi::kDvrTileW) *
                    (unsigned)((p->height + vdi::kDvrTileH - 1) / vdi::kDvrTileH));
    auto *out = reinterpret_cast<float4 *>(out_rgba);
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const bool f64 = p->precision == VDI_DVR_F64;
    auto kernel = vdi::by_kind(
        G, [&](auto k) { return f64 ? vdi::k_dvr_f64<decltype(k)::value> : vdi::k_dvr_f32<decltype(k)::value>; });
    kernel<<<grid, 64, 0, st>>>(G, out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return vdi::hip_error(e, "DVR launch");
    return VDI_OK;
}

extern "C" int vdi_image_quality(const float *image, const float *reference, int32_t width, int32_t height,
                                 double *ssim, double *psnr, void *stream)
{
    if (!image || !reference || !ssim || !psnr) return vdi::set_error(VDI_ERR_ARG, "null argument");
    if (width < 2 * vdi::kSsimR + 1 || height < 2 * vdi::kSsimR + 1 || width > 16384 || height > 16384)
        return vdi::set_error(VDI_ERR_ARG, "images must be 11x11 to 16384x16384 (the SSIM window is 11x11)");
    vdi::SsimWeights g;
    double sum = 0.0;
    for (int k = -vdi::kSsimR; k <= vdi::kSsimR; ++k) sum += (g.w[k + vdi::kSsimR] = exp(-(k * k) / (2.0 * 1.5 * 1.5)));
    for (double &w : g.w) w /= sum;
    const size_t n = (size_t)width * height;
    const int nparts = ((width + vdi::kQualityTW - 1) / vdi::kQualityTW) * ((height + vdi::kQualityTH - 1) / vdi::kQualityTH);
    hipStream_t st = static_cast<hipStream_t>(stream);
    double2 *d_part = nullptr;
    hipError_t e = hipMallocAsync((void **)&d_part, (nparts + 1) * sizeof(double2), st);
    if (e != hipSuccess) return vdi::hip_error(e, "quality scratch");
    vdi::k_quality_partials<<<nparts, vdi::kQualityBlock, 0, st>>>(reinterpret_cast<const float4 *>(image),
                                                                   reinterpret_cast<const float4 *>(reference), width,
                                                                   height, g, d_part);
    vdi::k_quality_sum<<<1, vdi::kQualityBlock, 0, st>>>(d_part, nparts, d_part + nparts);
    double2 tot = make_double2(0.0, 0.0);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&tot, d_part + nparts, sizeof tot, hipMemcpyDeviceToHost, st);
    const hipError_t e2 = hipFreeAsync(d_part, st);
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return vdi::hip_error(e, "quality");
    const double valid = (double)(width - 2 * vdi::kSsimR) * (height - 2 * vdi::kSsimR) * 3.0;
    *ssim = tot.x / valid;
    const double mse = tot.y / (3.0 * (double)n);
    *psnr = mse > 0.0 ? 10.0 * log10(1.0 / mse) : INFINITY;
    return VDI_OK;
}
