// gfx950 kernels of the virtual-particle (VP) transport.
//
// One lane carries one VP history at a time (Methods A: every VP, primary or
// secondary, follows the same model, so lanes of a wavefront run the same
// code).  Each workgroup stages the physics tables of the materials it meets
// (17 to 51 KB by kernel) and, where the beam line runs, the aperture polygon in
// LDS.  The step loop is FP32; the VP energy is kept
// as an unevaluated FP32 pair so per-step losses telescope without drift;
// every deposit is converted to int64 fixed point and added with a 64-bit
// atomic, which makes the tally independent of execution order.
#include <math.h>

#include <mutex>

#include "vpmc_internal.hpp"

namespace vpmc {
namespace {

constexpr float kELo = 1.0f;
constexpr float kSegPerLog2 = (float)(NE - 1) / 8.0f;   // E_HI / E_LO = 2^8
constexpr int kThreads = 256;

// ------------------------------------------------------------ random numbers
// Philox4x32-10 (Salmon et al., SC'11); counter (block, history, spot, 0),
// key (seed_lo, seed_hi ^ field).
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // full 64-bit products (one v_mad_u64_u32 each)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x, p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0);
    }
    return c;
}

// (top 23 bits + 1/2) times 2^-23, strictly inside (0, 1): the bits as the
// mantissa of a float in [1, 2), less 1 - 2^-24 (exact: an odd multiple of
// 2^-24 below 2^24 of them)
__device__ __forceinline__ float unit_open(uint32_t w) {
    return __uint_as_float(__builtin_amdgcn_alignbit(127u, w, 9u)) - 0x1.fffffep-1f;
}

// natural logarithm of a positive finite number: hardware log2 and a two-part
// product with ln 2
__device__ __forceinline__ float ln_pos(float x) {
    const float y = __builtin_amdgcn_logf(x);
    const float r = y * 0x1.62e42ep-1f;
    return r + fmaf(y, 0x1.efa39ep-25f, fmaf(y, 0x1.62e42ep-1f, -r));
}

struct Lane {
    float px, py, pz, dx, dy, dz;
    float pzlo;               // low part of the depth (slab depth, or voxel-local z)
    float pxlo, pylo;         // low parts of the voxel-local x, y (patient only)
    float E, Elo;             // energy as an unevaluated pair E + Elo
    uint32_t nblk, spot, hist, k0, k1;
    unsigned physics;
    uint32_t nsteps;
};

// ---------------------------------------------------- double-float values
// An unevaluated FP32 pair h + l with |l| <= ulp(h)/2, built from error-free
// transformations: Knuth's TwoSum, Dekker's Fast2Sum (|a| >= |b| or a = 0)
// and the FMA-based exact product.  The CSDA bookkeeping (energy, residual
// range, path lengths, densities) runs on pairs, so a track's energy does not
// drift by FP32 rounding step after step; the drift would otherwise reach the
// residual deposit at the end of range amplified by S(E_end)/S(E_start).
struct DF {
    float h, l;
};

__device__ __forceinline__ DF fast2(float a, float b) {
    const float s = a + b;
    return {s, b - (s - a)};
}

__device__ __forceinline__ DF two_sum(float a, float b) {
    const float s = a + b;
    const float bb = s - a;
    return {s, (a - (s - bb)) + (b - bb)};
}

__device__ __forceinline__ DF df_add(DF a, DF b) {
    const DF s = two_sum(a.h, b.h);
    return fast2(s.h, s.l + (a.l + b.l));
}

__device__ __forceinline__ DF df_sub(DF a, DF b) { return df_add(a, {-b.h, -b.l}); }

__device__ __forceinline__ DF df_mul(DF a, DF b) {
    const float p = a.h * b.h;
    const float e = fmaf(a.h, b.h, -p) + (a.h * b.l + a.l * b.h);
    return fast2(p, e);
}

__device__ __forceinline__ DF df_mul_f(DF a, float b) {
    const float p = a.h * b;
    return fast2(p, fmaf(a.l, b, fmaf(a.h, b, -p)));
}

// a / b: FP32 quotient, then one correction from the exact remainder
__device__ __forceinline__ DF df_div(DF a, DF b) {
    const float rb = __builtin_amdgcn_rcpf(b.h);
    const float q = a.h * rb;
    const DF r = df_sub(a, df_mul_f(b, q));
    return fast2(q, (r.h + r.l) * rb);
}

__device__ __forceinline__ bool df_le(DF a, DF b) { return a.h < b.h || (a.h == b.h && a.l <= b.l); }

__device__ __forceinline__ uint4 draw(Lane &v) {
    const uint4 w = philox4x32_10(make_uint4(v.nblk, v.hist, v.spot, 0u), v.k0, v.k1);
    v.nblk++;
    return w;
}

// Sampling arithmetic of the physics steps uses the hardware square root
// (about 1 ulp); the straight-mode bookkeeping never calls it.
__device__ __forceinline__ float sqrt_hw(float x) { return __builtin_amdgcn_sqrtf(x); }

// step normals: hardware sin/cos take the angle in turns
__device__ __forceinline__ void box_muller_fast(uint32_t a, uint32_t b, float &z1, float &z2) {
    const float r = sqrt_hw(-2.0f * ln_pos(unit_open(a)));
    const float t = unit_open(b);
    z1 = r * __builtin_amdgcn_cosf(t);
    z2 = r * __builtin_amdgcn_sinf(t);
}

// ------------------------------------------------------------ table lookups
// The staged tables of a kernel: high parts, low parts (deterministic mode
// only) and, in the kernels that stage them, where the beam line's materials are.
struct Tabs {
    const float *hi, *lo;
    int pmma, brass;
};

// Stages the shared tables and materials [m0, m0 + NM) of the blob in LDS.
template <bool X, int NM>
__device__ __forceinline__ void stage_tables(float *hi, float *lo, const float *blob, int m0) {
    constexpr int n0 = TAB_SHARED / 4, n1 = NM * TAB_PER_MAT / 4, l0 = TABL_SHARED / 4, l1 = NM * TAB_PER_LMAT / 4;
    const float4 *b = reinterpret_cast<const float4 *>(blob), *bm = b + n0 + m0 * (TAB_PER_MAT / 4);
    for (int i = threadIdx.x; i < n0 + n1; i += blockDim.x)
        reinterpret_cast<float4 *>(hi)[i] = i < n0 ? b[i] : bm[i - n0];
    if constexpr (X) {
        const float4 *l = b + TAB_HI_FLOATS / 4, *lm = l + l0 + m0 * (TAB_PER_LMAT / 4);
        for (int i = threadIdx.x; i < l0 + l1; i += blockDim.x)
            reinterpret_cast<float4 *>(lo)[i] = i < l0 ? l[i] : lm[i - l0];
    }
}

// segment i with E_i <= E < E_i+1, clamped to [0, NE-2].  The nodes are
// log-spaced, so the hardware logarithm (error below 1e-4 of a segment)
// misses it by one at most.
__device__ __forceinline__ int seg_of(const float *tab, float E) {
    int i = (int)(__builtin_amdgcn_logf(E) * kSegPerLog2);
    i = min(max(i, 0), NE - 2);
    const float a = tab[TAB_E + i], b = tab[TAB_E + i + 1];
    i += (E >= b ? 1 : 0) - (E < a ? 1 : 0);
    return min(max(i, 0), NE - 2);
}

// position of E on the node grid: segment and clamped fraction, shared by
// every table interpolated at the same energy (linear in E between nodes)
struct NodePos {
    int i;
    float f;
};

// position of an energy E < E_i+1 known to lie at or below segment i (the
// search walks down from i to the unique segment with E_j <= E < E_j+1; the
// sentinel before the first node ends it)
__device__ __forceinline__ NodePos node_pos_below(const float *tab, float E, int i) {
    while (E < tab[TAB_E + i]) --i;
    i = max(i, 0);
    const float f = (E - tab[TAB_E + i]) * tab[TAB_RDW + i];
    return {i, fminf(fmaxf(f, 0.0f), 1.0f)};
}

// Standard normal quantile of u in (0, 1), z = sqrt(2) erfinv(2u - 1), for
// the straggling draw.  The structure is M. Giles' single-precision erfinv
// ("Approximating the erfinv function", GPU Computing Gems Jade Edition,
// 2011): with w = -log(1 - t^2) = -log(4u(1 - u)), erfinv(t)/t is a
// polynomial in w - 2.5 for w < 5 and in sqrt(w) - 3 above.  The degree-8
// coefficients are this library's own weighted least-squares fits to the FP64
// function (gen_quantile.py), largest relative error 2.7e-7 over the uniform
// grid u = (k + 1/2) 2^-23.
__device__ __forceinline__ float normal_quantile(float u) {
    const float t = 2.0f * u - 1.0f;
    const float w = -ln_pos(4.0f * u * (1.0f - u));
    float p;
    if (w < 5.0f) {   // central part (all but 0.34 % of the draws)
        const float s1 = w - 2.5f;
        float a = 2.798955610e-08f;
        a = fmaf(a, s1, 3.430734327e-07f);
        a = fmaf(a, s1, -3.522236486e-06f);
        a = fmaf(a, s1, -4.389634286e-06f);
        a = fmaf(a, s1, 2.185773789e-04f);
        a = fmaf(a, s1, -1.253729840e-03f);
        a = fmaf(a, s1, -4.177678720e-03f);
        a = fmaf(a, s1, 2.466407436e-01f);
        p = fmaf(a, s1, 1.501409417e+00f);
    } else {
        const float s2 = sqrt_hw(w) - 3.0f;
        float b = -2.393541571e-04f;
        b = fmaf(b, s2, 1.079666834e-04f);
        b = fmaf(b, s2, 1.402476381e-03f);
        b = fmaf(b, s2, -3.678024843e-03f);
        b = fmaf(b, s2, 5.716959691e-03f);
        b = fmaf(b, s2, -7.622124629e-03f);
        b = fmaf(b, s2, 9.441883054e-03f);
        b = fmaf(b, s2, 1.001674163e+00f);
        p = fmaf(b, s2, 2.832976859e+00f);
    }
    return 1.41421356237f * p * t;
}

// 1 - exp(-x) for x >= 0 (nuclear removal over a step): the series to x^5
// below 1/8 (truncation below x^6/720), else through exp
__device__ __forceinline__ float one_minus_exp_neg(float x) {
    if (x < 0.125f) return x * (1.0f - x * (0.5f - x * (0.16666667f - x * (0.041666668f - x * 0.0083333338f))));
    return 1.0f - __expf(-x);
}

__device__ __forceinline__ float node_lerp(const float *y, NodePos p) {
    return fmaf(p.f, y[p.i + 1] - y[p.i], y[p.i]);
}

__device__ __forceinline__ void rotate_dir(Lane &v, float ax, float ay) {
    const float th2 = ax * ax + ay * ay;
    if (th2 == 0.0f) return;
    const float sg = copysignf(1.0f, v.dz);
    const float a = -__builtin_amdgcn_rcpf(sg + v.dz);
    const float b = v.dx * v.dy * a;
    const float e1x = 1.0f + sg * v.dx * v.dx * a, e1y = sg * b, e1z = -sg * v.dx;
    const float e2x = b, e2y = sg + v.dy * v.dy * a, e2z = -v.dy;
    // cos(th) and sin(th)/th: series in th^2 below th^2 = 0.01 (multiple
    // scattering per step; truncation below 3e-10), else from sin and cos
    float c, k;
    if (th2 < 0.01f) {
        c = 1.0f - th2 * (0.5f - th2 * (0.041666668f - th2 * 0.0013888889f));
        k = 1.0f - th2 * (0.16666667f - th2 * (0.0083333338f - th2 * 0.00019841270f));
    } else {
        const float th = sqrt_hw(th2);
        float sn;
        __sincosf(th, &sn, &c);
        k = sn * __builtin_amdgcn_rcpf(th);
    }
    float nx = c * v.dx + k * (ax * e1x + ay * e2x);
    float ny = c * v.dy + k * (ax * e1y + ay * e2y);
    float nz = c * v.dz + k * (ax * e1z + ay * e2z);
    const float inv = rsqrtf(nx * nx + ny * ny + nz * nz);
    v.dx = nx * inv;
    v.dy = ny * inv;
    v.dz = nz * inv;
}




enum { ST_STOP = 0, ST_GEO = 1, ST_INNER = 2 };

__device__ __forceinline__ DF df_div_f(DF a, float b) {
    const float rb = __builtin_amdgcn_rcpf(b);
    const float q = a.h * rb;
    const DF r = df_sub(a, df_mul_f({q, 0.0f}, b));
    return fast2(q, (r.h + r.l) * rb);
}

// 1/b to within about half an ulp: hardware estimate and one Newton step
// (the raw estimate's error has a fixed sign)
__device__ __forceinline__ float rcp_nr(float b) {
    const float r = __builtin_amdgcn_rcpf(b);
    return fmaf(r, fmaf(-b, r, 1.0f), r);
}

// Arithmetic of the two transport instantiations.  Exact (deterministic
// mode, checked against the FP64 reference to 1e-5 per voxel): double-float
// pairs.  Physics mode: plain FP32 on the high parts, the low parts constant
// zero and folded away; the per-step losses carry the straggling noise, next
// to which FP32 rounding is immaterial.
template <bool X>
struct Ar;

template <>
struct Ar<true> {
    static __device__ __forceinline__ DF pair(float h, float l) { return {h, l}; }
    static __device__ __forceinline__ DF add(DF a, DF b) { return df_add(a, b); }
    static __device__ __forceinline__ DF sub(DF a, DF b) { return df_sub(a, b); }
    static __device__ __forceinline__ DF mul(DF a, DF b) { return df_mul(a, b); }
    static __device__ __forceinline__ DF mul_f(DF a, float b) { return df_mul_f(a, b); }
    static __device__ __forceinline__ DF div(DF a, DF b) { return df_div(a, b); }
    static __device__ __forceinline__ DF div_f(DF a, float b) { return df_div_f(a, b); }
    static __device__ __forceinline__ bool le(DF a, DF b) { return df_le(a, b); }
};

template <>
struct Ar<false> {
    static __device__ __forceinline__ DF pair(float h, float) { return {h, 0.0f}; }
    static __device__ __forceinline__ DF add(DF a, DF b) { return {a.h + b.h, 0.0f}; }
    static __device__ __forceinline__ DF sub(DF a, DF b) { return {a.h - b.h, 0.0f}; }
    static __device__ __forceinline__ DF mul(DF a, DF b) { return {a.h * b.h, 0.0f}; }
    static __device__ __forceinline__ DF mul_f(DF a, float b) { return {a.h * b, 0.0f}; }
    static __device__ __forceinline__ DF div(DF a, DF b) { return {a.h * rcp_nr(b.h), 0.0f}; }
    static __device__ __forceinline__ DF div_f(DF a, float b) { return {a.h * rcp_nr(b), 0.0f}; }
    static __device__ __forceinline__ bool le(DF a, DF b) { return a.h <= b.h; }
};

// move by the path length h along d: the depth as a pair; in the patient
// (voxel-local frame) x and y as pairs too, in a slab plain FP32
template <bool Slab, bool X>
__device__ __forceinline__ void move(Lane &v, DF h) {
    using A = Ar<X>;
    const DF z = A::add(A::pair(v.pz, v.pzlo), A::mul_f(h, v.dz));
    v.pz = z.h;
    v.pzlo = z.l;
    if (Slab || !X) {
        v.px = fmaf(h.h, v.dx, v.px);
        v.py = fmaf(h.h, v.dy, v.py);
    } else {
        const DF x = df_add({v.px, v.pxlo}, df_mul_f(h, v.dx));
        const DF y = df_add({v.py, v.pylo}, df_mul_f(h, v.dy));
        v.px = x.h;
        v.pxlo = x.l;
        v.py = y.h;
        v.pylo = y.l;
    }
}

// (E, Elo) -= dE: exact pair arithmetic, or in physics mode the FP32 loss
// compensated into the pair (so the energy still telescopes)
template <bool X>
__device__ __forceinline__ void sub_energy(Lane &v, DF dE) {
    const DF e = df_sub({v.E, v.Elo}, X ? dE : DF{dE.h, 0.0f});
    v.E = e.h;
    v.Elo = e.l;
}

// Energy lost while traversing r (density x mm), starting at E = E_i + x in
// segment i of the piecewise-linear CSDA relation E(R), whose range within
// the segment is rem = x / slope_i.  Whole segments crossed contribute their
// exact energy width; the last partial segment r * slope_j.  All in pairs.
// tm: the material's high tables, tl: its low tables (read only when X).  The
// walk ends at the latest at index -1, whose width is infinite and slope zero.
template <bool X>
__device__ __forceinline__ DF csda_loss(const Tabs &T, const float *tm, const float *tl, int i, DF x, DF rem,
                                        DF r) {
    using A = Ar<X>;
    if (A::le(r, rem)) return A::mul(r, A::pair(tm[T_SH * NE + i], X ? tl[L_SL * NE + i] : 0.0f));
    DF dE = x;
    r = A::sub(r, rem);
    for (--i;; --i) {
        const DF dR = A::pair(tm[T_DH * NE + i], X ? tl[L_DL * NE + i] : 0.0f);
        if (A::le(r, dR)) break;
        dE = A::add(dE, A::pair(T.hi[TAB_DWH + i], X ? T.lo[TABL_DW + i] : 0.0f));
        r = A::sub(r, dR);
    }
    return A::add(dE, A::mul(r, A::pair(tm[T_SH * NE + i], X ? tl[L_SL * NE + i] : 0.0f)));
}

// One condensed-history step in a homogeneous region: CSDA loss from the
// range table, Bohr straggling, Gaussian multiple scattering applied at the
// step midpoint (hinge), nuclear removal turning the VP into its leading
// secondary.  rho_loss scales energy loss and straggling (range scenarios),
// rho scattering and nuclear removal.  dg: distance to the region boundary.
// Energy, residual range, path and density are pairs (double-float); the
// decisions (range-out, step length) and the physics sampling use FP32.
// let: the step's LET in MeV/mm (= keV/um) for the dose-averaged LET tally:
// the mean CSDA stopping power over the step (dE_csda / s); for a VP that
// stops, its energy over its residual path (E rho / R); at the cut-off, the
// slope of the CSDA relation's first segment times the density.
// P: the processes, compiled in (-1: read from the lane).
template <bool Slab, bool X, int P = X ? 0 : -1>
__device__ __forceinline__ int phys_step(Lane &v, const Tabs &T, int m, DF rho_loss, float rho, DF dg, float &dep,
                                         float &esc, float &let) {
    using A = Ar<X>;
    const unsigned phys = P >= 0 ? (unsigned)P : v.physics;
    esc = 0.0f;
    let = 0.0f;
    v.nsteps++;
    const float *tab = T.hi;
    const float *tm = tab + TAB_SHARED + m * TAB_PER_MAT;
    const float *tl = T.lo + TABL_SHARED + m * TAB_PER_LMAT;
    const float tot = v.E + v.Elo;
    int i = seg_of(tab, v.E);
    // E - E_i: the high parts subtract exactly (same binade), the low parts add
    DF x = X ? two_sum(v.E - tab[TAB_E + i], v.Elo - T.lo[TABL_E + i])
             : DF{(v.E - tab[TAB_E + i]) + v.Elo, 0.0f};
    if (x.h < 0.0f && i > 0) {
        --i;
        x = X ? two_sum(v.E - tab[TAB_E + i], v.Elo - T.lo[TABL_E + i])
              : DF{(v.E - tab[TAB_E + i]) + v.Elo, 0.0f};
    }
    DF rem;
    if constexpr (X) rem = A::div(x, {tm[T_SH * NE + i], tl[L_SL * NE + i]});
    else rem = {x.h * tm[T_RS * NE + i], 0.0f};
    const float R = tm[T_R * NE + i] + rem.h;
    // at the cut-off, or without the range to reach the boundary: stops here
    const bool cut = tot <= kELo;
    if (cut || rho_loss.h * dg.h >= R) {
        let = cut ? rho_loss.h * tm[T_SH * NE] : tot * rho_loss.h * __builtin_amdgcn_rcpf(R);
        dep = tot;
        v.E = v.Elo = 0.0f;
        return ST_STOP;
    }
    const float smax = STEP_FRACTION * R * __builtin_amdgcn_rcpf(rho_loss.h);
    const bool geo = dg.h <= smax;
    const DF s = geo ? dg : DF{smax, 0.0f};
    const DF r = A::mul(rho_loss, s);   // density x mm (the tables' unit)
    DF dE = csda_loss<X>(T, tm, tl, i, x, rem, r);
    if (s.h > 0.0f) let = (dE.h + dE.l) / (s.h + s.l);
    const float Ebar = v.E - 0.5f * dE.h;
    uint4 w = make_uint4(0u, 0u, 0u, 0xFFFFFFFFu);
    NodePos pb{0, 0.0f};
    if (phys) {
        w = draw(v);
        pb = node_pos_below(tab, Ebar, i);
    }
    if (phys & PH_STRAGGLE) {
        const float var = r.h * node_lerp(tm + T_W2 * NE, pb);
        const float z = normal_quantile(unit_open(w.z));
        dE = A::add(dE, {-(sqrt_hw(var) * z), 0.0f});
        if (!(dE.h + dE.l > 0.0f)) dE = {0.0f, 0.0f};
        else if (dE.h + dE.l > tot) dE = {v.E, v.Elo};
    }
    dep = dE.h + dE.l;
    sub_energy<X>(v, dE);
    if (phys & PH_MCS) {
        const float th0 = sqrt_hw(rho * s.h * node_lerp(tm + T_T * NE, pb));
        float z1, z2;
        box_muller_fast(w.x, w.y, z1, z2);
        const DF h = {0.5f * s.h, 0.5f * s.l};
        move<Slab, X>(v, h);
        rotate_dir(v, th0 * z1, th0 * z2);
        move<Slab, X>(v, h);
    } else {
        move<Slab, X>(v, s);
    }
    if (phys & PH_NUCLEAR) {
        // 1 - exp(-x) <= x: the few lanes with u below x look closer
        const float xn = rho * s.h * node_lerp(tm + T_SN * NE, pb), u = unit_open(w.w);
        if (u < xn && u < one_minus_exp_neg(xn)) {
            const uint4 w2 = draw(v);
            const float E1 = v.E + v.Elo;
            const float loc = NUC_F_LOCAL * E1, out = NUC_F_ESCAPE * E1;
            v.E = (E1 - loc) - out;
            v.Elo = 0.0f;
            dep += loc;
            esc = out;
            float n1, n2;
            box_muller_fast(w2.x, w2.y, n1, n2);
            rotate_dir(v, NUC_SIGMA_RAD * n1, NUC_SIGMA_RAD * n2);
        }
    }
    return geo ? ST_GEO : ST_INNER;
}

// ------------------------------------------------------------ tallies
struct Acc {
    long long led[NLEDGER];
    unsigned long long steps, hist;
};

__device__ __forceinline__ long long to_fixed(float e, float scale) {
    return (long long)rintf(e * scale);
}

// the same, quick where the result lies in [0, 2^32) (as the float's bits
// tell: positive floats order like their bits, negative ones come after)
__device__ __forceinline__ long long to_fixed_deposit(float e, float scale) {
    const float r = rintf(e * scale);
    if (__float_as_uint(r) < 0x4F800000u) return (long long)(uint32_t)r;
    return (long long)r;
}

__device__ __forceinline__ void ledger_add(Acc &a, int j, float e, float scale) {
    a.led[j] += to_fixed(e, scale);
}

// dense tally: one 64-bit atomic per deposit
struct DenseSink {
    unsigned long long *tally;
    unsigned long long *let = nullptr;   // dose-averaged LET numerator, or none
    static constexpr bool kLet = true;
    __device__ __forceinline__ void add_let(uint32_t v, const int *, long long q) const {
        atomicAdd(let + v, (unsigned long long)q);
    }
    __device__ __forceinline__ void add(uint32_t v, const int *, long long q) const {
        atomicAdd(tally + v, (unsigned long long)q);
    }
};

// per-row tally of the influence-matrix builder: a non-returning 64-bit
// atomic into the row's dense slot grid and a store of 1 into the
// touched-block byte map (one byte per 32 voxels).  Every writer stores the
// same value and the marks are read only by later kernels, so the store is
// relaxed at workgroup scope: it stays in L2 (write-back, merged per line)
// instead of being written through to memory on every step.
struct SparseSink {
    unsigned long long *grid;
    uint8_t *mark;
    static constexpr bool kLet = false;
    unsigned long long *let = nullptr;
    __device__ __forceinline__ void add_let(uint32_t, const int *, long long) const {}
    __device__ __forceinline__ void add(uint32_t v, const int *, long long q) const {
        put(v, q);
    }
    __device__ __forceinline__ void put(uint32_t v, long long q) const {
        atomicAdd(grid + v, (unsigned long long)q);
        __hip_atomic_store(mark + (v >> 5), (uint8_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// Row tile of the work queue: a dense box of the CT grid in LDS around the
// row's particles, shared by the waves of a workgroup that work on the same
// row.  Deposits inside the box are LDS atomics, the others go to the row's
// grid; the box is added into the grid once when its last user leaves.  On
// this GPU the int64 tally atomics to device memory are performed on the
// memory side, beyond the XCD's L2, and their rate bounds the step loop; the
// tile takes most of them off that path.  An entry holds the low 32 bits of its
// voxel's sum: the deposit's high half and the carry out of the entry (the
// returned old value tells) go to the grid, where the entry's bits are added
// once at the end, so the int64 sum is exact.  At 4 bytes a voxel the box is
// twice as large as with int64 entries, and a carry comes once per few hundred
// deposits.  MARKS: influence-matrix slots with their touched-block marks, else
// dense tallies.  LET: a second box behind the first for the numerator of the
// dose-averaged LET.
//
// LET runs keep the two sums of a voxel side by side in memory (dose, LET
// numerator; 16 bytes), and what a step leaves for memory waits in the lane
// until the whole wavefront is there: memory_adds then issues the dose sums
// from 32 lanes and the LET sums of the same voxels from the other 32 in one
// instruction, and lanes of one 64-byte line are one memory-side operation
// (8.7e8 of them at 2.17e10/s were 40 of 42 ms for 950 spots x 3000 particles in
// three scenarios; 31 ms this way).
struct Pending {
    uint32_t vox;
    long long dose, let;
};
struct NoPending {};

template <bool MARKS, bool LET>
struct TileSink {
    uint32_t *tile;     // nullptr: this wave does not use the tile
    int lo0, lo1, lo2;
    uint32_t n0, n1, n2;
    SparseSink gs;
    uint32_t let_off;          // entries from a voxel's tally to its LET entry
    mutable typename std::conditional<LET, Pending, NoPending>::type pend;
    static constexpr bool kLet = LET, let = LET;
    __device__ __forceinline__ void put(uint32_t v, long long q) const {
        if constexpr (MARKS) gs.put(v, q);
        else atomicAdd(gs.grid + v, (unsigned long long)q);
    }
    // the low half into a tile entry; true when the rest (in q) is not zero
    static __device__ __forceinline__ bool carry(uint32_t *e, long long &q) {
        const uint32_t ql = (uint32_t)q;
        const uint32_t old = atomicAdd(e, ql);
        const int qh = (int)(q >> 32) + (old + ql < ql ? 1 : 0);
        q = (long long)qh << 32;
        return qh != 0;
    }
    __device__ __forceinline__ bool inside(const int *idx, uint32_t &at) const {
        const uint32_t u0 = (uint32_t)(idx[0] - lo0), u1 = (uint32_t)(idx[1] - lo1), u2 = (uint32_t)(idx[2] - lo2);
        at = u0 + n0 * (u1 + n1 * u2);
        return u0 < n0 && u1 < n1 && u2 < n2;
    }
    __device__ __forceinline__ void add_let(uint32_t v, const int *idx, long long q) const {
        uint32_t at;
        if (tile && inside(idx, at) && !carry(tile + let_off + at, q)) return;
        pend.vox = v;
        pend.let = q;
    }
    __device__ __forceinline__ void add(uint32_t v, const int *idx, long long q) const {
        uint32_t at;
        if (tile && inside(idx, at) && !carry(tile + at, q)) return;
        if constexpr (LET) {
            pend.vox = v;
            pend.dose = q;
        } else {
            put(v, q);
        }
    }
    // adds what waits in the lanes (every lane of the wavefront calls this)
    __device__ __forceinline__ void memory_adds(int lane) const {
        unsigned long long m = __ballot((pend.dose | pend.let) != 0);
        while (m) {
            const int rank = __popcll(m & ((1ull << lane) - 1ull)), n = min(32, __popcll(m));
            const bool mine = (m >> lane & 1ull) && rank < 32;
            // lane k and lane 32 + k take the k-th waiting lane's two sums
            const int from = __builtin_amdgcn_ds_bpermute(
                4 * (lane & 31), __builtin_amdgcn_ds_permute(4 * (mine ? rank : 63), lane));
            const uint32_t v = (uint32_t)__shfl((int)pend.vox, from);
            const long long d = __shfl(pend.dose, from), l = __shfl(pend.let, from);
            const long long q = lane < 32 ? d : l;
            if ((lane & 31) < n && q != 0)
                atomicAdd(gs.grid + 2 * (size_t)v + (lane >> 5), (unsigned long long)q);
            m &= ~__ballot(mine);
        }
    }
};

// ------------------------------------------------------------ aperture
// crossing number (ray casting) with the half-open rule
__device__ __forceinline__ bool in_polygon(const float2 *poly, int nv, float x, float y) {
    bool c = false;
    float2 b = poly[nv - 1];
    for (int i = 0; i < nv; ++i) {
        const float2 a = poly[i];
        if ((a.y > y) != (b.y > y)) {
            const float xc = a.x + (y - a.y) * (b.x - a.x) / (b.y - a.y);
            if (x < xc) c = !c;
        }
        b = a;
    }
    return c;
}

// Conservative distance from (x, y) to the aperture polygon's boundary, read
// from the field's distance raster: the stored distance at the cell centre
// less the farthest a point of the cell can be from it (distances are
// 1-Lipschitz).  Returns 0 when the point may lie near the boundary (the
// exact edge loops then decide) and sets `inside` when the bound is > 0.
__device__ __forceinline__ float sdf_bound(const FieldDev &f, float x, float y, bool &inside) {
    inside = false;
    if (!f.sdf || !(x == x) || !(y == y)) return 0.0f;
    const float fx = (x - f.sdf_x0) * f.sdf_ih, fy = (y - f.sdf_y0) * f.sdf_ih;
    if (!(fx >= 0.0f && fy >= 0.0f && fx < (float)f.sdf_nx && fy < (float)f.sdf_ny)) return f.sdf_far;
    const float d = f.sdf[(int)fy * f.sdf_nx + (int)fx];
    inside = d > 0.0f;
    return fmaxf(fabsf(d) - f.sdf_r, 0.0f);
}

// true when a BEV ray of lateral speed `lat` cannot reach the boundary within
// path length t, with room for the FP32 rounding of the exact edge distance
__device__ __forceinline__ bool no_edge_within(float lb, float lat, float t) {
    return lb > 0.0f && lat * t < lb * (1.0f - 1e-5f) - 1e-4f;
}

// The exact side of (x, y) and the path length along (u, v) to the first
// edge, from the edges listed for the point's raster cell (non-divergent
// block): the cell's reference point has a known side, each listed edge that
// the segment from it to (x, y) crosses flips the side (half-open
// orientation tests), and no unlisted edge lies within list_reach of (x, y).
// Returns 0 (the caller takes the loops over every edge) when the cell has
// no reference point, 1 when te is the exact first-edge distance or the
// caller's path length t ends before any edge, and 2 when only the side is
// known: the first listed hit and t both lie beyond list_reach laterally
// (lat = |(u, v)|), so an unlisted edge may come first and the caller takes
// the loop over every edge for te.  A listed hit within list_reach is the
// first hit: an earlier one would lie closer to (x, y), so on a listed edge.
// Each listed edge's crossing arithmetic is edge_distance's.
__device__ __forceinline__ int listed_edges(const FieldDev &f, const float2 *poly, int nv, float x, float y,
                                            float u, float v, float lat, float t, bool &inside, float &te) {
    if (!f.cell) return 0;
    const float fx = (x - f.sdf_x0) * f.sdf_ih, fy = (y - f.sdf_y0) * f.sdf_ih;
    if (!(fx >= 0.0f && fy >= 0.0f && fx < (float)f.sdf_nx && fy < (float)f.sdf_ny)) return 0;
    const int cell = (int)fy * f.sdf_nx + (int)fx;
    const uint2 oc = f.cell[cell];
    const uint32_t o0 = oc.x, o1 = oc.y;
    if (!(o0 & 0x40000000u)) return 0;
    const float2 r = f.cell_ref[cell];
    bool in = (o0 & 0x80000000u) != 0u;
    float best = INFINITY;
    const float sx = x - r.x, sy = y - r.y;
    for (uint32_t k = o0 & 0x3fffffffu; k < o1; ++k) {
        const int e = f.cell_edge[k];
        const float2 a = poly[e], b = poly[e + 1 < nv ? e + 1 : 0];
        const float ex = b.x - a.x, ey = b.y - a.y;
        const float o_r = ex * (r.y - a.y) - ey * (r.x - a.x);
        const float o_p = ex * (y - a.y) - ey * (x - a.x);
        const float o_a = sx * (a.y - r.y) - sy * (a.x - r.x);
        const float o_b = sx * (b.y - r.y) - sy * (b.x - r.x);
        if ((o_r > 0.0f) != (o_p > 0.0f) && (o_a > 0.0f) != (o_b > 0.0f)) in = !in;
        const float den = u * ey - v * ex;
        if (den != 0.0f) {
            const float wx = a.x - x, wy = a.y - y;
            const float inv = 1.0f / den;
            const float th = (wx * ey - wy * ex) * inv;
            const float lam = (wx * v - wy * u) * inv;
            if (th > 0.0f && lam >= 0.0f && lam <= 1.0f) best = fminf(best, th);
        }
    }
    inside = in;
    te = best;
    return lat * fminf(best, t) <= f.list_reach ? 1 : 2;
}

// path length along (u, v) until the beam's-eye-view ray from (x, y) meets an
// edge (a non-divergent block)
__device__ __forceinline__ float edge_distance(const float2 *poly, int nv, float x, float y, float u,
                                               float v) {
    float best = INFINITY;
    float2 a = poly[nv - 1];
    for (int i = 0; i < nv; ++i) {
        const float2 b = poly[i];
        const float ex = b.x - a.x, ey = b.y - a.y;
        const float den = u * ey - v * ex;
        if (den != 0.0f) {
            const float wx = a.x - x, wy = a.y - y;
            const float inv = 1.0f / den;
            const float t = (wx * ey - wy * ex) * inv;
            const float lam = (wx * v - wy * u) * inv;
            if (t > 0.0f && lam >= 0.0f && lam <= 1.0f) best = fminf(best, t);
        }
        a = b;
    }
    return best;
}

// Path length along the ray (x, y) + t (u, v) to the first wall of the block
// (INFINITY if none).  Every wall is the plane through the focus and an edge
// of the polygon: at opening scale s0 (s = s0 + t kw along the ray) the ray
// meets the wall of edge (a, b) where p + t d = s (a + lam (b - a)), linear
// in t.  A non-divergent block has s0 = 1, kw = 0: the beam's-eye-view
// ray-segment intersection.
__device__ __forceinline__ float edge_distance_div(const float2 *poly, int nv, float x, float y, float u,
                                                   float v, float s0, float kw) {
    float best = INFINITY;
    float2 a = poly[nv - 1];
    for (int i = 0; i < nv; ++i) {
        const float2 b = poly[i];
        const float ex = b.x - a.x, ey = b.y - a.y;
        const float ux = u - kw * a.x, uy = v - kw * a.y;
        const float den = ux * ey - uy * ex;
        if (den != 0.0f) {
            const float wx = s0 * a.x - x, wy = s0 * a.y - y;
            const float inv = 1.0f / den;
            const float t = (wx * ey - wy * ex) * inv;
            const float mu = (wx * uy - wy * ux) * inv;
            const float st = fmaf(t, kw, s0);
            if (t > 0.0f && st > 0.0f && mu >= 0.0f && mu <= st) best = fminf(best, t);
        }
        a = b;
    }
    return best;
}

// push the projected position EDGE_PUSH_MM further along the projected
// direction, depth unchanged, across the edge just reached (non-divergent)
__device__ __forceinline__ void edge_push(Lane &v) {
    const float n2 = v.dx * v.dx + v.dy * v.dy;
    if (n2 > 0.0f) {
        const float k = EDGE_PUSH_MM * rsqrtf(n2);
        v.px = fmaf(k, v.dx, v.px);
        v.py = fmaf(k, v.dy, v.py);
    }
}

// edge push in the block: along the scaled position's direction of travel
// d_xy - kw X, which crosses the wall just reached (d_xy for a non-divergent
// block, where kw = 0)
__device__ __forceinline__ void edge_push_blk(Lane &v, const FieldDev &f) {
    const float isc = 1.0f / fmaf(v.pz, f.fs, f.fc0), kw = v.dz * f.fs;
    const float cx = v.dx - kw * (v.px * isc), cy = v.dy - kw * (v.py * isc);
    const float n2 = cx * cx + cy * cy;
    if (n2 > 0.0f) {
        const float k = EDGE_PUSH_MM * rsqrtf(n2);
        v.px = fmaf(k, cx, v.px);
        v.py = fmaf(k, cy, v.py);
    }
}

// Inside a slab (range shifter or block) the depth is kept relative to the
// slab's upstream face as a pair (pz + pzlo) and the thickness is a pair, so
// the path to the exit plane is exact to the pairs' precision rather than to
// FP32 rounding of the step lengths or of the absolute beam-frame depth.
template <bool X>
__device__ __forceinline__ DF plane_distance(const Lane &v, DF thick, bool &down) {
    using A = Ar<X>;
    DF t = {INFINITY, 0.0f};
    down = true;
    if (v.dz > 0.0f) t = A::div_f(A::sub(thick, A::pair(v.pz, v.pzlo)), v.dz);
    else if (v.dz < 0.0f) { down = false; t = A::div_f(A::pair(-v.pz, -v.pzlo), v.dz); }
    return t.h > 0.0f ? t : DF{0.0f, 0.0f};
}

enum { EX_DOWN = 0, EX_GONE = 1 };

// homogeneous slab (range shifter): local depth 0 .. thick; on return the
// depth is the global plane z the VP left through
template <bool X>
__device__ int slab_transport(Lane &v, Acc &acc, float scale, const Tabs &T, int m, DF rho,
                              float zu, float zd, DF thick, int ledger) {
    v.pz = 0.0f;
    v.pzlo = 0.0f;
    for (int it = 0; it < MAX_STEPS; ++it) {
        bool down;
        const DF tp = plane_distance<X>(v, thick, down);
        float dep, esc;
        float let;
        const int st = phys_step<true, X>(v, T, m, rho, rho.h, tp, dep, esc, let);
        ledger_add(acc, ledger, dep, scale);
        ledger_add(acc, L_NUC, esc, scale);
        if (st == ST_STOP) return EX_GONE;
        if (st == ST_GEO || v.pz >= thick.h || v.pz <= 0.0f) {
            const bool out_down = (st == ST_GEO) ? down : (v.pz >= thick.h);
            v.pz = out_down ? zd : zu;
            v.pzlo = 0.0f;
            if (out_down) return EX_DOWN;
            ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
            return EX_GONE;
        }
    }
    ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
    return EX_GONE;
}

// Searches over every edge of the polygon for the lanes with `need`, one such
// lane at a time: its point and direction are broadcast and the edges are
// divided among the lanes of the wave that are here (a lane alone would walk
// all edges with the others waiting: 128 edges of ~27 instructions against
// ~80 per searching lane this way; with more than 40 lanes in need each takes
// its own loop again).  Each edge's arithmetic and the minimum (parity) over
// the edges are those of the loops above, so the results are the same bits.
// DIV: the divergent block's walls at opening scale s0, rate kw.
template <bool DIV>
__device__ __forceinline__ float wave_edge_distance(const float2 *poly, int nv, float x, float y, float u, float v,
                                                    float s0, float kw, bool need) {
    float res = INFINITY;
    unsigned long long todo = __ballot(need);
    if (todo == 0ull) return res;
    if (__popcll(todo) > 40) {
        if (need) res = DIV ? edge_distance_div(poly, nv, x, y, u, v, s0, kw) : edge_distance(poly, nv, x, y, u, v);
        return res;
    }
    const unsigned long long here = __ballot(true);
    const int lane = threadIdx.x & 63, n = __popcll(here), rank = __popcll(here & ((1ull << lane) - 1ull));
    auto bc = [](float f, int l) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(f), l));
    };
    for (; todo; todo &= todo - 1ull) {
        const int l = __ffsll((long long)todo) - 1;
        const float xs = bc(x, l), ys = bc(y, l), us = bc(u, l), vs = bc(v, l);
        const float ss = DIV ? bc(s0, l) : 1.0f, ks = DIV ? bc(kw, l) : 0.0f;
        float best = INFINITY;
        for (int i = rank; i < nv; i += n) {
            const float2 a = poly[i ? i - 1 : nv - 1], b = poly[i];
            const float ex = b.x - a.x, ey = b.y - a.y;
            const float ux = DIV ? us - ks * a.x : us, uy = DIV ? vs - ks * a.y : vs;
            const float den = ux * ey - uy * ex;
            if (den != 0.0f) {
                const float wx = DIV ? ss * a.x - xs : a.x - xs, wy = DIV ? ss * a.y - ys : a.y - ys;
                const float inv = 1.0f / den;
                const float t = (wx * ey - wy * ex) * inv;
                const float mu = (wx * uy - wy * ux) * inv;
                const float st = DIV ? fmaf(t, ks, ss) : 1.0f;
                if (t > 0.0f && (!DIV || st > 0.0f) && mu >= 0.0f && mu <= st) best = fminf(best, t);
            }
        }
        float m = INFINITY;
        for (unsigned long long hits = __ballot(best < INFINITY); hits; hits &= hits - 1ull)
            m = fminf(m, bc(best, __ffsll((long long)hits) - 1));
        if (lane == l) res = m;
    }
    return res;
}

__device__ __forceinline__ bool wave_in_polygon(const float2 *poly, int nv, float x, float y, bool need) {
    bool res = false;
    unsigned long long todo = __ballot(need);
    if (todo == 0ull) return res;
    if (__popcll(todo) > 40) {
        if (need) res = in_polygon(poly, nv, x, y);
        return res;
    }
    const unsigned long long here = __ballot(true);
    const int lane = threadIdx.x & 63, n = __popcll(here), rank = __popcll(here & ((1ull << lane) - 1ull));
    for (; todo; todo &= todo - 1ull) {
        const int l = __ffsll((long long)todo) - 1;
        const float xs = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), l));
        const float ys = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(y), l));
        bool c = false;
        for (int i = rank; i < nv; i += n) {
            const float2 a = poly[i], b = poly[i ? i - 1 : nv - 1];
            if ((a.y > ys) != (b.y > ys)) {
                const float xc = a.x + (ys - a.y) * (b.x - a.x) / (b.y - a.y);
                if (xs < xc) c = !c;
            }
        }
        const bool in = (__popcll(__ballot(c)) & 1) != 0;
        if (lane == l) res = in;
    }
    return res;
}

// Where a point in the block stands: its side of the opening and the path
// length te to the first wall, exact wherever it is below the path length t
// that matters.  `on` lanes only; every lane of the wave that calls takes
// part in the searches.  In the brass (`R` > 0: the residual range times
// 1.001 over the density) no wall beyond R matters either: the particle
// stops or steps short of it, with the same result wherever it is.
template <bool D>
__device__ __forceinline__ void block_side(const FieldDev &f, const float2 *poly, bool on, float x, float y, float dx,
                                           float dy, float dz, float z, float t, float R, bool far_side, bool &open,
                                           float &te) {
    const int nv = f.nv;
    open = false;
    te = INFINITY;
    if (nv < 3) return;   // closed block
    if (!(D && f.div)) {
        bool need = false, inside;
        const float lat = sqrtf(dx * dx + dy * dy);
        if (on) {
            const float lb = sdf_bound(f, x, y, inside);
            if (no_edge_within(lb, lat, t)) {
                open = inside;
            } else {
                const int ls = listed_edges(f, poly, nv, x, y, dx, dy, lat, t, open, te);
                if (ls == 0) open = lb > 0.0f ? inside : in_polygon(poly, nv, x, y);
                // (far_side: the caller does not use te in the brass)
                need = ls != 1 && !(far_side && !open);
                if (need && !open && R > 0.0f) {
                    const float tr = fminf(t, R);
                    if (no_edge_within(lb, lat, tr)) { te = INFINITY; need = false; }
                    else if (ls == 2 && lat * fminf(te, tr) <= f.list_reach) need = false;
                }
            }
        }
        const float full = wave_edge_distance<false>(poly, nv, x, y, dx, dy, 1.0f, 0.0f, need);
        if (need) te = full;
    } else {
        // divergent block: opening scale at this depth and its rate of change
        // along the ray; far from every edge for the whole path to the exit
        // plane the side is known and the exact edge distance exceeds t (the
        // scaled position moves by at most t |d_xy - kw (bx, by)| / min s)
        const float sc = fmaf(z, f.fs, f.fc0), kw = dz * f.fs;
        const float isc = 1.0f / sc;
        const float bx = x * isc, by = y * isc;
        const float cx = dx - kw * bx, cy = dy - kw * by;
        bool side = false, need = false, inside;
        if (on) {
            const float lb = sdf_bound(f, bx, by, inside);
            if (no_edge_within(lb, sqrtf(cx * cx + cy * cy) / fminf(sc, fmaf(t, kw, sc)), t)) {
                open = inside;
            } else {
                need = true;
                side = !(lb > 0.0f);
                open = lb > 0.0f && inside;
            }
        }
        const bool in = wave_in_polygon(poly, nv, bx, by, side);
        if (side) open = in;
        if (far_side && !open) need = false;
        const float full = wave_edge_distance<true>(poly, nv, x, y, dx, dy, sc, kw, need);
        if (need) te = full;
    }
}

// CSDA range of the particle's energy in a material (density x mm), as
// phys_step finds it up to rounding
__device__ __forceinline__ float residual_range(const Lane &v, const Tabs &T, int m) {
    const int i = seg_of(T.hi, v.E);
    const float *tm = T.hi + TAB_SHARED + m * TAB_PER_MAT;
    return tm[T_R * NE + i] + (v.E - T.hi[TAB_E + i]) * __builtin_amdgcn_rcpf(tm[T_SH * NE + i]);
}

enum { BK_IN = 0, BK_DOWN = 1, BK_GONE = 2 };

// One step of a traversal of the aperture block (Methods B: between the
// block's entrance and exit planes the crossing number at the particle's
// projected position decides, at every step, opening (straight transport, no
// random numbers) or brass).  The depth is local to the block.  `on` lanes
// step; every lane of the wave that calls takes part in the edge searches.
// D = false compiles the plain (non-divergent) geometry only; D = true adds
// the divergent block's.  A non-divergent block takes the same code, and so
// gives the same bits, in both.
template <bool X, bool D>
__device__ __forceinline__ int block_step(Lane &v, bool on, uint32_t &it, Acc &acc, float scale, const Tabs &T,
                                          const float2 *poly, const FieldDev &f) {
    const DF thick = {f.blk_t, f.blk_tl};
    bool down = true, open = false;
    DF tpp = {0.0f, 0.0f};
    float te = INFINITY, R = 0.0f;
    if (on && it++ >= (uint32_t)MAX_BLOCK_ITER) {
        ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
        return BK_GONE;
    }
    if (on) {
        tpp = plane_distance<X>(v, thick, down);
        // (E_LO: at the cut-off the particle stops whatever the distance)
        R = v.E > kELo ? 1.001f * residual_range(v, T, T.brass) / f.blk_rho : 0.0f;
    }
    block_side<D>(f, poly, on, v.px, v.py, v.dx, v.dy, v.dz, v.pz, tpp.h, R, false, open, te);
    if (!on) return BK_IN;
    const float tp = tpp.h;
    auto leave = [&](bool out_down) {
        v.pz = out_down ? f.blk_zd : f.blk_zu;
        v.pzlo = 0.0f;
        if (out_down) return (int)BK_DOWN;
        ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
        return (int)BK_GONE;
    };
    if (open) {
        if (tp <= te) {
            v.px = fmaf(tp, v.dx, v.px);
            v.py = fmaf(tp, v.dy, v.py);
            return leave(down);
        }
        move<true, X>(v, {te, 0.0f});
        if constexpr (D) edge_push_blk(v, f);
        else edge_push(v);
        return BK_IN;
    }
    const DF dg = te < tp ? DF{te, 0.0f} : tpp;
    float dep, esc, let;
    const int st = phys_step<true, X>(v, T, T.brass, {f.blk_rho, 0.0f}, f.blk_rho, dg, dep, esc, let);
    ledger_add(acc, L_BLOCK, dep, scale);
    ledger_add(acc, L_NUC, esc, scale);
    if (st == ST_STOP) return BK_GONE;
    if (st == ST_GEO && tp <= te) return leave(down);
    if (st == ST_GEO) {
        if constexpr (D) edge_push_blk(v, f);
        else edge_push(v);
    }
    if (v.pz >= thick.h) { v.pz = f.blk_zd; v.pzlo = 0.0f; return BK_DOWN; }
    if (v.pz <= 0.0f) return leave(false);
    return BK_IN;
}

// Whole traversals of the lanes with `on` (depth local to the block); true
// for those that leave through the downstream face.
template <bool X, bool D>
__device__ bool block_transport(Lane &v, bool on, Acc &acc, float scale, const Tabs &T, const float2 *poly,
                                const FieldDev &f) {
    uint32_t it = 0;
    int st = on ? BK_IN : BK_GONE;
    while (__ballot(st == BK_IN) != 0ull) {
        const bool in = st == BK_IN;
        const int s = block_step<X, D>(v, in, it, acc, scale, T, poly, f);
        if (in) st = s;
    }
    return st == BK_DOWN;
}

// distance from (x, y) to the polygon's boundary (minimum over edges of the
// point-to-segment distance)
__device__ float dist_to_polygon(const float2 *poly, int nv, float x, float y) {
    float best = INFINITY;
    float2 a = poly[nv - 1];
    for (int i = 0; i < nv; ++i) {
        const float2 b = poly[i];
        const float ex = b.x - a.x, ey = b.y - a.y;
        const float wx = x - a.x, wy = y - a.y;
        const float l2 = ex * ex + ey * ey;
        float t = l2 > 0.0f ? (wx * ex + wy * ey) / l2 : 0.0f;
        t = fminf(fmaxf(t, 0.0f), 1.0f);
        const float dx = wx - t * ex, dy = wy - t * ey;
        best = fminf(best, dx * dx + dy * dy);
        a = b;
    }
    return sqrtf(best);
}

// Range shifter, then the block's upstream face, in the beam frame, for the
// lanes with `on`: BL_PATIENT with tmin the ray parameter of the last exit
// plane ((p, d) is then on the particle's ray), BL_BLOCK when the block's
// brass or walls are met (the particle is on the upstream face, depth local),
// BL_DEFER when the surrogate takes the traversal, else BL_STOP.
enum { BL_STOP = 0, BL_PATIENT = 1, BL_DEFER = 2, BL_BLOCK = 3 };

template <bool X, bool D>
__device__ __forceinline__ int beam_entry(Lane &v, bool on, Acc &acc, float scale, const Tabs &T, const float2 *poly,
                                          const FieldDev &f, float &tmin, const SurDev *sur, uint32_t tag) {
    tmin = -INFINITY;
    int st = on ? BL_PATIENT : BL_STOP;
    if (on && f.has_rs) {
        const float t = (f.rs_zu - v.pz) / v.dz;
        const float qx = fmaf(t, v.dx, v.px), qy = fmaf(t, v.dy, v.py);
        if (qx * qx + qy * qy <= f.rs_r2) {
            v.px = qx;
            v.py = qy;
            v.pz = f.rs_zu;
            if (slab_transport<X>(v, acc, scale, T, T.pmma, {f.rs_rho, f.rs_rhol}, f.rs_zu, f.rs_zd,
                                  {f.rs_t, f.rs_tl}, L_RS) == EX_DOWN)
                tmin = 0.0f;
            else
                st = BL_STOP;
        }
    }
    if (!f.has_block) return st;
    if (st == BL_PATIENT && !(v.dz > 0.0f)) {
        ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
        st = BL_STOP;
    }
    const bool face = st == BL_PATIENT;
    const float t = (f.blk_zu - v.pz) / v.dz;
    const float qx = fmaf(t, v.dx, v.px), qy = fmaf(t, v.dy, v.py);
    const float tx = f.blk_t / v.dz;
    bool open;
    float te;
    block_side<D>(f, poly, face, qx, qy, v.dx, v.dy, v.dz, 0.0f, tx, 0.0f, true, open, te);
    if (!face) return st;
    if (open && te >= tx) {   // straight through the opening
        tmin = (f.blk_zd - v.pz) / v.dz;
        return BL_PATIENT;
    }
    if (!open && sur && sur->enabled && !(D && f.div)) {
        // enters through brass: far enough from the opening's edge, the
        // learned surrogate takes over the traversal (queued for it)
        const float de = f.nv >= 3 ? dist_to_polygon(poly, f.nv, qx, qy) : 1000.0f;
        if (de >= sur->d_fallback) {
            const unsigned long long slot = atomicAdd(sur->count, 1ull);
            if (slot < sur->capacity) {
                DeferRec r;
                r.spot = v.spot;
                r.hist = v.hist;
                r.nblk = v.nblk;
                r.tag = tag;
                r.x = qx;
                r.y = qy;
                r.u = v.dx;
                r.v = v.dy;
                r.w = v.dz;
                r.E = v.E;
                r.Elo = v.Elo;
                r.pzlo = v.pzlo;
                r.d_edge = de;
                r.thick = f.blk_t;
                r.pad[0] = r.pad[1] = 0.0f;
                sur->rec[slot] = r;
                return BL_DEFER;
            }
        }
    }
    v.px = qx;
    v.py = qy;
    v.pz = 0.0f;
    v.pzlo = 0.0f;
    return BL_BLOCK;
}

// range shifter and block of one lane's particle: true when it goes on to
// the patient with tmin set
template <bool X, bool D>
__device__ bool beamline(Lane &v, bool on, Acc &acc, float scale, const Tabs &T, const float2 *poly, const FieldDev &f,
                         float &tmin, const SurDev *sur) {
    const int st = beam_entry<X, D>(v, on, acc, scale, T, poly, f, tmin, sur, 0u);
    if (!f.has_block) return st == BL_PATIENT;
    const bool down = block_transport<X, D>(v, st == BL_BLOCK, acc, scale, T, poly, f);
    if (down) tmin = 0.0f;
    return down || st == BL_PATIENT;
}

// ------------------------------------------------------------ patient
// CT calibration: density piecewise linear through (-1000, 0.00121)
// (0, 1) (1000, 1.6) (1500, 1.85) (3071, 2.8); class air / tissue / bone.
// The density is a pair: node values and slopes are FP64 constants split at
// compile time, the CT number is an exact integer.
struct PairC {
    float h, l;
};
constexpr PairC pairc(double x) { return {(float)x, (float)(x - (double)(float)x)}; }
constexpr PairC kCalY[4] = {pairc(0.00121), pairc(1.0), pairc(1.6), pairc(1.85)};
constexpr PairC kCalB[4] = {pairc((1.0 - 0.00121) / 1000.0), pairc(0.6 / 1000.0), pairc(0.25 / 500.0),
                            pairc(0.95 / 1571.0)};
constexpr float kCalX[4] = {-1000.0f, 0.0f, 1000.0f, 1500.0f};

template <bool X>
__device__ __forceinline__ DF hu_density(int hu, int &m) {
    const int hc = min(max(hu, -1000), 3071);
    m = hu < -900 ? DM_AIR : hu < 150 ? DM_WATER : DM_BONE;
    if (!X) {
        // physics mode: the same piecewise-linear calibration as a sum of
        // clamped segments (register arithmetic; a per-segment lookup of the
        // nodes compiles to two dependent memory loads per step)
        const float x = (float)hc;
        float r = fmaf(kCalB[0].h, fminf(x, 0.0f) + 1000.0f, kCalY[0].h);
        r = fmaf(kCalB[1].h, fminf(fmaxf(x, 0.0f), 1000.0f), r);
        r = fmaf(kCalB[2].h, fminf(fmaxf(x - 1000.0f, 0.0f), 500.0f), r);
        r = fmaf(kCalB[3].h, fmaxf(x - 1500.0f, 0.0f), r);
        return {r, 0.0f};
    }
    const int k = hc <= 0 ? 0 : hc <= 1000 ? 1 : hc <= 1500 ? 2 : 3;
    const PairC y = k == 0 ? kCalY[0] : k == 1 ? kCalY[1] : k == 2 ? kCalY[2] : kCalY[3];
    const PairC b = k == 0 ? kCalB[0] : k == 1 ? kCalB[1] : k == 2 ? kCalB[2] : kCalB[3];
    const float x0 = k == 0 ? kCalX[0] : k == 1 ? kCalX[1] : k == 2 ? kCalX[2] : kCalX[3];
    return df_add({y.h, y.l}, df_mul_f({b.h, b.l}, (float)hc - x0));
}

__device__ __forceinline__ void hu_material(int hu, int &m, float &rho) {
    const DF d = hu_density<true>(hu, m);
    rho = d.h + d.l;
}

// keep a voxel-local coordinate inside [0, sp]
template <bool X>
__device__ __forceinline__ void clamp_local(float &h, float &l, float sp) {
    if constexpr (!X) {
        h = __builtin_amdgcn_fmed3f(h, 0.0f, sp);
    } else {
        if (h < 0.0f || (h == 0.0f && l < 0.0f)) { h = 0.0f; l = 0.0f; }
        else if (h > sp || (h == sp && l > 0.0f)) { h = sp; l = 0.0f; }
    }
}

// position of a VP inside the CT grid between steps
struct PState {
    int idx[3];
    uint32_t vox;   // linear index of voxel idx
    uint32_t cell;  // its CT number (X) or the bits of its density (CT geometry)
};

// Between two CT numbers that the calibration assigns to different materials
// (-901 | -900 and 149 | 150): it grows with the CT number, so in physics mode
// the density tells the material.
constexpr float kRhoTissue = 0.1006f, kRhoBone = 1.0897f;

template <bool X>
__device__ __forceinline__ uint32_t cell_of(const GeomDev &g, uint32_t vox) {
    if constexpr (X) return g.kind == 1 ? (uint32_t)(int)g.hu[vox] : 0u;
    return __float_as_uint(g.kind == 1 ? g.rho[vox] : 1.0f);
}

// Entry into the CT grid: beam frame -> CT frame with the scenario shift,
// ray-box intersection from the last exit plane (tmin), voxel-local
// coordinates.  Returns false when the VP misses the grid (its energy goes
// to the escaped ledger).
template <bool X>
__device__ bool patient_enter(Lane &v, Acc &acc, float scale, const GeomDev &g, const FieldDev &f,
                              const float *shift, float tmin, PState &ps) {
    float p[3], d[3];
    {
        const float bx = v.px, by = v.py, bz = v.pz;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            p[k] = (f.iso[k] + (bx * f.ex[k] + by * f.ey[k] + bz * f.ez[k])) - shift[k];
            d[k] = v.dx * f.ex[k] + v.dy * f.ey[k] + v.dz * f.ez[k];
        }
    }
    const int n[3] = {g.nx, g.ny, g.nz};
    float hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) hi[k] = g.lo[k] + n[k] * g.sp[k];
    float tnear = -INFINITY, tfar = INFINITY;
    int axn = -1;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (d[k] == 0.0f) {
            if (p[k] < g.lo[k] || p[k] >= hi[k]) {
                ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
                return false;
            }
            continue;
        }
        const float t1 = (g.lo[k] - p[k]) / d[k], t2 = (hi[k] - p[k]) / d[k];
        const float a = fminf(t1, t2), b = fmaxf(t1, t2);
        if (a > tnear) { tnear = a; axn = k; }
        tfar = fminf(tfar, b);
    }
    const float t0 = fmaxf(tnear, tmin);
    if (!(tfar > t0)) {
        ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
        return false;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k] = fmaf(t0, d[k], p[k]);
    if (t0 == tnear) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == axn) p[k] = d[k] > 0.0f ? g.lo[k] : hi[k];
    }
    int idx[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float c = floorf((p[k] - g.lo[k]) / g.sp[k]);
        idx[k] = !(c >= 0.0f) ? 0 : c > (float)(n[k] - 1) ? n[k] - 1 : (int)c;   // NaN -> 0
    }
    // From here the position is kept relative to the lower corner of the
    // current voxel (0 <= u_k <= spacing_k): FP32 resolves it to ~1e-7 of a
    // voxel wherever the voxel sits, so sub-voxel steps near the end of range
    // do not inherit the rounding of large absolute coordinates.
    {
        float u[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            u[k] = fminf(fmaxf(p[k] - (g.lo[k] + (float)idx[k] * g.sp[k]), 0.0f), g.sp[k]);
            if (t0 == tnear && k == axn) u[k] = d[k] > 0.0f ? 0.0f : g.sp[k];
        }
        v.px = u[0]; v.py = u[1]; v.pz = u[2];
        v.pxlo = v.pylo = v.pzlo = 0.0f;
    }
    v.dx = d[0]; v.dy = d[1]; v.dz = d[2];
    ps.idx[0] = idx[0];
    ps.idx[1] = idx[1];
    ps.idx[2] = idx[2];
    ps.vox = (uint32_t)idx[0] + (uint32_t)g.nx * ((uint32_t)idx[1] + (uint32_t)g.ny * (uint32_t)idx[2]);
    ps.cell = cell_of<X>(g, ps.vox);
    return true;
}

// One condensed-history step of a VP inside the CT grid; false once its
// transport has ended (stopped, or left the grid: then the escaped ledger).
// Written for instruction count (the work queue issues VALU instructions
// without a gap): the exit face is a pair of lane masks rather than an axis
// number, per-axis updates are selects and carry-ins on those masks, the next
// voxel's density is fetched without a bounds check, and only what a lane
// rarely needs is branched over.
template <class Sink, bool X, int P = X ? 0 : -1>
__device__ __forceinline__ bool patient_step(Lane &v, Acc &acc, float scale, const Tabs &T, const GeomDev &g,
                                             float range_scale, const Sink &sink, PState &ps) {
    if (v.nsteps >= (uint32_t)MAX_STEPS) {
        ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
        return false;
    }
    int m = DM_WATER;
    DF rho = {1.0f, 0.0f};
    if constexpr (X) {
        if (g.kind == 1) rho = hu_density<true>((int)ps.cell, m);
    } else {
        rho.h = __uint_as_float(ps.cell);
        m = rho.h < kRhoTissue ? DM_AIR : rho.h < kRhoBone ? DM_WATER : DM_BONE;
    }
    const DF rho_loss = Ar<X>::mul_f(rho, range_scale);
    // exit face: the axis with the shortest FP32 distance (the first of equal
    // ones), then in pairs that distance from the pair coordinate
    const bool u0 = v.dx > 0.0f, u1 = v.dy > 0.0f, u2 = v.dz > 0.0f;
    const float a0 = u0 ? g.sp[0] : 0.0f, a1 = u1 ? g.sp[1] : 0.0f, a2 = u2 ? g.sp[2] : 0.0f;
    auto dist = [](float a, float p, float l, float d) {
        float t = a - p;
        if constexpr (X) t -= l;
        return fmaxf(t * __builtin_amdgcn_rcpf(d), 0.0f);
    };
    float t0 = dist(a0, v.px, v.pxlo, v.dx), t1 = dist(a1, v.py, v.pylo, v.dy), t2 = dist(a2, v.pz, v.pzlo, v.dz);
    if (v.dx == 0.0f) t0 = INFINITY;
    if (v.dy == 0.0f) t1 = INFINITY;
    if (v.dz == 0.0f) t2 = INFINITY;
    const bool c1 = t1 < t0;
    const float t01 = c1 ? t1 : t0;
    const bool is2 = t2 < t01, is1 = !is2 && c1, is0 = !is2 && !c1;
    const bool up = (is0 && u0) || (is1 && u1) || (is2 && u2);
    DF dg = {is2 ? t2 : t01, 0.0f};
    if constexpr (X) {
        const float pa = is0 ? v.px : is1 ? v.py : v.pz;
        const float la = is0 ? v.pxlo : is1 ? v.pylo : v.pzlo;
        const float da = is0 ? v.dx : is1 ? v.dy : v.dz;
        const float aa = is0 ? a0 : is1 ? a1 : a2;
        if (dg.h < INFINITY) {
            dg = df_div_f(df_sub({aa, 0.0f}, {pa, la}), da);
            if (!(dg.h > 0.0f)) dg = {0.0f, 0.0f};
        }
    }
    // what lies behind the face this step may cross is fetched now, so its
    // latency overlaps the step's arithmetic
    const int stride = is2 ? g.nx * g.ny : is1 ? g.nx : 1;
    const int64_t nvox = voxel_behind(ps.vox, stride, up);
    uint32_t ncell = ps.cell;
    if (g.kind == 1) {
        if constexpr (X) {
            // (an index of the grid: the CT numbers have no margin)
            const int ia = is0 ? ps.idx[0] : is1 ? ps.idx[1] : ps.idx[2];
            const int na = is0 ? g.nx : is1 ? g.ny : g.nz;
            if (up ? ia + 1 < na : ia > 0) ncell = (uint32_t)(int)g.hu[nvox];
        } else {
            ncell = __float_as_uint(g.rho[nvox]);
        }
    }
    float dep, esc, let;
    const int st = phys_step<false, X, P>(v, T, m, rho_loss, rho.h, dg, dep, esc, let);
    const long long qd = to_fixed_deposit(dep, scale);
    if (qd != 0) sink.add(ps.vox, ps.idx, qd);
    if constexpr (Sink::kLet) {
        if (sink.let) {
            // numerator of the dose-averaged LET: rne(dep * LET * w/N * 2^(k - kLetShift))
            const long long ql = to_fixed(dep * let, scale * (1.0f / (float)(1 << kLetShift)));
            if (ql != 0) sink.add_let(ps.vox, ps.idx, ql);
        }
    }
    acc.led[L_GRID] += qd;
    if (esc != 0.0f) ledger_add(acc, L_NUC, esc, scale);
    if (st == ST_STOP) return false;
    const bool geo = st == ST_GEO, g0 = geo && is0, g1 = geo && is1, g2 = geo && is2;
    ps.idx[0] += (g0 && u0 ? 1 : 0) - (g0 && !u0 ? 1 : 0);
    ps.idx[1] += (g1 && u1 ? 1 : 0) - (g1 && !u1 ? 1 : 0);
    ps.idx[2] += (g2 && u2 ? 1 : 0) - (g2 && !u2 ? 1 : 0);
    if ((uint32_t)ps.idx[0] >= (uint32_t)g.nx || (uint32_t)ps.idx[1] >= (uint32_t)g.ny ||
        (uint32_t)ps.idx[2] >= (uint32_t)g.nz) {
        ledger_add(acc, L_ESCAPED, v.E + v.Elo, scale);
        return false;
    }
    // near face of the next voxel, exactly
    if (g0) { v.px = g.sp[0] - a0; v.pxlo = 0.0f; }
    if (g1) { v.py = g.sp[1] - a1; v.pylo = 0.0f; }
    if (g2) { v.pz = g.sp[2] - a2; v.pzlo = 0.0f; }
    ps.vox = geo ? (uint32_t)nvox : ps.vox;
    ps.cell = geo ? ncell : ps.cell;
    clamp_local<X>(v.px, v.pxlo, g.sp[0]);
    clamp_local<X>(v.py, v.pylo, g.sp[1]);
    clamp_local<X>(v.pz, v.pzlo, g.sp[2]);
    return true;
}

template <class Sink, bool X>
__device__ void patient(Lane &v, Acc &acc, float scale, const Tabs &T, const GeomDev &g,
                        const FieldDev &f, const float *shift, float range_scale, const Sink &sink,
                        float tmin) {
    PState ps;
    if (!patient_enter<X>(v, acc, scale, g, f, shift, tmin, ps)) return;
    while (patient_step<Sink, X>(v, acc, scale, T, g, range_scale, sink, ps)) {
    }
}

// ------------------------------------------------------------ source
__device__ void source(Lane &v, const SpotDev &sp, float vsad) {
    const uint4 w = draw(v);
    const float r = sqrtf(-2.0f * logf(unit_open(w.x)));
    float sn, c;
    sincospif(2.0f * unit_open(w.y), &sn, &c);
    v.px = fmaf(sp.sigma, r * c, sp.x);
    v.py = fmaf(sp.sigma, r * sn, sp.y);
    v.pz = 0.0f;
    v.pzlo = 0.0f;
    v.pxlo = v.pylo = 0.0f;
    v.dx = 0.0f; v.dy = 0.0f; v.dz = 1.0f;
    if (vsad > 0.0f) {
        // along the line from the virtual source through the start point
        const float inv = 1.0f / sqrtf(fmaf(v.px, v.px, fmaf(v.py, v.py, vsad * vsad)));
        v.dx = v.px * inv;
        v.dy = v.py * inv;
        v.dz = vsad * inv;
    }
    v.E = sp.e0;
    v.Elo = 0.0f;
    if (sp.esig > 0.0f) {
        const float z = 1.41421356237f * erfinvf(2.0f * unit_open(w.z) - 1.0f);
        v.E = fminf(fmaxf(fmaf(sp.esig, z, sp.e0), kELo), sp.emax);
    }
}

__device__ __forceinline__ int find_spot(const unsigned long long *off, int n, unsigned long long item) {
    int lo = 0, hi = n;   // off[lo] <= item < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= item) lo = mid; else hi = mid;
    }
    return lo;
}

// LDS of the kernels that run a whole history, all tables and the aperture's
// vertices: the vertices are allocated by the launch, as many as there are.  With
// up to 256 of them four workgroups of 256 threads fit a CU in physics mode and
// three in double-float mode; with room for 1024 in every workgroup it was three
// and two, and a run of 1.5e5 to 2.6e5 histories took a second round of them
// (10 mm opening: 2.3e5 histories 1.13 ms against 0.83, without processes 1.5e5
// 0.77 against 0.50).
constexpr int whole_lds(bool x) { return (TAB_HI_FLOATS + (x ? tab_lo_floats(NMAT) : 0)) * 4; }
static_assert(4 * (whole_lds(false) + 256 * 8) <= 160 * 1024, "four workgroups a CU");
static_assert(3 * (whole_lds(true) + 256 * 8) <= 160 * 1024, "three workgroups a CU");

template <bool X>
__global__ __launch_bounds__(512) void transport_kernel(GeomDev g, FieldDev f, LaunchDev L) {
    __shared__ __attribute__((aligned(16))) float hi[TAB_HI_FLOATS], lo[X ? tab_lo_floats(NMAT) : 1];
    extern __shared__ __attribute__((aligned(16))) float2 poly[];   // f.nv with a block
    stage_tables<X, NMAT>(hi, lo, L.tables, 0);
    const Tabs T{hi, lo, DM_PMMA, DM_BRASS};
    if (f.has_block)
        for (int i = threadIdx.x; i < f.nv; i += blockDim.x) poly[i] = f.poly[i];
    __syncthreads();

    Acc acc;
#pragma unroll
    for (int j = 0; j < NLEDGER; ++j) acc.led[j] = 0;
    acc.steps = acc.hist = 0;
    const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
    for (unsigned long long item = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x;
         item < L.n_items; item += stride) {
        const int s = find_spot(L.item_off, L.n_spots, item);
        const SpotDev sp = L.spots[s];
        Lane v;
        v.k0 = L.key0;
        v.k1 = L.key1;
        v.spot = (uint32_t)s;
        v.hist = (uint32_t)(L.batch + (unsigned long long)L.n_batches * (item - L.item_off[s]));
        v.nblk = 0;
        v.nsteps = 0;
        v.physics = L.physics;
        source(v, sp, f.vsad);
        float tmin;
        if (beamline<X, true>(v, true, acc, sp.scale, T, poly, f, tmin, &L.sur))
            patient<DenseSink, X>(v, acc, sp.scale, T, g, f, L.shift, L.range_scale, DenseSink{L.tally, L.let_tally},
                                  tmin);
        acc.steps += v.nsteps;
        acc.hist += 1;
    }
    // wavefront reduction of the ledgers, one atomic per wavefront
#pragma unroll
    for (int j = 0; j < NLEDGER; ++j) {
        long long x = acc.led[j];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if ((threadIdx.x & 63) == 0 && x != 0) atomicAdd(L.ledger + j, (unsigned long long)x);
    }
    unsigned long long st = acc.steps, hs = acc.hist;
    for (int o = 32; o > 0; o >>= 1) {
        st += __shfl_xor(st, o, 64);
        hs += __shfl_xor(hs, o, 64);
    }
    if ((threadIdx.x & 63) == 0 && hs != 0) {
        atomicAdd(L.stats + 0, st);
        atomicAdd(L.stats + 1, hs);
    }
}

// ------------------------------------------------------------ CSR mode
// A VP staged at its entry into the CT grid (64 B, four 16-byte words):
// voxel-local position, direction in the CT frame, energy pair, Philox block
// counter, history, step count, voxel (linear, per axis) and its CT number or density
// (in dense runs, whose rows hold several spots, the spot instead).
struct alignas(16) StagedVP {
    float px, py, pz, dx;
    float dy, dz, E, Elo;
    uint32_t nblk, hist, nsteps, vox;
    int i0, i1, i2;
    uint32_t cell;
};
static_assert(sizeof(StagedVP) == 4 * kStageFields, "staging record");

template <bool DENSE>
__device__ __forceinline__ void store_staged(StagedVP *to, const Lane &v, const PState &ps) {
    StagedVP s;
    s.px = v.px; s.py = v.py; s.pz = v.pz; s.dx = v.dx;
    s.dy = v.dy; s.dz = v.dz; s.E = v.E; s.Elo = v.Elo;
    s.nblk = v.nblk; s.hist = v.hist; s.nsteps = v.nsteps; s.vox = ps.vox;
    s.i0 = ps.idx[0]; s.i1 = ps.idx[1]; s.i2 = ps.idx[2]; s.cell = DENSE ? v.spot : ps.cell;
    *to = s;
}

// Word by word: single-word loads are not merged into 4-register tuples, so
// each field can land in the register the step loop carries it in.
template <bool DENSE, bool X>
__device__ __forceinline__ void load_staged(const StagedVP *from, const GeomDev &g, Lane &v, PState &ps) {
    const uint32_t *rw = reinterpret_cast<const uint32_t *>(from);
    auto ld = [&](int i) { return __hip_atomic_load(rw + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
    v.px = __uint_as_float(ld(0)); v.py = __uint_as_float(ld(1));
    v.pz = __uint_as_float(ld(2)); v.dx = __uint_as_float(ld(3));
    v.dy = __uint_as_float(ld(4)); v.dz = __uint_as_float(ld(5));
    v.E = __uint_as_float(ld(6)); v.Elo = __uint_as_float(ld(7));
    v.pxlo = v.pylo = v.pzlo = 0.0f;
    v.nblk = ld(8); v.hist = ld(9); v.nsteps = ld(10);
    ps.vox = ld(11);
    ps.idx[0] = (int)ld(12); ps.idx[1] = (int)ld(13); ps.idx[2] = (int)ld(14);
    if constexpr (DENSE) {
        v.spot = ld(15);
        ps.cell = cell_of<X>(g, ps.vox);
    } else {
        ps.cell = ld(15);
    }
}

constexpr uint32_t kRowNone = 0xFFFFFFFFu;   // workgroup row word: no row yet
constexpr uint32_t kRowPick = 0xFFFFFFFDu;   // a wave is picking the next row
constexpr uint32_t kRowEnd = 0xFFFFFFFEu;    // no work left in the epoch
constexpr uint32_t kTileBusy = 0xFFFFFFFFu;  // tile users field while it is added out
constexpr int kStealRows = 2048;             // last rows of a round that are looked through for work

__device__ __forceinline__ unsigned long long rd_lds64(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Adds the tile into its row's grid and clears it; one wave.
template <bool MARKS, bool LET>
__device__ void tile_flush(uint32_t *tile, const TileSink<MARKS, LET> &sink, const GeomDev &g, int lane) {
    const uint32_t n0 = sink.n0, n1 = sink.n1, tn = n0 * n1 * sink.n2;
    // e / n0 and e / (n0 n1) by FP32 reciprocals: exact, entries < 2^16
    const float i0 = 1.0f / (float)n0, i1 = 1.0f / (float)n1;
    // a voxel per lane, with LET per pair of lanes (dose, LET numerator)
    constexpr uint32_t per = LET ? 32u : 64u;
    const uint32_t part = LET ? (uint32_t)lane >> 5 : 0u;
    uint32_t *const mine = tile + (LET ? part * sink.let_off : 0u);
    for (uint32_t e0 = (uint32_t)lane & (per - 1u); e0 < tn; e0 += 4u * per) {
        uint32_t q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = e0 + per * j < tn ? mine[e0 + per * j] : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (q[j] == 0u) continue;
            const uint32_t e = e0 + per * j;
            const uint32_t e1 = (uint32_t)(((float)e + 0.5f) * i0), u0 = e - n0 * e1;
            const uint32_t u2 = (uint32_t)(((float)e1 + 0.5f) * i1), u1 = e1 - n1 * u2;
            const uint32_t v = (uint32_t)sink.lo0 + u0 + (uint32_t)g.nx * ((uint32_t)sink.lo1 + u1 +
                                                                           (uint32_t)g.ny * ((uint32_t)sink.lo2 + u2));
            mine[e] = 0u;
            if constexpr (LET) atomicAdd(sink.gs.grid + 2 * (size_t)v + part, (unsigned long long)q[j]);
            else sink.put(v, (long long)q[j]);
        }
    }
}

// Wave-wide ledger sums into one scenario's ledger, one atomic per entry and
// wave; clears the accumulators.
__device__ __forceinline__ void flush_ledger(Acc &acc, unsigned long long *ledger, int lane) {
#pragma unroll
    for (int k = 0; k < NLEDGER; ++k) {
        long long x = acc.led[k];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if (lane == 0 && x != 0) atomicAdd(ledger + k, (unsigned long long)x);
        acc.led[k] = 0;
    }
}

__device__ __forceinline__ void flush_stats(Acc &acc, unsigned long long *stats, int lane) {
    unsigned long long st = acc.steps, hs = acc.hist;
    for (int o = 32; o > 0; o >>= 1) {
        st += __shfl_xor(st, o, 64);
        hs += __shfl_xor(hs, o, 64);
    }
    if (lane == 0 && (st | hs) != 0) {
        atomicAdd(stats + 0, st);
        atomicAdd(stats + 1, hs);
    }
    acc.steps = acc.hist = 0;
}

// First staged record of a row in this round (its groups start at g_begin).
__device__ __forceinline__ size_t stage_base(const QueueDev &Q, uint32_t r) {
    const unsigned long long a = Q.grp_off[r];
    return (size_t)((a > Q.g_begin ? a : Q.g_begin) - Q.g_begin) * 64u;
}

// Appends the particles of the lanes with `in` to the staged lists of their
// rows: ballot compaction per row, one returning atomic per row and wave.
template <bool DENSE>
__device__ __forceinline__ void stage_out(const QueueDev &Q, bool in, uint32_t r, const Lane &v, const PState &ps,
                                          int lane) {
    for (unsigned long long todo = __ballot(in); todo;) {
        const uint32_t rr = (uint32_t)__builtin_amdgcn_readlane((int)r, __ffsll((long long)todo) - 1);
        const bool mine = in && r == rr;
        const unsigned long long m = __ballot(mine);
        unsigned int at = 0;
        if (lane == 0) at = atomicAdd(&Q.ctl[rr].staged, (unsigned int)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (mine)
            store_staged<DENSE>(reinterpret_cast<StagedVP *>(Q.stage) + stage_base(Q, rr) + at +
                                    (uint32_t)__popcll(m & ((1ull << lane) - 1ull)),
                                v, ps);
        todo &= ~m;
    }
}

// Beam line of a round's histories: source, range shifter, aperture block and
// CT entry; the particles that enter the grid are appended to their row's
// staged list.  A wave takes runs of groups of 64 histories of one row, the
// lanes in lock step through source and range shifter.  Most particles are
// then through the opening or stop; those that meet the block's brass or walls
// are pushed onto a small stack of the wave in LDS, and whenever it holds a
// wavefull they are stepped through the block together, until half of them
// are out and the rest goes back onto the stack.  So the block, whose
// traversals take from one to dozens of steps, runs with at least half of its
// lanes busy instead of the one or two that a group of 64 has left at its
// end, and the CT entries of a wavefull are done at once.  Bound by VALU issue
// and the table reads' latency at 12 waves per CU.  Measured on the 13-scenario
// matrix of the 0.4 cc head case (4.0e7 histories): 33.6 ms with each group's
// traversals run to their end in the group (12 % of the lanes busy), 9.3 ms
// this way with the edge searches divided among the lanes (47 %).
constexpr int kBlkStack = 128;   // up to 63 waiting + 64 pushed by a group

template <bool X, bool D, bool DENSE>
__global__ __launch_bounds__(256, 3) void beam_kernel(GeomDev g, QueueDev Q) {
    // words of a waiting particle (the spot only in dense runs, the low part of the depth only when X)
    constexpr int kSpot = 13, kLow = DENSE ? 14 : 13, kW = kLow + (X ? 1 : 0);
    __shared__ __attribute__((aligned(16))) float hi[tab_hi_floats(2)], lo[X ? tab_lo_floats(2) : 4];
    __shared__ float2 poly[POLY_LDS];
    __shared__ uint32_t stacks[4][kW][kBlkStack];
    stage_tables<X, 2>(hi, lo, Q.tables, DM_PMMA);   // PMMA and brass
    const Tabs T{hi, lo, 0, 1};
    for (int i = threadIdx.x; i < Q.n_poly_total; i += blockDim.x) poly[i] = Q.polys[i];
    __syncthreads();

    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned long long below = (1ull << lane) - 1ull;
    uint32_t(*const stk)[kBlkStack] = stacks[wv];
    const unsigned long long nwave = (unsigned long long)gridDim.x * (blockDim.x >> 6);
    unsigned long long run = (unsigned long long)blockIdx.x * (blockDim.x >> 6) + wv;
    const uint32_t row_end = (uint32_t)(Q.row_begin + Q.n_rows);
    Acc acc;
#pragma unroll
    for (int k = 0; k < NLEDGER; ++k) acc.led[k] = 0;
    acc.steps = acc.hist = 0;
    int cur_scen = -1, cur_field = -1;
    unsigned long long G = 0, G1 = 0;   // groups left of the current run
    uint32_t r = 0;                     // row of group G
    int nst = 0;                        // particles on the stack
    bool more = true;
    // moves on to the next group's row; the run's first row by bisection
    auto advance = [&]() {
        if (G >= G1) {
            G = Q.g_begin + run * (unsigned long long)Q.beam_groups;
            run += nwave;
            G1 = min(G + (unsigned long long)Q.beam_groups, Q.g_end);
            more = G < Q.g_end;
            if (!more) return;
            r = (uint32_t)Q.row_begin;
            for (uint32_t h = row_end; h - r > 1u;) {   // grp_off[r] <= G < grp_off[r + 1]
                const uint32_t mid = (r + h) >> 1;
                if (Q.grp_off[mid] <= G) r = mid;
                else h = mid;
            }
        }
        while (G >= Q.grp_off[r + 1]) ++r;   // (rows without histories have no group)
    };
    advance();
    for (;;) {
        bool same = false;   // the next group's row shares the field and the scenario of what waits
        if (more) same = Q.rows[r].scen == cur_scen && Q.rows[r].field == cur_field;
        if (more && (nst == 0 || (same && nst < 64))) {
            const RowDev row = Q.rows[r];
            if (row.scen != cur_scen) {
                if (cur_scen >= 0) flush_ledger(acc, Q.ledger + (size_t)cur_scen * NLEDGER, lane);
                cur_scen = row.scen;
            }
            cur_field = row.field;
            const FieldDev &f = Q.fields[row.field];
            const unsigned long long h = (G - Q.grp_off[r]) * 64ull + lane;
            const bool on = h < row.n_hist;
            uint32_t spot = row.spot, hist = (uint32_t)h, spot_at = row.spot_global;
            if constexpr (DENSE) {
                // the row's items run through the batch's spots: the spot of
                // the group's first item by bisection, the lanes' from there
                const unsigned long long *off = Q.item_off + (size_t)row.batch * ((size_t)Q.n_spots + 1);
                const unsigned long long i0 = row.item0 + (h - lane), item = row.item0 + h;
                uint32_t s = 0;
                for (uint32_t e = (uint32_t)Q.n_spots; e - s > 1u;) {   // off[s] <= i0 < off[e]
                    const uint32_t mid = (s + e) >> 1;
                    if (off[mid] <= i0) s = mid;
                    else e = mid;
                }
                s = (uint32_t)__builtin_amdgcn_readfirstlane((int)s);
                if (on)
                    while (item >= off[s + 1]) ++s;
                spot = spot_at = Q.spot_order[s];
                hist = row.batch + (uint32_t)Q.n_batches * (uint32_t)(item - off[s]);
            }
            const SpotDev sp = Q.spots[spot_at];
            Lane v;
            PState ps;
            v.k0 = Q.key0;
            v.k1 = Q.seed_hi ^ row.field_id;
            v.spot = spot;
            v.physics = Q.physics;
            v.hist = hist;
            v.nblk = 0;
            v.nsteps = 0;
            float tmin;
            if (on) source(v, sp, D ? f.vsad : 0.0f);
            const int st = beam_entry<X, D>(v, on, acc, sp.scale, T, poly + Q.poly_off[row.field], f, tmin, &Q.sur,
                                            (uint32_t)(r - Q.row_begin) + Q.slot0);
            const unsigned long long blk = __ballot(st == BL_BLOCK);
            if (st == BL_BLOCK) {
                const int at = nst + __popcll(blk & below);
                stk[0][at] = __float_as_uint(v.px); stk[1][at] = __float_as_uint(v.py);
                stk[2][at] = __float_as_uint(v.pz); stk[3][at] = __float_as_uint(v.dx);
                stk[4][at] = __float_as_uint(v.dy); stk[5][at] = __float_as_uint(v.dz);
                stk[6][at] = __float_as_uint(v.E); stk[7][at] = __float_as_uint(v.Elo);
                stk[8][at] = v.nblk; stk[9][at] = v.hist; stk[10][at] = v.nsteps;
                stk[11][at] = 0u; stk[12][at] = r;
                if constexpr (DENSE) stk[kSpot][at] = v.spot;
                if constexpr (X) stk[kLow][at] = __float_as_uint(v.pzlo);
            }
            nst += __popcll(blk);
            const bool in = st == BL_PATIENT && patient_enter<X>(v, acc, sp.scale, g, f, Q.scen[row.scen].shift, tmin, ps);
            if (on) {
                if (!in && st != BL_BLOCK) acc.steps += v.nsteps;
                acc.hist += 1;
            }
            stage_out<DENSE>(Q, in, r, v, ps, lane);
            ++G;
            advance();
            continue;
        }
        if (nst == 0) break;
        // the top of the stack through the block
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int take = min(nst, 64);
        nst -= take;
        const bool on = lane < take;
        const FieldDev &f = Q.fields[cur_field];
        const float2 *fpoly = poly + Q.poly_off[cur_field];
        Lane v;
        uint32_t it = 0, vr = 0;
        float scale = 0.0f;
        if (on) {
            const int at = nst + lane;
            v.px = __uint_as_float(stk[0][at]); v.py = __uint_as_float(stk[1][at]);
            v.pz = __uint_as_float(stk[2][at]); v.dx = __uint_as_float(stk[3][at]);
            v.dy = __uint_as_float(stk[4][at]); v.dz = __uint_as_float(stk[5][at]);
            v.E = __uint_as_float(stk[6][at]); v.Elo = __uint_as_float(stk[7][at]);
            v.nblk = stk[8][at]; v.hist = stk[9][at]; v.nsteps = stk[10][at];
            it = stk[11][at];
            vr = stk[12][at];
            v.pzlo = 0.0f;
            if constexpr (X) v.pzlo = __uint_as_float(stk[kLow][at]);
            const RowDev &row = Q.rows[vr];
            v.spot = DENSE ? stk[kSpot][at] : row.spot;
            v.k0 = Q.key0;
            v.k1 = Q.seed_hi ^ row.field_id;
            v.physics = Q.physics;
            scale = Q.spots[DENSE ? v.spot : row.spot_global].scale;
        }
        // half of a wavefull may go back when more can follow it
        const int park = nst > 0 || (more && same) ? 32 : 0;
        int st = on ? BK_IN : BK_GONE;
        do {
            const bool in = st == BK_IN;
            const int s = block_step<X, D>(v, in, it, acc, scale, T, fpoly, f);
            if (in) st = s;
        } while (__popcll(__ballot(st == BK_IN)) > park);
        PState ps;
        const bool in = st == BK_DOWN && patient_enter<X>(v, acc, scale, g, f, Q.scen[cur_scen].shift, 0.0f, ps);
        if (on && st != BK_IN && !in) acc.steps += v.nsteps;
        stage_out<DENSE>(Q, in, vr, v, ps, lane);
        const unsigned long long back = __ballot(st == BK_IN);
        if (st == BK_IN) {
            const int at = nst + __popcll(back & below);
            stk[0][at] = __float_as_uint(v.px); stk[1][at] = __float_as_uint(v.py);
            stk[2][at] = __float_as_uint(v.pz); stk[3][at] = __float_as_uint(v.dx);
            stk[4][at] = __float_as_uint(v.dy); stk[5][at] = __float_as_uint(v.dz);
            stk[6][at] = __float_as_uint(v.E); stk[7][at] = __float_as_uint(v.Elo);
            stk[8][at] = v.nblk; stk[9][at] = v.hist; stk[10][at] = v.nsteps;
            stk[11][at] = it;
            stk[12][at] = vr;
            if constexpr (DENSE) stk[kSpot][at] = v.spot;
            if constexpr (X) stk[kLow][at] = __float_as_uint(v.pzlo);
        }
        nst += __popcll(back);
    }
    if (cur_scen >= 0) flush_ledger(acc, Q.ledger + (size_t)cur_scen * NLEDGER, lane);
    flush_stats(acc, Q.stats, lane);
}

// LDS tile box of a round's rows (voxel indices, x fastest), one wave per row,
// from up to 256 of the particles that the beam line staged for it: along the
// main axis of their mean direction from the CT entry to 5 mm of water past
// 1.05 x the range of the most energetic one in the CT along the mean ray (the
// air before the head uses up no range), and across it around the mean ray's
// middle, as many standard deviations of the particles' spread there (with 3 %
// of the depth for the scattering in the patient) as fit into cap voxels, 4 at
// most.  The particles know what the spot's parameters do not: the aperture
// cuts an edge spot's beam to one side, and the range shifter's scattering
// widens it.  No box (tn = 0) when nothing fits.  (Any box gives the same sums.)
__global__ __launch_bounds__(256) void tile_box_kernel(GeomDev g, QueueDev Q, RowDev *rows) {
    const int lane = threadIdx.x & 63;
    const uint32_t rl = blockIdx.x * (blockDim.x >> 6) + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (rl >= (uint32_t)Q.n_rows) return;
    const uint32_t r = (uint32_t)Q.row_begin + rl;
    const uint32_t n = Q.ctl[r].staged;
    const StagedVP *stg = reinterpret_cast<const StagedVP *>(Q.stage) + stage_base(Q, r);
    const int gn[3] = {g.nx, g.ny, g.nz};
    auto sum = [](float x) {
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        return x;
    };
    // sums over the sample: directions, positions (mm from the grid's corner), largest energy
    const uint32_t ns = min(n, 256u), step = ns ? max(n / ns, 1u) : 1u;
    float d[3] = {0, 0, 0}, p[3] = {0, 0, 0}, emax = 0.0f;
    for (uint32_t j = (uint32_t)lane; j < ns; j += 64) {
        const StagedVP q = stg[j * step];
        d[0] += q.dx; d[1] += q.dy; d[2] += q.dz;
        p[0] += q.i0 * g.sp[0] + q.px; p[1] += q.i1 * g.sp[1] + q.py; p[2] += q.i2 * g.sp[2] + q.pz;
        emax = fmaxf(emax, q.E);
    }
    for (int o = 32; o > 0; o >>= 1) emax = fmaxf(emax, __shfl_xor(emax, o, 64));
    const float in = ns ? 1.0f / (float)ns : 0.0f;
    for (int k = 0; k < 3; ++k) {
        d[k] = sum(d[k]) * in;
        p[k] = sum(p[k]) * in;
    }
    int a = 0;
    for (int k = 1; k < 3; ++k)
        if (fabsf(d[k]) > fabsf(d[a])) a = k;
    int tlo[3] = {0, 0, 0}, tn[3] = {0, 0, 0};
    if (ns != 0u && fabsf(d[a]) > 1e-3f && Q.tile_cap > 0) {
        // depth along the mean ray
        const float *tab = Q.tables;
        const int i = seg_of(tab, emax);
        const float R = tab[TAB_SHARED + T_R * NE + i] + (emax - tab[TAB_E + i]) / tab[TAB_SHARED + T_SH * NE + i];
        const float need = 1.05f * R + 5.0f, rs = Q.scen[rows[r].scen].range_scale;
        const float ds = fminf(fminf(g.sp[0], g.sp[1]), g.sp[2]);
        auto cell = [&](int k, float x) { return min(max((int)floorf(x / g.sp[k]), 0), gn[k] - 1); };
        float t = 0.0f;
        if (g.kind == 1) {
            // 64 samples of the ray at a time, one per lane
            float we = 0.0f;
            for (int it = 0; it < 4096 && we < need; ++it) {
                const float tm = t + ((float)lane + 0.5f) * ds;
                float x[3];
                bool ok = true;
                for (int k = 0; k < 3; ++k) {
                    x[k] = p[k] + tm * d[k];
                    ok = ok && x[k] >= 0.0f && x[k] < gn[k] * g.sp[k];
                }
                float w = 0.0f;
                if (ok)
                    w = g.rho[(size_t)cell(0, x[0]) +
                              (size_t)g.nx * ((size_t)cell(1, x[1]) + (size_t)g.ny * (size_t)cell(2, x[2]))] * rs * ds;
                for (int o = 1; o < 64; o <<= 1) {   // inclusive prefix over the lanes
                    const float y = __shfl_up(w, o, 64);
                    if (lane >= o) w += y;
                }
                const unsigned long long past = __ballot(!ok || we + w >= need);
                if (past) {
                    t += (float)__ffsll((long long)past) * ds;
                    break;
                }
                we += __shfl(w, 63, 64);
                t += 64.0f * ds;
            }
        } else {
            t = need / rs;
        }
        // spread across the main axis at 60 % of the depth
        float var[3] = {0, 0, 0};
        for (uint32_t j = (uint32_t)lane; j < ns; j += 64) {
            const StagedVP q = stg[j * step];
            const float e[3] = {q.dx - d[0], q.dy - d[1], q.dz - d[2]};
            const float y[3] = {q.i0 * g.sp[0] + q.px - p[0], q.i1 * g.sp[1] + q.py - p[1], q.i2 * g.sp[2] + q.pz - p[2]};
            for (int k = 0; k < 3; ++k) {
                const float z = y[k] + 0.6f * t * e[k];
                var[k] += z * z;
            }
        }
        float sd[3];
        for (int k = 0; k < 3; ++k) sd[k] = sqrtf(sum(var[k]) * in) + 0.03f * 0.6f * t + 0.1f;
        for (float kap = 4.0f; kap > 0.0f; kap -= 0.1f) {
            int l[3], w[3];
            unsigned long long vol = 1;
            for (int k = 0; k < 3; ++k) {
                const float e0 = p[k], e1 = p[k] + t * d[k];
                float x0 = fminf(e0, e1), x1 = fmaxf(e0, e1);
                if (k != a) {
                    x0 -= kap * sd[k];
                    x1 += kap * sd[k];
                }
                l[k] = cell(k, x0);
                w[k] = cell(k, x1) - l[k] + 1;
                vol *= (unsigned long long)w[k];
                if (vol > (1ull << 32)) vol = 1ull << 32;
            }
            if (vol <= (unsigned long long)Q.tile_cap) {
                for (int k = 0; k < 3; ++k) {
                    tlo[k] = l[k];
                    tn[k] = w[k];
                }
                break;
            }
        }
    }
    if (lane == 0)
        for (int k = 0; k < 3; ++k) {
            rows[r].tlo[k] = tlo[k];
            rows[r].tn[k] = tn[k];
        }
}

// Patient transport of a round's staged particles.  Each row has a counter of
// drawn records; a workgroup works on one current row at a time, its waves
// drawing 64 * hist_per_lane records of it at a time, and when the row is
// exhausted one wave picks the next: a fresh row from the round's row head,
// else (work stealing) any row with records left, else the end.  A lane whose
// particle has ended takes the next drawn record as soon as refill_min lanes
// are idle (or all remaining records fit), and the wave draws again while its
// other lanes are in flight: lanes run dry only when the row does, once per
// row instead of once per chunk.  The workgroup's LDS tile holds one row's box
// at a time (RowDev::tlo/tn): a wave joins it at a draw if it holds that row
// or is free, and the last wave to leave adds it into the slot grid; waves
// that did not get it deposit straight into the slot grid.
// Draws are of one wavefull by default: more keep waves longer on rows other
// than the tile's (0.4 cc head matrix, transport of all epochs: 137, 123 and
// 114 ms at 256, 128 and 64 records a draw).  Bound by VALU issue (431
// instructions a wave-step, 0.87 of its lanes with a particle, 0.78 of the
// issued lanes at work; 93 % of the launch at 4 clocks each, and the 64-bit
// products and transcendentals take more), then by the memory-side atomics
// (1.1e10 of 2.0e10 per second).  Measured on the 13-scenario matrices, 0.4 cc /
// 8 cc head: 110 / 546 ms as one kernel with source and beam line, a drain
// after every chunk and int64 tile entries; 71.5 / 399 ms with staged draws,
// 32-bit entries and the tile joined in flight; 57 / 311 ms with the step
// rewritten for instruction count and exhausted rows leaving the tile; 56 / 306
// ms with the round keys made in the step.
// Each history's arithmetic and random stream are those of a lane running it
// alone, and the tallies are integer sums: the result does not depend on
// the schedule.  The only waits between waves are for the wave that is
// replacing the current row, which does so without waiting on anyone.
template <bool X, int P, bool DENSE, bool LET>
// Physics mode: up to 1024 threads (16 waves at <= 128 VGPRs, one workgroup
// per CU with a ~120 KiB tile); double-float mode: up to 768 (12 waves; its 99 to
// 110 VGPRs would leave room for 16).
__global__ __launch_bounds__(X ? 768 : 1024) void queue_kernel(GeomDev g, QueueDev Q) {
    __shared__ __attribute__((aligned(16))) float hi[tab_hi_floats(3)], lo[X ? tab_lo_floats(3) : 4];
    __shared__ unsigned long long s_row;    // current row (high word; kRowNone while replaced)
    __shared__ unsigned long long s_tile;   // (row of the tile << 32) | users, kTileBusy while flushed
    extern __shared__ __attribute__((aligned(16))) uint32_t tile[];   // Q.tile_cap entries (twice with LET)
    stage_tables<X, 3>(hi, lo, Q.tables, DM_WATER);   // water, air, bone
    const Tabs T{hi, lo, -1, -1};
    for (int i = threadIdx.x; i < Q.tile_cap * (LET ? 2 : 1); i += blockDim.x) tile[i] = 0u;
    if (threadIdx.x == 0) {
        s_row = (unsigned long long)kRowNone << 32;
        s_tile = (unsigned long long)kRowNone << 32;
    }
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    RowCtl *const ctl = Q.ctl + Q.row_begin;
    const uint32_t draw_n = 64u * (uint32_t)min(Q.hist_per_lane, kStageHpl);   // (few enough for the 32-bit counters)
    unsigned long long iters = 0;   // in quarters
    for (;;) {
        // ---- bounded queue: a wavefront that has made iter_cap iterations
        // (draws, row picks, waits) leaves and reports it; it holds no row
        // pick and no tile here, so the other waves finish as before
        iters += 4;
        if (iters > Q.iter_cap) {
            if (lane == 0) atomicOr(Q.flags, kFlagAborted);
            break;
        }
        // ---- the workgroup's current row, and records of it
        const uint32_t cur = __builtin_amdgcn_readfirstlane((uint32_t)(rd_lds64(&s_row) >> 32));
        if (cur == kRowEnd) break;
        if (cur == kRowPick) {   // another wave is picking the next row (it waits on nobody)
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        uint32_t next = 0, end = 0, n_staged = 0;
        auto draw = [&]() {
            unsigned int at = 0;
            if (lane == 0) at = atomicAdd(&ctl[cur].next, draw_n);
            next = __builtin_amdgcn_readfirstlane(at);
            // a counter past its row's end means the row is exhausted
            end = next < n_staged ? min(n_staged, next + draw_n) : next;
        };
        if (cur != kRowNone) {
            n_staged = __builtin_amdgcn_readfirstlane(ctl[cur].staged);
            draw();
        }
        if (next >= end) {
            // no row yet, or this one is exhausted: the one wave that swaps
            // the row word from cur to kRowPick picks the next row
            bool mine = false;
            if (lane == 0) {
                unsigned long long w = (unsigned long long)cur << 32;
                mine = __hip_atomic_compare_exchange_strong(&s_row, &w, (unsigned long long)kRowPick << 32,
                                                            __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            if (__builtin_amdgcn_readfirstlane((uint32_t)mine) != 0u) {
                // a fresh row from the round's head, else the first row with
                // records left (64 rows per probe), else the end
                unsigned long long f = 0;
                if (lane == 0) f = atomicAdd(Q.head, 1ull);
                f = __builtin_amdgcn_readfirstlane((uint32_t)f);   // < 2^32 rows
                uint32_t nr = kRowEnd;
                if (f < (unsigned long long)Q.n_rows) {
                    nr = (uint32_t)f;
                } else {
                    // (rows are handed out in order: those with records left
                    // are among the last ones)
                    for (int r0 = max(0, Q.n_rows - kStealRows); r0 < Q.n_rows; r0 += 64) {
                        const int r = r0 + lane;
                        bool left = false;
                        if (r < Q.n_rows)
                            left = __hip_atomic_load(&ctl[r].next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                                   ctl[r].staged;
                        const unsigned long long m = __ballot(left);
                        if (m) {
                            nr = (uint32_t)(r0 + __ffsll((long long)m) - 1);
                            break;
                        }
                    }
                }
                if (lane == 0)
                    __hip_atomic_store(&s_row, (unsigned long long)nr << 32, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            continue;
        }
        iters -= 4u - Q.draw_cost;   // (not a pick or a wait)
        const uint32_t rl = cur;
        const RowDev row = Q.rows[Q.row_begin + rl];
        float scale = DENSE ? 0.0f : Q.spots[row.spot_global].scale;   // (dense rows: per lane)
        const ScenDev sc = Q.scen[row.scen];
        const StagedVP *const stg = reinterpret_cast<const StagedVP *>(Q.stage) + stage_base(Q, Q.row_begin + rl);
        const SparseSink gsink{Q.grid + (size_t)(DENSE ? row.dest : rl) * Q.gstride * (LET ? 2 : 1),
                               DENSE ? nullptr : Q.mark + (size_t)rl * Q.mstride};
        TileSink<!DENSE, LET> sink{nullptr, row.tlo[0], row.tlo[1], row.tlo[2],
                                   (uint32_t)row.tn[0], (uint32_t)row.tn[1], (uint32_t)row.tn[2], gsink,
                                   (uint32_t)Q.tile_cap, {}};
        // join the tile if it holds this row (or is free and clear)
        const uint32_t tn = (uint32_t)row.tn[0] * (uint32_t)row.tn[1] * (uint32_t)row.tn[2];
        const bool boxed = tn != 0u && tn <= (uint32_t)Q.tile_cap;
        auto join = [&]() {
            bool joined = false;
            if (lane == 0) {
                for (;;) {
                    unsigned long long t = rd_lds64(&s_tile);
                    const uint32_t tr = (uint32_t)(t >> 32), us = (uint32_t)t;
                    unsigned long long want;
                    if (us == kTileBusy) break;
                    if (tr == rl) want = t + 1ull;
                    else if (us == 0u) want = ((unsigned long long)rl << 32) | 1ull;
                    else break;
                    if (__hip_atomic_compare_exchange_strong(&s_tile, &t, want, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_WORKGROUP)) {
                        joined = true;
                        break;
                    }
                }
            }
            if (__builtin_amdgcn_readfirstlane((uint32_t)joined) != 0u) sink.tile = tile;
        };
        // leaves the tile; the last user adds it out and frees it
        auto leave = [&]() {
            sink.tile = nullptr;
            bool flusher = false;
            if (lane == 0) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                for (;;) {
                    unsigned long long t = rd_lds64(&s_tile);
                    const bool last = (uint32_t)t == 1u;
                    const unsigned long long want = last ? (((unsigned long long)rl << 32) | kTileBusy) : t - 1ull;
                    if (__hip_atomic_compare_exchange_strong(&s_tile, &t, want, __ATOMIC_ACQ_REL, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_WORKGROUP)) {
                        flusher = last;
                        break;
                    }
                }
            }
            flusher = __builtin_amdgcn_readfirstlane((uint32_t)flusher) != 0u;
            if (flusher) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                tile_flush(tile, sink, g, lane);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                if (lane == 0)
                    __hip_atomic_store(&s_tile, (unsigned long long)rl << 32, __ATOMIC_RELEASE,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        if (boxed) join();
        Acc acc;
#pragma unroll
        for (int k = 0; k < NLEDGER; ++k) acc.led[k] = 0;
        acc.steps = acc.hist = 0;
        Lane v;
        v.k0 = Q.key0;
        v.k1 = __builtin_amdgcn_readfirstlane(Q.seed_hi ^ row.field_id);
        v.spot = row.spot;
        v.physics = Q.physics;
        bool active = false;
        uint32_t since = 0;
        PState ps;
        for (;;) {
            const unsigned long long idle = __ballot(!active);
            const uint32_t nidle = (uint32_t)__popcll(idle);
            if (next >= end && end < n_staged && nidle >= (uint32_t)Q.refill_min) {
                if (iters >= Q.iter_cap) {   // no further draw: the lanes in flight finish, then the wave leaves
                    n_staged = end;
                } else {
                    draw();
                    if (next >= end) n_staged = end = next = 0;   // the row is exhausted
                    else iters += Q.draw_cost;
                }
            }
            // a wave that started beside the previous row's stragglers gets
            // the tile soon after they have left it
            if (boxed && sink.tile == nullptr && n_staged != 0u && (++since & 3u) == 0u) join();
            const bool refill = next < end && nidle >= min((uint32_t)Q.refill_min, end - next);
            if (!refill && nidle == 64u) break;
            // an exhausted row's last particles (those that miss the head cross
            // the whole grid in air, 2.5 times the mean steps) do not hold the
            // tile: the wave leaves it once kLeaveIdle lanes are idle
            if (n_staged == 0u && nidle >= kLeaveIdle && sink.tile != nullptr) leave();
            const uint32_t k = next + (uint32_t)__popcll(idle & below);
            if (refill && !active && k < end) {
                load_staged<DENSE, X>(stg + k, g, v, ps);
                if constexpr (DENSE) scale = Q.spots[v.spot].scale;
                active = true;
            }
            if (refill) next = min(end, next + nidle);
            // (opaque here: the round keys are made from these by scalar adds
            // in each step; hoisted out of the loop they overflow the scalar
            // registers and come back as 32 v_readlane a step)
            asm volatile("" : "+s"(v.k0), "+s"(v.k1));
            if constexpr (LET) sink.pend.dose = sink.pend.let = 0;
            if (active) {
                active = patient_step<TileSink<!DENSE, LET>, X, P>(v, acc, scale, T, g, sc.range_scale, sink, ps);
                if (!active) acc.steps += v.nsteps;
            }
            if constexpr (LET) sink.memory_adds(lane);
        }
        if (sink.tile != nullptr) leave();
        flush_ledger(acc, Q.ledger + (size_t)row.scen * NLEDGER, lane);
        flush_stats(acc, Q.stats, lane);
    }
}

// ---- compaction of an epoch's rows into CSR (three passes per epoch)
// A chunk is 256 touched-block bytes (8192 voxels) of one row, handled by
// one wave: lane l reads mark bytes 4l..4l+3 as one word (the mark stride is
// a multiple of 256, so the word stays inside the row's marks), the marked
// blocks are listed in ascending order in the wave's LDS, and then the two
// half-waves read two blocks' 32 slot values (coalesced 256 B each) at a
// time, kCsrUnroll such pairs in flight before any is used.  A wave visits
// kCsrGroup consecutive (row, chunk) pairs at once, their mark words loaded
// together; the waves of the launch stride over the epoch's groups,
// consecutive waves on consecutive groups.  A chunk without marks costs one
// load (in flight with its group's) and a ballot.
constexpr int kCsrGroup = 4, kCsrUnroll = 4;

// mark words of the pairs [g * kCsrGroup, ...) of an epoch (0 past the end)
__device__ __forceinline__ void group_marks(const QueueDev &Q, size_t gi, size_t npair, int lane,
                                            uint32_t (&w)[kCsrGroup]) {
#pragma unroll
    for (int j = 0; j < kCsrGroup; ++j) {
        const size_t pair = gi * kCsrGroup + j;
        w[j] = 0u;
        if (pair < npair) {
            const size_t row = pair / Q.nchunk, chunk = pair - row * Q.nchunk;
            w[j] = *reinterpret_cast<const uint32_t *>(Q.mark + row * Q.mstride + chunk * 256 + 4 * lane);
        }
    }
}

// lists the marked blocks of a chunk (offsets 0..255) in ascending order;
// returns their count
__device__ __forceinline__ int chunk_blocks(uint32_t wv, int lane, int *list) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) c += ((wv >> (8 * k)) & 0xFFu) != 0u;
    int pre = c;   // inclusive prefix over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(pre, o, 64);
        if (lane >= o) pre += y;
    }
    const int tot = __shfl(pre, 63, 64);
    int at = pre - c;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (((wv >> (8 * k)) & 0xFFu) != 0u) list[at++] = 4 * lane + k;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return tot;
}

// pass 1: non-zero count of every (row, chunk)
__global__ __launch_bounds__(256) void csr_count_kernel(QueueDev Q, unsigned int *cnt) {
    __shared__ int lists[4][256];
    const int lane = threadIdx.x & 63, wv_id = threadIdx.x >> 6;
    int *list = lists[wv_id];
    const size_t npair = (size_t)Q.n_rows * Q.nchunk;
    const size_t ngroup = (npair + kCsrGroup - 1) / kCsrGroup;
    const size_t nwave = (size_t)gridDim.x * 4;
    for (size_t gi = (size_t)blockIdx.x * 4 + wv_id; gi < ngroup; gi += nwave) {
        uint32_t w[kCsrGroup];
        group_marks(Q, gi, npair, lane, w);
#pragma unroll
        for (int j = 0; j < kCsrGroup; ++j) {
            const size_t pair = gi * kCsrGroup + j;
            if (pair >= npair) break;
            unsigned int c = 0;
            if (__ballot(w[j] != 0u) != 0ull) {
                const size_t row = pair / Q.nchunk, chunk = pair - row * Q.nchunk;
                const size_t b0 = chunk * 256;
                const unsigned long long *grid = Q.grid + row * Q.gstride;
                const int nm = chunk_blocks(w[j], lane, list);
                for (int p = 0; 2 * p < nm; p += kCsrUnroll) {
                    unsigned long long q[kCsrUnroll];
#pragma unroll
                    for (int u = 0; u < kCsrUnroll; ++u) {
                        const int idx = 2 * (p + u) + (lane >> 5);
                        q[u] = idx < nm ? grid[(b0 + list[idx]) * 32 + (lane & 31)] : 0ull;
                    }
#pragma unroll
                    for (int u = 0; u < kCsrUnroll; ++u) c += q[u] != 0ull;
                }
                for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
                __builtin_amdgcn_wave_barrier();   // list reused by the next chunk
            }
            if (lane == 0) cnt[pair] = c;
        }
    }
}

// pass 2: per row, exclusive prefix of its chunk counts and the row total
__global__ __launch_bounds__(1024) void csr_chunk_scan_kernel(const unsigned int *cnt, unsigned int *coff,
                                                              unsigned int *rowcnt, size_t nchunk) {
    __shared__ unsigned int part[1024];
    __shared__ unsigned int carry;
    const int row = blockIdx.x, t = threadIdx.x;
    const unsigned int *c = cnt + (size_t)row * nchunk;
    unsigned int *o = coff + (size_t)row * nchunk;
    if (t == 0) carry = 0u;
    __syncthreads();
    for (size_t s0 = 0; s0 < nchunk; s0 += 1024) {
        const unsigned int x = s0 + t < nchunk ? c[s0 + t] : 0u;
        part[t] = x;
        __syncthreads();
        for (int k = 1; k < 1024; k <<= 1) {
            const unsigned int y = t >= k ? part[t - k] : 0u;
            __syncthreads();
            part[t] += y;
            __syncthreads();
        }
        if (s0 + t < nchunk) o[s0 + t] = carry + part[t] - x;
        __syncthreads();
        if (t == 1023) carry += part[1023];
        __syncthreads();
    }
    if (t == 0) rowcnt[row] = carry;
}

// exclusive scan of this epoch's row counts into global CSR offsets (rows
// are stored in row order, so the offsets are the final row pointers)
__global__ __launch_bounds__(1024) void csr_offsets_kernel(const unsigned int *nnz, int n_rows, int row_begin,
                                                           unsigned long long *row_off,
                                                           unsigned long long *row_nnz,
                                                           unsigned long long *used,
                                                           unsigned long long capacity, unsigned int *flags) {
    __shared__ unsigned long long part[1024];
    const int t = threadIdx.x;
    const unsigned long long x = t < n_rows ? nnz[t] : 0ull;
    part[t] = x;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const unsigned long long y = t >= o ? part[t - o] : 0ull;
        __syncthreads();
        part[t] += y;
        __syncthreads();
    }
    const unsigned long long base = *used;
    if (t < n_rows) {
        row_off[row_begin + t] = base + part[t] - x;
        row_nnz[row_begin + t] = x;
    }
    __syncthreads();
    if (t == 1023) {
        *used = base + part[1023];
        if (base + part[1023] > capacity) atomicOr(flags, 1u);
    }
}

// pass 3: emit (voxel, q) of every chunk at its place in ascending voxel
// order and clear exactly the touched blocks and their marks
__global__ __launch_bounds__(256) void csr_emit_kernel(QueueDev Q, const unsigned int *cnt, const unsigned int *coff,
                                                       const unsigned long long *row_off,
                                                       const unsigned long long *row_nnz, int32_t *col,
                                                       long long *qv, unsigned long long capacity,
                                                       unsigned int *flags) {
    __shared__ int lists[4][256];
    const int lane = threadIdx.x & 63, wv_id = threadIdx.x >> 6;
    int *list = lists[wv_id];
    const size_t npair = (size_t)Q.n_rows * Q.nchunk;
    const size_t ngroup = (npair + kCsrGroup - 1) / kCsrGroup;
    const size_t nwave = (size_t)gridDim.x * 4;
    for (size_t gi = (size_t)blockIdx.x * 4 + wv_id; gi < ngroup; gi += nwave) {
        uint32_t w[kCsrGroup];
        group_marks(Q, gi, npair, lane, w);
#pragma unroll
        for (int j = 0; j < kCsrGroup; ++j) {
            const size_t pair = gi * kCsrGroup + j;
            if (pair >= npair) break;
            if (__ballot(w[j] != 0u) == 0ull) continue;
            const size_t row = pair / Q.nchunk, chunk = pair - row * Q.nchunk;
            const size_t b0 = chunk * 256;
            uint8_t *mark = Q.mark + row * Q.mstride;
            unsigned long long *grid = Q.grid + row * Q.gstride;
            const int nm = chunk_blocks(w[j], lane, list);
            const unsigned long long rb = row_off[Q.row_begin + row];
            const bool write = rb + row_nnz[Q.row_begin + row] <= capacity;
            const unsigned long long p0 = rb + coff[pair];
            unsigned long long pos = p0;
            for (int p = 0; 2 * p < nm; p += kCsrUnroll) {
                unsigned long long q[kCsrUnroll];
                size_t v[kCsrUnroll];
#pragma unroll
                for (int u = 0; u < kCsrUnroll; ++u) {
                    const int idx = 2 * (p + u) + (lane >> 5);
                    v[u] = idx < nm ? (b0 + list[idx]) * 32 + (lane & 31) : 0;
                    q[u] = idx < nm ? grid[v[u]] : 0ull;
                }
#pragma unroll
                for (int u = 0; u < kCsrUnroll; ++u) {
                    const int idx = 2 * (p + u) + (lane >> 5);
                    const unsigned long long bal = __ballot(q[u] != 0ull);
                    if (q[u] != 0ull && write) {
                        const unsigned long long at = pos + __popcll(bal & ((1ull << lane) - 1ull));
                        col[at] = (int32_t)v[u];
                        qv[at] = (long long)q[u];
                    }
                    if (idx < nm) grid[v[u]] = 0ull;
                    pos += __popcll(bal);
                }
            }
            if (w[j] != 0u) *reinterpret_cast<uint32_t *>(mark + b0 + 4 * lane) = 0u;
            if (lane == 0 && pos - p0 != cnt[pair]) atomicOr(flags, 2u);
            __builtin_amdgcn_wave_barrier();   // list reused by the next chunk
        }
    }
}

// Rate of non-returning int64 atomic adds to device memory with the address
// pattern of the transport's deposits: each lane walks a track of `len`
// consecutive voxels along x (the beam axis of a lateral field) from a
// random depth, at a lateral (y, z) offset drawn around one of 64 spot axes
// with a Gaussian of sigma voxels (sum of 4 uniforms), so that hot spots
// form where tracks overlap.  Work: n_tracks x len atomics.
__global__ __launch_bounds__(256) void atomic_rate_kernel(unsigned long long *grid, int nx, int ny, int nz,
                                                          unsigned long long n_tracks, int len, float sigma,
                                                          uint32_t seed) {
    for (unsigned long long t = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; t < n_tracks;
         t += (unsigned long long)gridDim.x * blockDim.x) {
        uint32_t x = (uint32_t)t * 0x9E3779B9u ^ seed;
        auto next = [&]() {   // xorshift32
            x ^= x << 13; x ^= x >> 17; x ^= x << 5;
            return x;
        };
        next(); next();
        const uint32_t spot = (uint32_t)(t >> 12) & 63u;   // neighbouring tracks share a spot
        const float cy = 0.25f * ny + 0.5f * ny * (float)((spot * 2654435761u) >> 16 & 0xFFFFu) / 65536.0f;
        const float cz = 0.25f * nz + 0.5f * nz * (float)((spot * 2246822519u) >> 16 & 0xFFFFu) / 65536.0f;
        float gy = 0.0f, gz = 0.0f;
        for (int k = 0; k < 4; ++k) {
            gy += (float)(next() >> 8) * 0x1p-24f;
            gz += (float)(next() >> 8) * 0x1p-24f;
        }
        // sum of 4 U(0,1): mean 2, variance 1/3
        const int y = min(max((int)(cy + (gy - 2.0f) * 1.7320508f * sigma), 0), ny - 1);
        const int z = min(max((int)(cz + (gz - 2.0f) * 1.7320508f * 0.5f * sigma), 0), nz - 1);
        const int x0 = (int)(next() % (uint32_t)max(nx - len, 1));
        unsigned long long *row = grid + (size_t)nx * ((size_t)y + (size_t)ny * (size_t)z);
        for (int i = 0; i < len && x0 + i < nx; ++i) atomicAdd(row + x0 + i, 1ull);
    }
}

__global__ void fill_u64_kernel(unsigned long long *p, size_t n, unsigned long long v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void csr_scatter_kernel(const int32_t *col, const long long *qv, unsigned long long begin,
                                   unsigned long long end, unsigned long long *dense) {
    for (unsigned long long i = begin + (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < end;
         i += (unsigned long long)gridDim.x * blockDim.x)
        atomicAdd(dense + col[i], (unsigned long long)qv[i]);
}

// Rows handed out: any of columns, values (Gy per unit weight) and energies in
// one pass, four entries a thread (the library's arrays are 256-byte aligned;
// VEC: so are the outputs to 16 bytes, else they are stored one by one).
// HBM-bound: 12 bytes an entry read, up to 16 written.  As a copy per array and a
// value pass of one entry a thread, columns and values of 1.03e9 entries took
// 15.8 ms (the copies at 1 TB/s); in this pass 6.8.
template <bool VEC>
__global__ __launch_bounds__(256) void csr_export_kernel(const int32_t *col, const long long *qv, size_t n, GeomDev g,
                                                         double mev_scale, int32_t *ocol, float *val, long long *oq) {
    const float vol_kg = g.sp[0] * g.sp[1] * g.sp[2] * 1e-6f, ms = (float)mev_scale;
    for (size_t i = 4 * (blockIdx.x * (size_t)blockDim.x + threadIdx.x); i < n; i += 4 * (size_t)gridDim.x * blockDim.x) {
        int c[4];
        long long q[4];
        float v[4];
        const int m = (int)min((size_t)4, n - i);
        if (m == 4) {
            const int4 c4 = *reinterpret_cast<const int4 *>(col + i);
            const longlong2 q0 = reinterpret_cast<const longlong2 *>(qv + i)[0], q1 = reinterpret_cast<const longlong2 *>(qv + i)[1];
            c[0] = c4.x; c[1] = c4.y; c[2] = c4.z; c[3] = c4.w;
            q[0] = q0.x; q[1] = q0.y; q[2] = q1.x; q[3] = q1.y;
        } else {
            for (int j = 0; j < 4; ++j) {
                c[j] = col[i + (j < m ? j : 0)];
                q[j] = qv[i + (j < m ? j : 0)];
            }
        }
        if (val) {
            int hu[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) hu[j] = g.kind == 1 ? (int)g.hu[c[j]] : 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float rho = 1.0f;
                int mat;
                if (g.kind == 1) hu_material(hu[j], mat, rho);
                v[j] = (float)q[j] * (ms / (rho * vol_kg));
            }
        }
        if (VEC && m == 4) {
            if (ocol) *reinterpret_cast<int4 *>(ocol + i) = make_int4(c[0], c[1], c[2], c[3]);
            if (val) *reinterpret_cast<float4 *>(val + i) = make_float4(v[0], v[1], v[2], v[3]);
            if (oq) {
                reinterpret_cast<longlong2 *>(oq + i)[0] = make_longlong2(q[0], q[1]);
                reinterpret_cast<longlong2 *>(oq + i)[1] = make_longlong2(q[2], q[3]);
            }
        } else {
            for (int j = 0; j < m; ++j) {
                if (ocol) ocol[i + j] = c[j];
                if (val) val[i + j] = v[j];
                if (oq) oq[i + j] = q[j];
            }
        }
    }
}

// ------------------------------------------------------------ dynamic voxel spacing
// Influence-matrix rows merged into cells (the planning system's coarser
// voxels for organs at risk, Methods C): a cell is a run of consecutive
// voxels given by a non-decreasing voxel -> cell map, cstart[c] its first
// voxel.  Cell mass (kg) = the sum of its voxels' masses, in voxel order.
//
// The map's check and the cells' first voxels in one pass over it.  st[1],
// st[2]: its first and last cell; st[3] (preset to ~0): the first voxel at
// which it does not grow by 0 or 1.  cstart is whole only if the check passes.
__global__ __launch_bounds__(256) void cell_map_kernel(const int32_t *cmap, int nvox, int n_cells, int32_t *cstart,
                                                       unsigned *st) {
    unsigned bad = ~0u;
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < (size_t)nvox; v += (size_t)gridDim.x * blockDim.x) {
        const int c = cmap[v];
        if (v == 0) {
            st[1] = (unsigned)c;
            cstart[0] = 0;
            cstart[n_cells] = nvox;
        } else {
            const long long d = (long long)c - cmap[v - 1];
            if (d != 0 && d != 1) bad = min(bad, (unsigned)v);
            if (d == 1 && c >= 0 && c < n_cells) cstart[c] = (int32_t)v;
        }
        if (v + 1 == (size_t)nvox) st[2] = (unsigned)c;
    }
    if (bad != ~0u) atomicMin(st + 3, bad);
}

__global__ void cell_mass_kernel(GeomDev g, const int32_t *cstart, int n_cells, double *mass) {
    const double vol_kg = (double)g.sp[0] * (double)g.sp[1] * (double)g.sp[2] * 1e-6;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n_cells; c += gridDim.x * blockDim.x) {
        double m = 0.0;
        for (int v = cstart[c]; v < cstart[c + 1]; ++v) {
            float rho = 1.0f;
            int mm;
            if (g.kind == 1) hu_material(g.hu[v], mm, rho);
            m += (double)rho;
        }
        mass[c] = m * vol_kg;
    }
}

// (89 M entries on a 10.5 M voxel grid: 226 us with one window's loads at a time,
// 112 with four; the emit pass below 731 us without loads ahead and with all six
// scan steps, 532 so.)
// cells per piece (a wavefront per piece of at most kCellPiece entries of one
// row): runs of one cell that start inside the piece; flags columns outside
// the grid (bit 1) and columns not ascending within a row (bit 2)
__global__ __launch_bounds__(256) void cell_count_kernel(const long long *rp, const CellPiece *pcs,
                                                         long long n_pieces, const int32_t *col,
                                                         const int32_t *cmap, int nvox, unsigned long long *cnt,
                                                         unsigned *err) {
    const long long p = (long long)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6);
    if (p >= n_pieces) return;
    const int lane = (int)(threadIdx.x & 63);
    const CellPiece pc = pcs[p];
    const long long b = pc.begin, e = pc.begin + pc.len;
    int carry = -1, carry_col = -1;
    if (b > rp[pc.row]) {
        // the entry before the piece (checked by the piece that owns it)
        carry_col = col[b - 1];
        carry = (unsigned)carry_col < (unsigned)nvox ? cmap[carry_col] : -1;
    }
    unsigned long long n = 0;
    for (long long i0 = b; i0 < e; i0 += 256) {   // four windows' loads in flight
        int c[4], v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long i = i0 + 64 * u + lane;
            v[u] = i < e ? col[i] : -1;
        }
        unsigned bad = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = -1;
            if ((unsigned)v[u] < (unsigned)nvox) c[u] = cmap[v[u]];
            else if (i0 + 64 * u + lane < e) bad |= 1u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long i = i0 + 64 * u + lane;
            const bool valid = i < e;
            int pv = __shfl_up(v[u], 1);
            int pc_ = __shfl_up(c[u], 1);
            if (lane == 0) {
                pv = carry_col;
                pc_ = carry;
            }
            if (valid && (i > b || carry_col >= 0) && v[u] <= pv) bad |= 2u;
            n += (unsigned long long)__popcll(__ballot(valid && c[u] >= 0 && c[u] != pc_));
            carry = __shfl(c[u], 63);
            carry_col = __shfl(v[u], 63);
        }
        if (bad) atomicOr(err, bad);
    }
    if (lane == 0) cnt[p] = n;
}

// row r of the output starts where its first piece does
__global__ __launch_bounds__(256) void cell_rows_kernel(const long long *first_piece, const long long *pout,
                                                        size_t n, long long *rp_out) {
    const size_t r = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (r < n) rp_out[r] = pout[first_piece[r]];
}

// merged rows, a wavefront per piece: the runs that start inside the piece
// belong to it; segmented sums of their int64 energies (exact) over 64-entry
// windows, carried across windows; the piece's last run is followed past the
// piece's end up to the next start or the row's end.  The value is the
// cell's energy over its mass.
__global__ __launch_bounds__(256) void cell_emit_kernel(const long long *rp, const CellPiece *pcs, long long n_pieces,
                                                        const int32_t *col, const long long *q, const int32_t *cmap,
                                                        const long long *pout, const double *mass, double mev_scale,
                                                        int32_t *ocell, long long *oq, float *oval) {
    const long long p = (long long)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6);
    if (p >= n_pieces) return;
    const int lane = (int)(threadIdx.x & 63);
    const CellPiece pc = pcs[p];
    const long long re = rp[pc.row + 1];
    const long long b = pc.begin, e = pc.begin + pc.len;
    const long long o0 = pout[p], o1 = pout[p + 1];
    if (o0 == o1) return;   // no run starts in this piece
    int carry_cell = b > rp[pc.row] ? cmap[col[b - 1]] : -1;
    long long carry_sum = 0, starts_before = 0, e_eff = re;
    auto put = [&](long long k, int c, long long sum) {
        const long long pos = o0 + k;
        if (k >= 0 && pos < o1) {
            if (ocell) ocell[pos] = c;
            if (oq) oq[pos] = sum;
            if (oval) oval[pos] = (float)((double)sum * mev_scale / mass[c]);
        }
    };
    // a window's columns are loaded two windows ahead, its cells and energies one
    auto load_col = [&](long long i) { return i < re ? col[i] : -1; };
    auto load_cell = [&](int v) { return v >= 0 ? cmap[v] : -1; };
    auto load_q = [&](long long i) { return i < re ? q[i] : 0ll; };
    int v1 = load_col(b + lane), c1 = load_cell(v1);
    long long q1 = load_q(b + lane);
    v1 = load_col(b + 64 + lane);
    for (long long i0 = b;; i0 += 64) {
        const long long i = i0 + lane;
        const bool valid0 = i < re;
        const int c = c1;
        const long long qi = q1;
        c1 = load_cell(v1);
        q1 = load_q(i + 64);
        v1 = load_col(i + 128);
        int pcl = __shfl_up(c, 1);
        if (lane == 0) pcl = carry_cell;
        const bool start0 = valid0 && c != pcl;
        if (i0 + 64 > e) {
            // the first start at or after the piece's end closes its last run
            const unsigned long long m0 = __ballot(start0 && i >= e);
            if (m0) {
                const long long first = i0 + (long long)(__ffsll((long long)m0) - 1);
                e_eff = first < e_eff ? first : e_eff;
            }
        }
        const bool valid = valid0 && i < e_eff;
        const bool start = start0 && valid;
        const bool v0 = __shfl(valid ? 1 : 0, 0) != 0, s0 = __shfl(start ? 1 : 0, 0) != 0;
        // the run left open by the last window ends here
        if (lane == 0 && carry_cell >= 0 && (s0 || !v0)) put(starts_before - 1, carry_cell, carry_sum);
        if (!v0) break;
        long long x = valid ? qi : 0;
        if (lane == 0 && !start) x += carry_sum;
        long long sum = x;
        int f = start ? 1 : 0;
        for (int d = 1; d < 64; d <<= 1) {
            if (!__ballot(valid && lane >= d && !f)) break;   // (runs of few entries: two steps)
            const long long so = __shfl_up(sum, d);
            const int fo = __shfl_up(f, d);
            if (lane >= d && !f) sum += so;
            if (lane >= d) f |= fo;
        }
        const unsigned long long m = __ballot(start);
        const int last = (int)((e_eff - i0 < 64 ? e_eff - i0 : 64) - 1);
        const bool next_start = __shfl_down(start ? 1 : 0, 1) != 0;
        if (valid && lane < last && next_start)
            put(starts_before + (long long)__popcll(m & ((2ull << lane) - 1ull)) - 1, c, sum);
        carry_cell = __shfl(c, last);
        carry_sum = __shfl(sum, last);
        starts_before += (long long)__popcll(m);
    }
}

// ------------------------------------------------------------ surrogate data
// Plain brass traversals for the surrogate's training data: each entry state
// (x, y on the block's upstream face, direction cosines u, v, energy) crosses
// the field's block with the plain transport (crossing number at every step).
// Per VP: the 8 network inputs, the 3 normalised targets and the outcome
// (1 transmitted, 0 stopped or lost, -1 entered through the opening).
__global__ __launch_bounds__(256) void surrogate_sample_kernel(FieldDev f, const float *entries, int n,
                                                               uint32_t key0, uint32_t key1, unsigned physics,
                                                               const float *tables, float *xo, float *yo,
                                                               float *to) {
    __shared__ __attribute__((aligned(16))) float hi[TAB_HI_FLOATS];
    __shared__ float2 poly[POLY_LDS];
    stage_tables<false, NMAT>(hi, nullptr, tables, 0);
    const Tabs T{hi, nullptr, DM_PMMA, DM_BRASS};
    for (int i = threadIdx.x; i < f.nv; i += blockDim.x) poly[i] = f.poly[i];
    __syncthreads();
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float *e = entries + (size_t)i * 5;
        Lane v;
        v.k0 = key0;
        v.k1 = key1;
        v.spot = 0;
        v.hist = (uint32_t)i;
        v.nblk = 0;
        v.nsteps = 0;
        v.physics = physics;
        v.px = e[0];
        v.py = e[1];
        v.pz = f.blk_zu;
        v.pzlo = 0.0f;
        v.pxlo = v.pylo = 0.0f;
        v.dx = e[2];
        v.dy = e[3];
        v.dz = sqrtf(fmaxf(1.0f - e[2] * e[2] - e[3] * e[3], 0.0f));
        v.E = e[4];
        v.Elo = 0.0f;
        const float x0 = v.px, y0 = v.py, u0 = v.dx, w0 = v.dy, z0 = v.dz, E0 = v.E;
        const int nv = f.nv;
        const bool open = nv >= 3 && in_polygon(poly, nv, x0, y0);
        const float de = nv >= 3 ? dist_to_polygon(poly, nv, x0, y0) : 1000.0f;
        float *xr = xo + (size_t)i * 8;
        xr[0] = x0 / 20.0f;
        xr[1] = y0 / 20.0f;
        xr[2] = u0 / 0.05f;
        xr[3] = w0 / 0.05f;
        xr[4] = (E0 - 150.0f) / 50.0f;
        xr[5] = fminf(de, 100.0f) / 10.0f;
        xr[6] = f.blk_t / 30.0f;
        xr[7] = 0.0f;   // brass
        float *yr = yo + (size_t)i * 3;
        yr[0] = yr[1] = yr[2] = 0.0f;
        if (open) {
            to[i] = -1.0f;
            continue;
        }
        Acc acc;
#pragma unroll
        for (int k = 0; k < NLEDGER; ++k) acc.led[k] = 0;
        v.pz = 0.0f;   // depth local to the block
        if (!block_transport<false, true>(v, true, acc, 1.0f, T, poly, f)) {
            to[i] = 0.0f;
            continue;
        }
        to[i] = 1.0f;
        const float Eo = v.E + v.Elo;
        const float c = fminf(fmaxf(u0 * v.dx + w0 * v.dy + z0 * v.dz, -1.0f), 1.0f);
        const float tx = f.blk_t / z0;
        const float xs = fmaf(tx, u0, x0), ys = fmaf(tx, w0, y0);
        yr[0] = ((E0 - Eo) / E0 - 0.5f) / 0.25f;
        yr[1] = acosf(c) / 0.05f;
        yr[2] = sqrtf((v.px - xs) * (v.px - xs) + (v.py - ys) * (v.py - ys)) / 2.0f;
    }
}


// Resume one deferred VP: where the network is confident the traversal is
// sampled from it (transmission, then one mixture component and its
// outgoing energy loss, angle and offset; azimuth uniform, shared by angle
// and offset); otherwise the plain brass transport runs from the recorded
// state.  Then the patient.
template <class Sink, bool X>
__device__ void resume_deferred(Lane &v, Acc &acc, float scale, const Tabs &T, const float2 *poly,
                                const FieldDev &f, const float *o, float p_lo, float p_hi, const GeomDev &g,
                                const float *shift, float range_scale, const Sink &sink) {
    const float ptrans = 1.0f / (1.0f + __expf(-o[0]));
    bool go = true;
    if (!(ptrans < p_lo || ptrans > p_hi)) {
        v.pz = 0.0f;   // depth local to the block
        v.pzlo = 0.0f;
        go = block_transport<X, true>(v, true, acc, scale, T, poly, f);
    } else {
        v.E += v.Elo;
        v.Elo = 0.0f;
        const uint4 w = draw(v);
        if (!(unit_open(w.x) < ptrans)) {
            ledger_add(acc, L_BLOCK, v.E, scale);   // stopped in brass
            go = false;
        } else {
            // mixture component from the softmax of the weight logits
            float mw = o[1];
            for (int c = 1; c < 4; ++c) mw = fmaxf(mw, o[1 + c]);
            float pc[4], tot = 0.0f;
            for (int c = 0; c < 4; ++c) { pc[c] = __expf(o[1 + c] - mw); tot += pc[c]; }
            const float uc = unit_open(w.y) * tot;
            int c = 0;
            float acc_p = pc[0];
            while (c < 3 && uc > acc_p) { ++c; acc_p += pc[c]; }
            const uint4 w2 = draw(v);
            float z0, z1, z2, z3;
            box_muller_fast(w2.x, w2.y, z0, z1);
            box_muller_fast(w2.z, w2.w, z2, z3);
            const float y0 = o[5 + 3 * c + 0] + __expf(o[17 + 3 * c + 0]) * z0;
            const float y1 = o[5 + 3 * c + 1] + __expf(o[17 + 3 * c + 1]) * z1;
            const float y2 = o[5 + 3 * c + 2] + __expf(o[17 + 3 * c + 2]) * z2;
            const float frac = fminf(fmaxf(0.5f + 0.25f * y0, 0.0f), 1.0f);
            const float theta = fmaxf(y1, 0.0f) * 0.05f;
            const float off = fmaxf(y2, 0.0f) * 2.0f;
            const float phi = unit_open(w.z);   // turns
            const float cph = __builtin_amdgcn_cosf(phi), sph = __builtin_amdgcn_sinf(phi);
            const float Eout = v.E * (1.0f - frac);
            ledger_add(acc, L_BLOCK, v.E - Eout, scale);
            const float tx = f.blk_t / v.dz;
            v.px = fmaf(tx, v.dx, v.px) + off * cph;
            v.py = fmaf(tx, v.dy, v.py) + off * sph;
            rotate_dir(v, theta * cph, theta * sph);
            v.pz = f.blk_zd;
            v.E = Eout;
            if (!(v.dz > 0.0f) || Eout <= kELo) {
                ledger_add(acc, (v.dz > 0.0f) ? L_BLOCK : L_ESCAPED, Eout, scale);
                go = false;
            }
        }
    }
    if (go) patient<Sink, X>(v, acc, scale, T, g, f, shift, range_scale, sink, 0.0f);
}

__device__ __forceinline__ void lane_from_record(Lane &v, const DeferRec &r, uint32_t k0, uint32_t k1,
                                                 unsigned physics, float zu) {
    v.k0 = k0;
    v.k1 = k1;
    v.spot = r.spot;
    v.hist = r.hist;
    v.nblk = r.nblk;
    v.nsteps = 0;
    v.physics = physics;
    v.px = r.x;
    v.py = r.y;
    v.pz = zu;
    v.pzlo = r.pzlo;
    v.pxlo = v.pylo = 0.0f;
    v.dx = r.u;
    v.dy = r.v;
    v.dz = r.w;
    v.E = r.E;
    v.Elo = r.Elo;
}

__device__ __forceinline__ void flush_ledger_steps(Acc &acc, unsigned long long *ledger, unsigned long long *stats) {
#pragma unroll
    for (int j = 0; j < NLEDGER; ++j) {
        long long x = acc.led[j];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if ((threadIdx.x & 63) == 0 && x != 0) atomicAdd(ledger + j, (unsigned long long)x);
        acc.led[j] = 0;
    }
    unsigned long long st = acc.steps;
    for (int o = 32; o > 0; o >>= 1) st += __shfl_xor(st, o, 64);
    if ((threadIdx.x & 63) == 0 && st != 0) atomicAdd(stats + 0, st);
    acc.steps = 0;
}

// dense runs: one field, one scenario per launch
template <bool X>
__global__ __launch_bounds__(256) void sur_resume_kernel(GeomDev g, FieldDev f, LaunchDev L, const DeferRec *rec,
                                                         const float *out, unsigned long long n, float p_lo,
                                                         float p_hi) {
    __shared__ __attribute__((aligned(16))) float hi[TAB_HI_FLOATS], lo[X ? tab_lo_floats(NMAT) : 1];
    extern __shared__ __attribute__((aligned(16))) float2 poly[];
    stage_tables<X, NMAT>(hi, lo, L.tables, 0);
    const Tabs T{hi, lo, DM_PMMA, DM_BRASS};
    for (int i = threadIdx.x; i < f.nv; i += blockDim.x) poly[i] = f.poly[i];
    __syncthreads();
    Acc acc;
#pragma unroll
    for (int j = 0; j < NLEDGER; ++j) acc.led[j] = 0;
    acc.steps = acc.hist = 0;
    const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const DeferRec r = rec[i];
        Lane v;
        lane_from_record(v, r, L.key0, L.key1, L.physics, f.blk_zu);
        resume_deferred<DenseSink, X>(v, acc, L.spots[r.spot].scale, T, poly, f, out + i * MLP_OUT, p_lo, p_hi, g, L.shift,
                        L.range_scale, DenseSink{L.tally, L.let_tally});
        acc.steps += v.nsteps;
    }
    flush_ledger_steps(acc, L.ledger, L.stats);
}

// influence-matrix runs: the record's tag is its row within the epoch, which
// selects the field, spot, scenario and the row's sparse slot
template <bool X>
__global__ __launch_bounds__(256) void sur_resume_csr_kernel(GeomDev g, QueueDev Q, const DeferRec *rec,
                                                             const float *out, unsigned long long n, float p_lo,
                                                             float p_hi) {
    __shared__ __attribute__((aligned(16))) float hi[TAB_HI_FLOATS], lo[X ? tab_lo_floats(NMAT) : 1];
    extern __shared__ __attribute__((aligned(16))) float2 poly[];
    stage_tables<X, NMAT>(hi, lo, Q.tables, 0);
    const Tabs T{hi, lo, DM_PMMA, DM_BRASS};
    for (int i = threadIdx.x; i < Q.n_poly_total; i += blockDim.x) poly[i] = Q.polys[i];
    __syncthreads();
    Acc acc;
#pragma unroll
    for (int j = 0; j < NLEDGER; ++j) acc.led[j] = 0;
    acc.steps = acc.hist = 0;
    int cur_scen = -1;   // scenario whose ledger this lane is accumulating
    const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const DeferRec r = rec[i];
        const int rl = (int)r.tag;
        const RowDev row = Q.rows[Q.row_begin + rl];
        const FieldDev f = Q.fields[row.field];
        const ScenDev sc = Q.scen[row.scen];
        const SparseSink sink{Q.grid + (size_t)rl * Q.gstride, Q.mark + (size_t)rl * Q.mstride};
        if (row.scen != cur_scen) {
            // ledgers are per scenario: this lane's sums so far go out with
            // plain per-lane atomics (lanes of a wave may differ in scenario)
            if (cur_scen >= 0)
                for (int j = 0; j < NLEDGER; ++j)
                    if (acc.led[j] != 0) {
                        atomicAdd(Q.ledger + (size_t)cur_scen * NLEDGER + j, (unsigned long long)acc.led[j]);
                        acc.led[j] = 0;
                    }
            cur_scen = row.scen;
        }
        Lane v;
        lane_from_record(v, r, Q.key0, Q.seed_hi ^ row.field_id, Q.physics, f.blk_zu);
        resume_deferred<SparseSink, X>(v, acc, Q.spots[row.spot_global].scale, T, poly + Q.poly_off[row.field], f,
                        out + i * MLP_OUT, p_lo, p_hi, g, sc.shift, sc.range_scale, sink);
        acc.steps += v.nsteps;
    }
    // every lane of the wave is back here: the ledgers reduce per wave and
    // scenario (an epoch's records span one or two scenarios), one atomic per
    // group instead of one per lane
    bool pending = cur_scen >= 0;
    for (;;) {
        const unsigned long long m = __ballot(pending);
        if (!m) break;
        const int leader = __ffsll((long long)m) - 1;
        const int sc = __shfl(cur_scen, leader, 64);
        const bool mine = pending && cur_scen == sc;
#pragma unroll
        for (int j = 0; j < NLEDGER; ++j) {
            long long x = mine ? acc.led[j] : 0ll;
            for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
            if ((int)(threadIdx.x & 63) == leader && x != 0)
                atomicAdd(Q.ledger + (size_t)sc * NLEDGER + j, (unsigned long long)x);
        }
        if (mine) pending = false;
    }
    unsigned long long st = acc.steps;
    for (int o = 32; o > 0; o >>= 1) st += __shfl_xor(st, o, 64);
    if ((threadIdx.x & 63) == 0 && st != 0) atomicAdd(Q.stats + 0, st);
}

// Reciprocal tables of a blob: segment widths (hardware estimate) and slopes
// (estimate and one Newton step), as the steps used to compute them; the last
// entries stay (sentinels).
__global__ void derive_tables_kernel(float *blob) {
    const int i = threadIdx.x;
    if (i >= NE - 1) return;
    if (blockIdx.x == 0) blob[TAB_RDW + i] = __builtin_amdgcn_rcpf(blob[TAB_DWH + i]);
    float *tm = blob + TAB_SHARED + blockIdx.x * TAB_PER_MAT;
    tm[T_RS * NE + i] = rcp_nr(tm[T_SH * NE + i]);
}

// densities of n voxels between two margins of zeros
__global__ void density_kernel(const int16_t *hu, float *rho, size_t margin, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n + 2 * margin; i += (size_t)gridDim.x * blockDim.x) {
        int m;
        rho[i] = i - margin < n ? hu_density<false>((int)hu[i - margin], m).h : 0.0f;
    }
}

// ------------------------------------------------------------ aperture raster
// One wave per raster cell, its lanes over the polygon's edges (FP64).
// Pass 1: signed distance (+ inside, by the kernels' half-open crossing-number
// rule) from the cell centre to the boundary; for a cell within radius + h of
// it a reference point (FP32, the cell centre moved by at most 0.01 mm off any
// edge closer than 1e-4 mm) with its side, and the number of edges within
// `radius` of it.  A point p of the cell is on the reference point's side unless
// listed edges cross the segment from it to p, and a ray from p meets no
// unlisted edge within radius - |p - ref|, so the kernels test a handful of
// edges instead of every edge there.  Cells farther from the boundary get no
// reference point (the distance bound decides them).  Pass 2: the lists, edges
// in ascending order, each cell's wherever the counter put it.  On the host
// these took 50 ms for a 128-gon of 35 mm (61 ms with its checks) and as much
// for every call that sets a field again; 41 000 cells are 0.1 ms here.
struct EdgeScan {
    double best;   // smallest squared distance
    bool in;
};

__device__ __forceinline__ double edge_dist2(const float2 a, const float2 b, double x, double y) {
    const double ex = (double)b.x - a.x, ey = (double)b.y - a.y, l2 = ex * ex + ey * ey;
    double t = l2 > 0.0 ? ((x - a.x) * ex + (y - a.y) * ey) / l2 : 0.0;
    t = fmin(fmax(t, 0.0), 1.0);
    const double dx = x - a.x - t * ex, dy = y - a.y - t * ey;
    return dx * dx + dy * dy;
}

__device__ EdgeScan scan_edges(const Raster &r, double x, double y, int lane) {
    double best = 1e300;
    unsigned long long flips = 0;
    for (int k0 = 0; k0 < r.nv; k0 += 64) {
        const int k = k0 + lane;
        bool flip = false;
        if (k < r.nv) {
            const float2 b = r.poly[k], a = r.poly[k ? k - 1 : r.nv - 1];
            if (((double)a.y > y) != ((double)b.y > y)) {
                const double xc = a.x + (y - a.y) * ((double)b.x - a.x) / ((double)b.y - a.y);
                flip = x < xc;
            }
            best = fmin(best, edge_dist2(a, b, x, y));
        }
        flips += __popcll(__ballot(flip));
    }
    for (int o = 32; o > 0; o >>= 1) best = fmin(best, __shfl_xor(best, o, 64));
    return {best, (flips & 1ull) != 0};
}

__global__ __launch_bounds__(256) void raster_kernel(Raster r) {
    const int lane = threadIdx.x & 63;
    const int c = (int)(blockIdx.x * (blockDim.x >> 6)) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c >= r.nx * r.ny) return;
    const int j = c / r.nx, i = c - j * r.nx;
    const double x = r.x0 + (i + 0.5) * r.h, y = r.y0 + (j + 0.5) * r.h;
    const EdgeScan s = scan_edges(r, x, y, lane);
    const float d = (float)(s.in ? sqrt(s.best) : -sqrt(s.best));
    uint2 cell = make_uint2(0u, 0u);
    float2 q = make_float2(0.0f, 0.0f);
    if (fabs((double)d) <= r.radius + r.h) {
        q = make_float2((float)x, (float)y);
        EdgeScan e{0.0, false};
        for (int tries = 0; tries < 8; ++tries) {
            e = scan_edges(r, q.x, q.y, lane);
            if (sqrt(e.best) > 1e-4) break;
            q = make_float2(q.x + 0.0013f, q.y + 0.0009f);
        }
        e = scan_edges(r, q.x, q.y, lane);
        unsigned n = 0;
        for (int k0 = 0; k0 < r.nv; k0 += 64) {
            const int k = k0 + lane;
            n += (unsigned)__popcll(__ballot(k < r.nv && sqrt(edge_dist2(r.poly[min(k, r.nv - 1)], r.poly[k + 1 < r.nv ? k + 1 : 0],
                                                                         q.x, q.y)) <= r.radius));
        }
        cell = make_uint2(0x40000000u | (e.in ? 0x80000000u : 0u), n);
        if (lane == 0 && n) atomicAdd(r.count, (unsigned long long)n);
    }
    if (lane == 0) {
        r.d[c] = d;
        r.cell[c] = cell;
        r.ref[c] = q;
    }
}

__global__ __launch_bounds__(256) void raster_lists_kernel(Raster r) {
    const int lane = threadIdx.x & 63;
    const int c = (int)(blockIdx.x * (blockDim.x >> 6)) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c >= r.nx * r.ny) return;
    const uint2 cell = r.cell[c];
    if (!(cell.x & 0x40000000u)) return;
    const float2 q = r.ref[c];
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(r.count + 1, (unsigned long long)cell.y);
    uint32_t o = __builtin_amdgcn_readfirstlane((uint32_t)at);
    const uint32_t first = o;
    for (int k0 = 0; k0 < r.nv; k0 += 64) {
        const int k = k0 + lane;
        const bool near = k < r.nv && sqrt(edge_dist2(r.poly[min(k, r.nv - 1)], r.poly[k + 1 < r.nv ? k + 1 : 0], q.x,
                                                      q.y)) <= r.radius;
        const unsigned long long m = __ballot(near);
        if (near) r.edge[o + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)k;
        o += (uint32_t)__popcll(m);
    }
    if (lane == 0) r.cell[c] = make_uint2(cell.x | first, o);
}

// A batch grid's sums of a voxel: the dose, with LET runs beside the numerator
// of its dose-averaged LET (their grids hold 16 bytes a voxel).
template <bool LET>
struct GridSums {
    long long q, let;
    __device__ bool empty() const { return (q | (LET ? let : 0)) == 0; }
};

template <bool LET>
__device__ __forceinline__ GridSums<LET> read_sums(const unsigned long long *qb, size_t i) {
    if constexpr (LET) {
        const ulonglong2 p = reinterpret_cast<const ulonglong2 *>(qb)[i];
        return {(long long)p.x, (long long)p.y};
    } else {
        return {(long long)qb[i], 0};
    }
}

template <bool LET>
__device__ __forceinline__ void clear_sums(unsigned long long *qb, size_t i) {
    if constexpr (LET) reinterpret_cast<ulonglong2 *>(qb)[i] = make_ulonglong2(0ull, 0ull);
    else qb[i] = 0ull;
}

template <bool LET>
__device__ __forceinline__ GridSums<LET> take_sums(unsigned long long *qb, size_t i) {
    const GridSums<LET> g = read_sums<LET>(qb, i);
    if (!g.empty()) clear_sums<LET>(qb, i);
    return g;
}

// ------------------------------------------------------------ batches, dose
// fold nb batches, in order: total += q_b, sum of squares += q_b^2 (FP64), clear q_b
template <bool LET>
__global__ void fold_batch_kernel(unsigned long long *qb, int nb, long long *qt, double *s2, long long *let, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        long long tot = 0, tl = 0;
        double s = 0.0;
        bool any = false;
        for (int b = 0; b < nb; ++b) {
            const GridSums<LET> g = take_sums<LET>(qb, (size_t)b * n + i);
            tl += g.let;
            if (g.q == 0) continue;
            if (!any) {
                any = true;
                s = s2[i];
            }
            tot += g.q;
            s += (double)g.q * (double)g.q;
        }
        if (any) {
            qt[i] += tot;
            s2[i] = s;
        }
        if (LET && tl != 0) let[i] += tl;
    }
}

__global__ void dose_kernel(const long long *q, const double *s2, int B, GeomDev g, double mev_scale,
                            float *dose, float *sigma, size_t n) {
    const float vol_kg = g.sp[0] * g.sp[1] * g.sp[2] * 1e-6f;   // mm^3 -> cm^3 -> kg at 1 g/cm^3
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        float rho = 1.0f;
        int m;
        if (g.kind == 1) hu_material(g.hu[i], m, rho);
        const float conv = (float)mev_scale / (rho * vol_kg);   // Gy per (q unit)
        const long long qi = q[i];
        if (dose) dose[i] = (float)qi * conv;
        if (sigma) {
            // batch estimator of the standard error of the mean (FP64)
            const double D = (double)qi;
            const double var = fmax((double)B * s2[i] - D * D, 0.0) / (double)(B - 1);
            sigma[i] = (float)sqrt(var) * conv;
        }
    }
}

// All batches of a scenario at once: fold_batch_kernel into nothing, then
// dose_kernel, in one pass over the batch grids (8 B a voxel and batch read, 16
// with LET, 16 or 24 B a voxel written; four batches' loads in flight).
// HBM-bound.
template <bool LET>
__global__ __launch_bounds__(256) void fold_dose_kernel(unsigned long long *qb, int B, long long *qt, long long *let,
                                                        GeomDev g, double mev_scale, float *dose, float *sigma,
                                                        size_t n) {
    const float vol_kg = g.sp[0] * g.sp[1] * g.sp[2] * 1e-6f;   // mm^3 -> cm^3 -> kg at 1 g/cm^3
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        long long tot = 0, tl = 0;
        double s = 0.0;
        for (int b0 = 0; b0 < B; b0 += 4) {
            GridSums<LET> q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                q[j] = b0 + j < B ? read_sums<LET>(qb, (size_t)(b0 + j) * n + i) : GridSums<LET>{0, 0};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (q[j].empty()) continue;
                tot += q[j].q;
                tl += q[j].let;
                s += (double)q[j].q * (double)q[j].q;
                clear_sums<LET>(qb, (size_t)(b0 + j) * n + i);
            }
        }
        if (LET) let[i] = tl;
        qt[i] = tot;
        float rho = 1.0f;
        int m;
        if (g.kind == 1) hu_material(g.hu[i], m, rho);
        const float conv = (float)mev_scale / (rho * vol_kg);   // Gy per (q unit)
        if (dose) dose[i] = (float)tot * conv;
        if (sigma) {
            const double D = (double)tot;
            const double var = fmax((double)B * s - D * D, 0.0) / (double)(B - 1);
            sigma[i] = (float)sqrt(var) * conv;
        }
    }
}

}  // namespace

hipError_t launch_transport(const GeomDev &g, const FieldDev &f, const LaunchDev &L, int blocks,
                            int threads, hipStream_t s) {
    if (threads != 256 && threads != 512) threads = kThreads;
    const size_t lds = f.has_block ? (size_t)f.nv * sizeof(float2) : 0;
    // deterministic mode: the double-float instantiation
    if (L.physics == 0) hipLaunchKernelGGL(transport_kernel<true>, dim3(blocks), dim3(threads), lds, s, g, f, L);
    else hipLaunchKernelGGL(transport_kernel<false>, dim3(blocks), dim3(threads), lds, s, g, f, L);
    return hipGetLastError();
}

int queue_threads(unsigned physics, int threads) {
    const int cap = physics == 0 ? 768 : 1024;
    if (threads != 256 && threads != 512 && threads != 768 && threads != 1024) threads = cap;
    return std::min(threads, cap);
}

// LDS per CU (160 KiB) shared by the workgroups that give the CU its target
// waves (16 in physics mode, 12 in double-float mode), less the static tables
int queue_tile_cap(unsigned physics, int threads) {
    threads = queue_threads(physics, threads);
    const int waves_cu = physics == 0 ? 12 : 16;
    const int wgs = std::max(1, waves_cu / (threads / 64));
    const int per_wg = 160 * 1024 / wgs - (int)queue_static_lds(physics);
    return std::max(0, per_wg / 4);
}

size_t queue_static_lds(unsigned physics) { return (tab_hi_floats(3) + (physics == 0 ? tab_lo_floats(3) : 4)) * 4 + 256; }

hipError_t launch_raster(const Raster &r, hipStream_t s) {
    hipLaunchKernelGGL(raster_kernel, dim3((unsigned)((r.nx * r.ny + 3) / 4)), dim3(256), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_raster_lists(const Raster &r, hipStream_t s) {
    hipLaunchKernelGGL(raster_lists_kernel, dim3((unsigned)((r.nx * r.ny + 3) / 4)), dim3(256), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_derive_tables(float *blob, hipStream_t s) {
    hipLaunchKernelGGL(derive_tables_kernel, dim3(NMAT), dim3(NE), 0, s, blob);
    return hipGetLastError();
}

hipError_t launch_density(const int16_t *hu, float *rho, size_t margin, size_t n, hipStream_t s) {
    const int blocks = (int)std::min<size_t>((n + 2 * margin + 255) / 256, 8192);
    hipLaunchKernelGGL(density_kernel, dim3(blocks), dim3(256), 0, s, hu, rho, margin, n);
    return hipGetLastError();
}

hipError_t launch_tile_box(const GeomDev &g, const QueueDev &Q, RowDev *rows, hipStream_t s) {
    if (Q.n_rows > 0)
        hipLaunchKernelGGL(tile_box_kernel, dim3((Q.n_rows + 3) / 4), dim3(256), 0, s, g, Q, rows);
    return hipGetLastError();
}

// beam line of a round: up to 3 workgroups of 256 threads per CU, which is a
// resident set in physics mode (52 to 54 KB of LDS each; with the low tables of
// the double-float mode it is 60 to 62, two fit and the third runs behind them),
// each wave striding over runs of Q.beam_groups groups
hipError_t launch_beam(const GeomDev &g, QueueDev Q, int cus, hipStream_t s) {
    const unsigned long long groups = Q.g_end - Q.g_begin;
    if (groups == 0) return hipSuccess;
    // runs as long as kBeamGroups, shorter where that leaves waves without one
    const unsigned long long waves = (unsigned long long)cus * 12;
    Q.beam_groups = (int)std::max<unsigned long long>(1, std::min<unsigned long long>(kBeamGroups, groups / waves));
    const unsigned long long runs = (groups + Q.beam_groups - 1) / Q.beam_groups;
    const int blocks = (int)std::min<unsigned long long>((runs + 3) / 4, waves / 4);
    const bool x = Q.physics == 0, d = Q.div != 0, de = Q.dense != 0;
#define VPMC_BEAM(X_, D_, E_) hipLaunchKernelGGL((beam_kernel<X_, D_, E_>), dim3(blocks), dim3(256), 0, s, g, Q)
    if (x) {
        if (d) { if (de) VPMC_BEAM(true, true, true); else VPMC_BEAM(true, true, false); }
        else { if (de) VPMC_BEAM(true, false, true); else VPMC_BEAM(true, false, false); }
    } else {
        if (d) { if (de) VPMC_BEAM(false, true, true); else VPMC_BEAM(false, true, false); }
        else { if (de) VPMC_BEAM(false, false, true); else VPMC_BEAM(false, false, false); }
    }
#undef VPMC_BEAM
    return hipGetLastError();
}

hipError_t launch_queue(const GeomDev &g, const QueueDev &Q, int blocks, int threads, hipStream_t s) {
    threads = queue_threads(Q.physics, threads);
    const bool let = Q.dense && Q.let;
    const size_t tile_bytes = (size_t)Q.tile_cap * (let ? 2 : 1) * sizeof(uint32_t);
    constexpr int kAll = PH_STRAGGLE | PH_MCS | PH_NUCLEAR;
#define VPMC_QUEUE(X_, P_)                                                                                         \
    do {                                                                                                           \
        if (!Q.dense)                                                                                              \
            hipLaunchKernelGGL((queue_kernel<X_, P_, false, false>), dim3(blocks), dim3(threads), tile_bytes, s, g, Q); \
        else if (let)                                                                                              \
            hipLaunchKernelGGL((queue_kernel<X_, P_, true, true>), dim3(blocks), dim3(threads), tile_bytes, s, g, Q);   \
        else                                                                                                       \
            hipLaunchKernelGGL((queue_kernel<X_, P_, true, false>), dim3(blocks), dim3(threads), tile_bytes, s, g, Q);  \
    } while (0)
    // all processes together are compiled in; a part of them is read per launch
    if (Q.physics == 0) VPMC_QUEUE(true, 0);
    else if (Q.physics == kAll) VPMC_QUEUE(false, kAll);
    else VPMC_QUEUE(false, -1);
#undef VPMC_QUEUE
    return hipGetLastError();
}

// workgroups (4 waves each) of the compaction passes: one wave per group of
// kCsrGroup (row, chunk) pairs up to 16384 workgroups, the waves striding over
// the rest.  Few chunks hold most of a row, so what an early wave finds is
// uneven: 494 rows of 256 x 256 x 160 voxels (41 M entries) took 761 (count) and
// 1267 us (emit) with 4096 workgroups, 640 and 1045 with 16384, 667 and 1152
// without a limit.
static unsigned csr_pass_blocks(const QueueDev &Q) {
    const size_t ngroup = ((size_t)Q.n_rows * Q.nchunk + kCsrGroup - 1) / kCsrGroup;
    return (unsigned)std::max<size_t>(1, std::min<size_t>((ngroup + 3) / 4, 16384));
}

hipError_t launch_csr_count(const QueueDev &Q, unsigned int *cnt, hipStream_t s) {
    hipLaunchKernelGGL(csr_count_kernel, dim3(csr_pass_blocks(Q)), dim3(256), 0, s, Q, cnt);
    return hipGetLastError();
}

hipError_t launch_csr_chunk_scan(const unsigned int *cnt, unsigned int *coff, unsigned int *rowcnt, int n_rows,
                                 size_t nchunk, hipStream_t s) {
    hipLaunchKernelGGL(csr_chunk_scan_kernel, dim3(n_rows), dim3(1024), 0, s, cnt, coff, rowcnt, nchunk);
    return hipGetLastError();
}

hipError_t launch_csr_offsets(const unsigned int *nnz, int n_rows, int row_begin, unsigned long long *row_off,
                              unsigned long long *row_nnz, unsigned long long *used, unsigned long long capacity,
                              unsigned int *flags, hipStream_t s) {
    hipLaunchKernelGGL(csr_offsets_kernel, dim3(1), dim3(1024), 0, s, nnz, n_rows, row_begin, row_off, row_nnz, used,
                       capacity, flags);
    return hipGetLastError();
}

hipError_t launch_csr_emit(const QueueDev &Q, const unsigned int *cnt, const unsigned int *coff,
                           const unsigned long long *row_off, const unsigned long long *row_nnz, int32_t *col,
                           long long *qv, unsigned long long capacity, unsigned int *flags, hipStream_t s) {
    hipLaunchKernelGGL(csr_emit_kernel, dim3(csr_pass_blocks(Q)), dim3(256), 0, s, Q, cnt, coff, row_off,
                       row_nnz, col, qv, capacity, flags);
    return hipGetLastError();
}

hipError_t launch_atomic_rate(unsigned long long *grid, int nx, int ny, int nz, unsigned long long n_tracks, int len,
                              float sigma, uint32_t seed, hipStream_t s) {
    hipLaunchKernelGGL(atomic_rate_kernel, dim3(4096), dim3(256), 0, s, grid, nx, ny, nz, n_tracks, len, sigma, seed);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, size_t n, unsigned long long v, hipStream_t s) {
    const int blocks = (int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_csr_scatter(const int32_t *col, const long long *qv, unsigned long long begin,
                              unsigned long long end, unsigned long long *dense, hipStream_t s) {
    const unsigned long long n = end - begin;
    const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
    if (blocks > 0) hipLaunchKernelGGL(csr_scatter_kernel, dim3(blocks), dim3(256), 0, s, col, qv, begin, end, dense);
    return hipGetLastError();
}

hipError_t launch_csr_export(const int32_t *col, const long long *qv, size_t n, const GeomDev &g, double mev_scale,
                             int32_t *ocol, float *val, long long *oq, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const int blocks = (int)std::min<size_t>((n + 1023) / 1024, 65536);
    const bool vec = (((uintptr_t)ocol | (uintptr_t)val | (uintptr_t)oq) & 15u) == 0;
    if (vec) hipLaunchKernelGGL(csr_export_kernel<true>, dim3(blocks), dim3(256), 0, s, col, qv, n, g, mev_scale, ocol, val, oq);
    else hipLaunchKernelGGL(csr_export_kernel<false>, dim3(blocks), dim3(256), 0, s, col, qv, n, g, mev_scale, ocol, val, oq);
    return hipGetLastError();
}

hipError_t launch_cell_map(const int32_t *cmap, int nvox, int n_cells, int32_t *cstart, unsigned *st, hipStream_t s) {
    const hipError_t e = launch_fill_u64((unsigned long long *)st, 2, ~0ull, s);
    if (e != hipSuccess) return e;
    const int blocks = std::max(1, std::min((nvox + 255) / 256, 8192));
    hipLaunchKernelGGL(cell_map_kernel, dim3(blocks), dim3(256), 0, s, cmap, nvox, n_cells, cstart, st);
    return hipGetLastError();
}

hipError_t launch_cell_mass(const GeomDev &g, const int32_t *cstart, int n_cells, double *mass, hipStream_t s) {
    const int blocks = std::max(1, std::min((n_cells + 255) / 256, 8192));
    hipLaunchKernelGGL(cell_mass_kernel, dim3(blocks), dim3(256), 0, s, g, cstart, n_cells, mass);
    return hipGetLastError();
}

hipError_t launch_cell_count(const long long *rp, const CellPiece *pcs, long long n_pieces, const int32_t *col,
                             const int32_t *cmap, int nvox, unsigned long long *cnt, unsigned *err, hipStream_t s) {
    if (n_pieces == 0) return hipSuccess;
    const long long blocks = (n_pieces * 64 + 255) / 256;
    hipLaunchKernelGGL(cell_count_kernel, dim3((unsigned)blocks), dim3(256), 0, s, rp, pcs, n_pieces, col, cmap, nvox,
                       cnt, err);
    return hipGetLastError();
}

hipError_t launch_cell_rows(const long long *first_piece, const long long *pout, size_t n, long long *rp_out,
                            hipStream_t s) {
    hipLaunchKernelGGL(cell_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, first_piece, pout, n, rp_out);
    return hipGetLastError();
}

hipError_t launch_cell_emit(const long long *rp, const CellPiece *pcs, long long n_pieces, const int32_t *col,
                            const long long *q, const int32_t *cmap, const long long *pout, const double *mass,
                            double mev_scale, int32_t *ocell, long long *oq, float *oval, hipStream_t s) {
    if (n_pieces == 0) return hipSuccess;
    const long long blocks = (n_pieces * 64 + 255) / 256;
    hipLaunchKernelGGL(cell_emit_kernel, dim3((unsigned)blocks), dim3(256), 0, s, rp, pcs, n_pieces, col, q, cmap,
                       pout, mass, mev_scale, ocell, oq, oval);
    return hipGetLastError();
}

hipError_t launch_sur_resume(const GeomDev &g, const FieldDev &f, const LaunchDev &L, const DeferRec *rec,
                             const float *out, unsigned long long n, float p_lo, float p_hi, hipStream_t s) {
    const int blocks = (int)std::max<unsigned long long>(1, std::min<unsigned long long>((n + 255) / 256, 4096));
    const size_t lds = (size_t)f.nv * sizeof(float2);
    if (L.physics == 0)
        hipLaunchKernelGGL(sur_resume_kernel<true>, dim3(blocks), dim3(256), lds, s, g, f, L, rec, out, n, p_lo, p_hi);
    else
        hipLaunchKernelGGL(sur_resume_kernel<false>, dim3(blocks), dim3(256), lds, s, g, f, L, rec, out, n, p_lo, p_hi);
    return hipGetLastError();
}

hipError_t launch_sur_resume_csr(const GeomDev &g, const QueueDev &Q, const DeferRec *rec, const float *out,
                                 unsigned long long n, float p_lo, float p_hi, hipStream_t s) {
    const int blocks = (int)std::max<unsigned long long>(1, std::min<unsigned long long>((n + 255) / 256, 4096));
    const size_t lds = (size_t)Q.n_poly_total * sizeof(float2);
    if (Q.physics == 0)
        hipLaunchKernelGGL(sur_resume_csr_kernel<true>, dim3(blocks), dim3(256), lds, s, g, Q, rec, out, n, p_lo, p_hi);
    else
        hipLaunchKernelGGL(sur_resume_csr_kernel<false>, dim3(blocks), dim3(256), lds, s, g, Q, rec, out, n, p_lo, p_hi);
    return hipGetLastError();
}

hipError_t launch_surrogate_sample(const FieldDev &f, const float *entries, int n, uint32_t key0, uint32_t key1,
                                   unsigned physics, const float *tables, float *x, float *y, float *t, hipStream_t s) {
    const int blocks = std::max(1, std::min((n + 255) / 256, 4096));
    hipLaunchKernelGGL(surrogate_sample_kernel, dim3(blocks), dim3(256), 0, s, f, entries, n, key0, key1, physics,
                       tables, x, y, t);
    return hipGetLastError();
}

hipError_t launch_fold_batch(unsigned long long *qb, int nb, long long *qt, double *s2, long long *let, size_t n,
                             hipStream_t s) {
    const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
    if (let) hipLaunchKernelGGL(fold_batch_kernel<true>, dim3(blocks), dim3(256), 0, s, qb, nb, qt, s2, let, n);
    else hipLaunchKernelGGL(fold_batch_kernel<false>, dim3(blocks), dim3(256), 0, s, qb, nb, qt, s2, let, n);
    return hipGetLastError();
}

hipError_t launch_fold_dose(unsigned long long *qb, int B, long long *qt, long long *let, const GeomDev &g,
                            double mev_scale, float *dose, float *sigma, size_t n, hipStream_t s) {
    const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
    if (let) hipLaunchKernelGGL(fold_dose_kernel<true>, dim3(blocks), dim3(256), 0, s, qb, B, qt, let, g, mev_scale, dose, sigma, n);
    else hipLaunchKernelGGL(fold_dose_kernel<false>, dim3(blocks), dim3(256), 0, s, qb, B, qt, let, g, mev_scale, dose, sigma, n);
    return hipGetLastError();
}

hipError_t launch_dose(const long long *q, const double *s2, int B, const GeomDev &g, double mev_scale,
                       float *dose, float *sigma, size_t n, hipStream_t s) {
    const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
    hipLaunchKernelGGL(dose_kernel, dim3(blocks), dim3(256), 0, s, q, s2, B, g, mev_scale, dose, sigma, n);
    return hipGetLastError();
}

// Scratch of the allocation-free dense run.  In host code the name `scratch`
// is only a host-side stand-in for the array: kernels and copies get the
// device address from scratch_device_ptr(), never the name itself.
static __device__ __align__(256) unsigned long long scratch[kScratchBytes / sizeof(unsigned long long)];

hipError_t scratch_device_ptr(int device, void **out) {
    static std::mutex mu;
    static void *addr[kMaxScratchDevices] = {};
    if (!out || device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;   // the symbol is looked up on the current device
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

}  // namespace vpmc
