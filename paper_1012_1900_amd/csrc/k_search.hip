// The gamma search (Algorithm A1 step 4 run as Algorithm A2 step 6, "Kernel 3").
//
// One lane per reference node, in the work order the sort produced.  A wave walks the
// sorted cell table in lockstep: entry n is wave-uniform (one scalar load of a 64-byte
// row), a lane takes part while key_n^2 < gamma^2 of that lane, and the wave leaves the
// walk as soon as no lane does (ballot).  This is the paper's early break, exact because
// the key is a lower bound of every face the cell owns.
//
// Faces.  The Kuhn triangulation splits each cube along its main diagonal; its faces are
// chains q -> q+1_B1 -> q+1_B1+1_B2 -> ... with disjoint non-empty axis blocks B_j.  A
// cell owns the faces anchored at its lower corner q: 1 vertex, 7 edges, 12 triangles and
// 6 tetrahedra in 3D (1, 3, 2 in 2D), so every face of the triangulation is evaluated by
// exactly one cell, and a face owned by cell q lies inside the closed cell q.  Like the
// paper's GPU kernel (Sec. 2.2) every face is evaluated instead of Ju's branching
// recursion.
//
// Projection.  In coordinates relative to the reference node, normalised by DTA and dD,
// a face point is  x_i = s_i (a_i + t_j) for i in B_j  (s_i = h_i / DTA, a = cell offset),
// dose G = g_0 + sum_j t_j Delta_j  (g_k = (D_e(v_k) - D_r) / dD, Delta_j = g_j - g_{j-1}),
// with 1 >= t_1 >= ... >= t_k >= 0.  The Gram matrix of the chain edges is
// diag(sigma_j^2) + Delta Delta^T (sigma_j^2 = sum_{i in B_j} s_i^2), whose inverse is
// closed-form (Sherman-Morrison).  With mu_j = sum_{i in B_j} s_i^2 a_i / sigma_j^2:
//     N = g_0 - sum_j Delta_j mu_j          (value of the face's affine dose at the node)
//     Den = 1 + sum_j Delta_j^2 / sigma_j^2
//     Lambda = N / Den,   t_j = -mu_j - Delta_j Lambda / sigma_j^2
//     dist^2 = perp + N Lambda               (perp: spatial part no t can remove)
// which is the normal-equation solution w = (V^T V)^-1 V^T P of Sec. 2.1 for this edge
// basis; the projection counts when the t_j satisfy the chain inequalities (all
// barycentric weights >= 0).  No residual is formed by subtracting large squares.
#include <cfloat>
#include <type_traits>

#include "internal.hpp"

namespace gammax {

namespace {

constexpr int WAVE = 64;
constexpr int SEARCH_THREADS = 256;

template <typename T>
struct Num;
template <>
struct Num<float> {
    static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float inf() { return __builtin_huge_valf(); }
    static __device__ __forceinline__ float min(float a, float b) { return __builtin_fminf(a, b); }
    static __device__ __forceinline__ float max(float a, float b) { return __builtin_fmaxf(a, b); }
};
template <>
struct Num<double> {
    static __device__ __forceinline__ double rcp(double x) { return 1.0 / x; }
    static __device__ __forceinline__ double inf() { return __builtin_huge_val(); }
    static __device__ __forceinline__ double min(double a, double b) { return __builtin_fmin(a, b); }
    static __device__ __forceinline__ double max(double a, double b) { return __builtin_fmax(a, b); }
};

template <typename T>
__device__ __forceinline__ T vmin(T a, T b) { return Num<T>::min(a, b); }
template <typename T>
__device__ __forceinline__ T vmax(T a, T b) { return Num<T>::max(a, b); }

// Fused multiply-add, written out: the projections below form every product-sum they fuse
// explicitly and the compiler contracts nothing else in them (contraction off), so each
// instantiation of a face (masked or not, in any kernel and any lane layout) computes the same
// bits whatever code surrounds it.
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// One chain step: Delta and w = Delta / sigma^2 (Delta^2 / sigma^2 = Delta w and Delta mu
// enter the sums below as fused products).
template <typename T>
struct Step {
    T d, w;
};
template <typename T>
__device__ __forceinline__ Step<T> mk_step(T hi, T lo, T inv_s2) {
#pragma clang fp contract(off)
    Step<T> s;
    s.d = hi - lo;
    s.w = s.d * inv_s2;
    return s;
}
// N after a step: N - Delta mu; Den after a step: Den + Delta^2 / sigma^2.
template <typename T>
__device__ __forceinline__ T n_step(T n, const Step<T>& s, T mu) { return fmadd(-s.d, mu, n); }
template <typename T>
__device__ __forceinline__ T den_step(T den, const Step<T>& s) { return fmadd(s.d, s.w, den); }
// Chain parameter of a step at Lambda: t = -mu - w Lambda.
template <typename T>
__device__ __forceinline__ T t_step(const Step<T>& s, T mu, T L) { return fmadd(-s.w, L, -mu); }

template <typename T>
__device__ __forceinline__ T face1(T g0, const Step<T>& a, T mua, T perp) {
#pragma clang fp contract(off)
    const T N = n_step(g0, a, mua);
    const T L = N * Num<T>::rcp(den_step(T(1), a));
    const T t1 = t_step(a, mua, L);
    return (t1 >= T(0) && t1 <= T(1)) ? fmadd(N, L, perp) : Num<T>::inf();
}
template <typename T>
__device__ __forceinline__ T face2(T g0, const Step<T>& a, T mua, const Step<T>& b, T mub, T perp) {
#pragma clang fp contract(off)
    const T N = n_step(n_step(g0, a, mua), b, mub);
    const T L = N * Num<T>::rcp(den_step(den_step(T(1), a), b));
    const T t1 = t_step(a, mua, L);
    const T t2 = t_step(b, mub, L);
    return (t1 <= T(1) && t1 >= t2 && t2 >= T(0)) ? fmadd(N, L, perp) : Num<T>::inf();
}
// The denominator of a tetrahedron (its guard measure) on its own.
template <typename T>
__device__ __forceinline__ T den3(const Step<T>& a, const Step<T>& b, const Step<T>& c) {
    return den_step(den_step(den_step(T(1), a), b), c);
}
template <typename T>
__device__ __forceinline__ T face3(T g0, const Step<T>& a, T mua, const Step<T>& b, T mub,
                                   const Step<T>& c, T muc, T& den_out) {
#pragma clang fp contract(off)
    const T N = n_step(n_step(n_step(g0, a, mua), b, mub), c, muc);
    const T den = den3(a, b, c);
    den_out = den;
    const T L = N * Num<T>::rcp(den);
    const T t1 = t_step(a, mua, L);
    const T t2 = t_step(b, mub, L);
    const T t3 = t_step(c, muc, L);
    return (t1 <= T(1) && t1 >= t2 && t2 >= t3 && t3 >= T(0)) ? N * L : Num<T>::inf();
}

// Spatial constants of one cell offset (uniform over the wave).
template <typename T>
struct Geo {
    T ax, ay, az, px, py, pz, vxy, vxz, vyz, vxyz, mxy, mxz, myz, mxyz;
};

__device__ __forceinline__ Geo<float> geo_from_row(const TabEntry& e) {
    Geo<float> g;
    g.ax = (float)e.ax; g.ay = (float)e.ay; g.az = (float)e.az;
    g.px = e.px; g.py = e.py; g.pz = e.pz;
    g.vxy = e.vxy; g.vxz = e.vxz; g.vyz = e.vyz; g.vxyz = e.vxyz;
    g.mxy = e.mxy; g.mxz = e.mxz; g.myz = e.myz; g.mxyz = e.mxyz;
    return g;
}

__device__ __forceinline__ Geo<double> geo_fp64(int iax, int iay, int iaz, double sx2, double sy2,
                                                double sz2) {
    Geo<double> g;
    const double ax = iax, ay = iay, az = iaz;
    g.ax = ax; g.ay = ay; g.az = az;
    g.px = sx2 * ax * ax; g.py = sy2 * ay * ay; g.pz = sz2 * az * az;
    const double dxy = ax - ay, dxz = ax - az, dyz = ay - az;
    g.vxy = sx2 * sy2 * dxy * dxy / (sx2 + sy2);
    g.mxy = (sx2 * ax + sy2 * ay) / (sx2 + sy2);
    if (sz2 > 0.0) {
        const double s = sx2 + sy2 + sz2;
        g.vxz = sx2 * sz2 * dxz * dxz / (sx2 + sz2);
        g.vyz = sy2 * sz2 * dyz * dyz / (sy2 + sz2);
        g.vxyz = (sx2 * sy2 * dxy * dxy + sx2 * sz2 * dxz * dxz + sy2 * sz2 * dyz * dyz) / s;
        g.mxz = (sx2 * ax + sz2 * az) / (sx2 + sz2);
        g.myz = (sy2 * ay + sz2 * az) / (sy2 + sz2);
        g.mxyz = (sx2 * ax + sy2 * ay + sz2 * az) / s;
    } else {
        g.vxz = g.vyz = g.vxyz = g.mxz = g.myz = g.mxyz = 0.0;
    }
    return g;
}

// 1/sigma^2 of the chain blocks x, y, z, xy, xz, yz, xyz.
template <typename T>
struct InvS2 {
    T x, y, z, xy, xz, yz, xyz;
};
template <typename T>
__device__ __forceinline__ InvS2<T> inv_s2(T sx2, T sy2, T sz2) {
    InvS2<T> r;
    r.x = T(1) / sx2;
    r.y = T(1) / sy2;
    r.z = sz2 > T(0) ? T(1) / sz2 : T(0);
    r.xy = T(1) / (sx2 + sy2);
    r.xz = sz2 > T(0) ? T(1) / (sx2 + sz2) : T(0);
    r.yz = sz2 > T(0) ? T(1) / (sy2 + sz2) : T(0);
    r.xyz = T(1) / (sx2 + sy2 + sz2);
    return r;
}

// The FP32 reciprocals as the host formed them for the search arguments (the same IEEE
// divisions as inv_s2<float>, once per map instead of once per lane).
__device__ __forceinline__ InvS2<float> inv_s2_of(const SearchArgs& a) {
    InvS2<float> r;
    r.x = a.inv_s2[0];
    r.y = a.inv_s2[1];
    r.z = a.inv_s2[2];
    r.xy = a.inv_s2[3];
    r.xz = a.inv_s2[4];
    r.yz = a.inv_s2[5];
    r.xyz = a.inv_s2[6];
    return r;
}

// The reciprocals in T (FP64: formed by the host too).
template <typename T>
__device__ __forceinline__ InvS2<T> inv_s2_for(const SearchArgs& a) {
    if constexpr (sizeof(T) == 8) {
        InvS2<double> r;
        r.x = a.inv_s2d[0];
        r.y = a.inv_s2d[1];
        r.z = a.inv_s2d[2];
        r.xy = a.inv_s2d[3];
        r.xz = a.inv_s2d[4];
        r.yz = a.inv_s2d[5];
        r.xyz = a.inv_s2d[6];
        return r;
    } else {
        return inv_s2_of(a);
    }
}

// 1 / dD of a node in the FP64 paths.
__device__ __forceinline__ double fp64_inv_dd(const SearchArgs& a, float dr) {
    return a.local ? 1.0 / (a.dd64 * (double)dr) : 1.0 / (a.dd64 * (double)ord_to_float(a.sc->dmax_ord));
}

// Tetrahedron of a 3D cell redone in FP64 (the precision guard).  The four corner doses
// are re-read from memory so that the common FP32 path keeps no extra registers alive.
// perm: 0 xyz, 1 xzy, 2 yxz, 3 yzx, 4 zxy, 5 zyx (order in which the axes are stepped).
struct GuardCtx {
    const float* ev;
    int base, ox, oy, oz;
    float dr;
    double inv_dd;
    int ax, ay, az;
    double sx2, sy2, sz2;
};

template <typename V>
__device__ __forceinline__ V pick3(int i, V x, V y, V z) {
    return i == 0 ? x : (i == 1 ? y : z);
}

__device__ __forceinline__ double tet_fp64(const GuardCtx& c, int perm) {
    // perm -> stepping order: first axis perm/2, then the other two ascending (even perm)
    // or descending (odd perm)
    const int first = perm >> 1;
    int r0 = first == 0 ? 1 : 0, r1 = first == 2 ? 1 : 2;
    if (perm & 1) {
        const int t = r0;
        r0 = r1;
        r1 = t;
    }
    const double dr = (double)c.dr;
    int idx = c.base;
    double gprev = ((double)c.ev[idx] - dr) * c.inv_dd;
    double N = gprev, den = 1.0;
    double tw0 = 0.0, tw1 = 0.0, tw2 = 0.0, mu0 = 0.0, mu1 = 0.0, mu2 = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int ax = j == 0 ? first : (j == 1 ? r0 : r1);
        idx += pick3(ax, c.ox, c.oy, c.oz);
        const double s2 = pick3(ax, c.sx2, c.sy2, c.sz2);
        const double aa = (double)pick3(ax, c.ax, c.ay, c.az);
        const double gnext = ((double)c.ev[idx] - dr) * c.inv_dd;
        const double d = gnext - gprev;
        N -= d * aa;
        den += d * d / s2;
        const double tw = d / s2;
        if (j == 0) { tw0 = tw; mu0 = aa; }
        if (j == 1) { tw1 = tw; mu1 = aa; }
        if (j == 2) { tw2 = tw; mu2 = aa; }
        gprev = gnext;
    }
    const double L = N / den;
    const double t1 = -mu0 - tw0 * L, t2 = -mu1 - tw1 * L, t3 = -mu2 - tw2 * L;
    return (t1 <= 1.0 && t1 >= t2 && t2 >= t3 && t3 >= 0.0) ? N * L : __builtin_huge_val();
}

// Normalised dose difference of a cell vertex, rounded as its own product: the walks of
// every tail layout feed the projections the same values, whatever the compiler fuses
// around them.
template <typename T>
__device__ __forceinline__ T dose_norm(T v, T dr, T inv) {
#pragma clang fp contract(off)
    return (v - dr) * inv;
}

// The corner doses of a cell whose lower corner has index b0 (a corner past the grid along an
// axis: the one before it).  The corners of a row are one 8-byte load (4-byte aligned; on the
// last column the pair before it): four loads per cell where eight gathers touched twice the
// cache lines.
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
template <int DIM>
__device__ __forceinline__ void cell_corners(const float* __restrict__ ev, int64_t b0, bool okx, int oy, int oz, float* v) {
    const float* p = ev + b0 - (okx ? 0 : 1);
#pragma unroll
    for (int k = 0; k < (DIM == 3 ? 4 : 2); ++k) {
        const f32x2u t = *reinterpret_cast<const f32x2u*>(p + ((k & 1) ? oy : 0) + ((k & 2) ? oz : 0));
        v[2 * k] = okx ? t.x : t.y;
        v[2 * k + 1] = t.y;
    }
}

// Whether any of the six tetrahedra of a 3D cell has a normal-equation denominator above
// den_guard: the test cell3 applies (GMODE 1), with its chain steps and its summation order.
__device__ __forceinline__ bool tets_ill(const float* g, const InvS2<float>& is, float den_guard) {
#pragma clang fp contract(off)
    const Step<float> s0x = mk_step(g[1], g[0], is.x), s0y = mk_step(g[2], g[0], is.y);
    const Step<float> s0z = mk_step(g[4], g[0], is.z);
    const Step<float> s1y = mk_step(g[3], g[1], is.y), s1z = mk_step(g[5], g[1], is.z);
    const Step<float> s2x = mk_step(g[3], g[2], is.x), s2z = mk_step(g[6], g[2], is.z);
    const Step<float> s4x = mk_step(g[5], g[4], is.x), s4y = mk_step(g[6], g[4], is.y);
    const Step<float> s3z = mk_step(g[7], g[3], is.z), s5y = mk_step(g[7], g[5], is.y);
    const Step<float> s6x = mk_step(g[7], g[6], is.x);
    bool ill = den3(s0x, s1y, s3z) > den_guard;
    ill = ill || den3(s0x, s1z, s5y) > den_guard;
    ill = ill || den3(s0y, s2x, s3z) > den_guard;
    ill = ill || den3(s0y, s2z, s6x) > den_guard;
    ill = ill || den3(s0z, s4x, s5y) > den_guard;
    ill = ill || den3(s0z, s4y, s6x) > den_guard;
    return ill;
}

// All faces owned by one 3D cell; returns the smallest dist^2 (or +inf).
// ok_*: the cell extends along that axis inside the grid (MASKED only).
// GMODE 0: no guard; 1: flag an ill-conditioned tetrahedron (ill = true); 2: project it
// again in FP64.
template <typename T, bool MASKED, int GMODE>
__device__ __forceinline__ T cell3(const T* g, const Geo<T>& G, const InvS2<T>& is, bool okx, bool oky,
                                   bool okz, T den_guard, const GuardCtx& gc, uint32_t& n_fp64,
                                   bool& ill) {
#pragma clang fp contract(off)
    const T INF = Num<T>::inf();
    const T g0 = g[0];
    // chain steps, named by start vertex bits and block (x = bit0, y = bit1, z = bit2)
    const Step<T> s0x = mk_step(g[1], g[0], is.x);
    const Step<T> s0y = mk_step(g[2], g[0], is.y);
    const Step<T> s0z = mk_step(g[4], g[0], is.z);
    const Step<T> s0xy = mk_step(g[3], g[0], is.xy);
    const Step<T> s0xz = mk_step(g[5], g[0], is.xz);
    const Step<T> s0yz = mk_step(g[6], g[0], is.yz);
    const Step<T> s0xyz = mk_step(g[7], g[0], is.xyz);
    const Step<T> s1y = mk_step(g[3], g[1], is.y);
    const Step<T> s1z = mk_step(g[5], g[1], is.z);
    const Step<T> s1yz = mk_step(g[7], g[1], is.yz);
    const Step<T> s2x = mk_step(g[3], g[2], is.x);
    const Step<T> s2z = mk_step(g[6], g[2], is.z);
    const Step<T> s2xz = mk_step(g[7], g[2], is.xz);
    const Step<T> s4x = mk_step(g[5], g[4], is.x);
    const Step<T> s4y = mk_step(g[6], g[4], is.y);
    const Step<T> s4xy = mk_step(g[7], g[4], is.xy);
    const Step<T> s3z = mk_step(g[7], g[3], is.z);
    const Step<T> s5y = mk_step(g[7], g[5], is.y);
    const Step<T> s6x = mk_step(g[7], g[6], is.x);
    // vertex q
    T best = fmadd(g0, g0, (G.px + G.py) + G.pz);
    // edges
    T e;
    e = face1(g0, s0x, G.ax, G.py + G.pz);
    best = vmin<T>(best, (!MASKED || okx) ? e : INF);
    e = face1(g0, s0y, G.ay, G.px + G.pz);
    best = vmin<T>(best, (!MASKED || oky) ? e : INF);
    e = face1(g0, s0z, G.az, G.px + G.py);
    best = vmin<T>(best, (!MASKED || okz) ? e : INF);
    e = face1(g0, s0xy, G.mxy, G.pz + G.vxy);
    best = vmin<T>(best, (!MASKED || (okx && oky)) ? e : INF);
    e = face1(g0, s0xz, G.mxz, G.py + G.vxz);
    best = vmin<T>(best, (!MASKED || (okx && okz)) ? e : INF);
    e = face1(g0, s0yz, G.myz, G.px + G.vyz);
    best = vmin<T>(best, (!MASKED || (oky && okz)) ? e : INF);
    const bool all = !MASKED || (okx && oky && okz);
    e = face1(g0, s0xyz, G.mxyz, G.vxyz);
    best = vmin<T>(best, all ? e : INF);
    // triangles in the cube faces through q
    T tri = vmin<T>(face2(g0, s0x, G.ax, s1y, G.ay, G.pz), face2(g0, s0y, G.ay, s2x, G.ax, G.pz));
    best = vmin<T>(best, (!MASKED || (okx && oky)) ? tri : INF);
    tri = vmin<T>(face2(g0, s0x, G.ax, s1z, G.az, G.py), face2(g0, s0z, G.az, s4x, G.ax, G.py));
    best = vmin<T>(best, (!MASKED || (okx && okz)) ? tri : INF);
    tri = vmin<T>(face2(g0, s0y, G.ay, s2z, G.az, G.px), face2(g0, s0z, G.az, s4y, G.ay, G.px));
    best = vmin<T>(best, (!MASKED || (oky && okz)) ? tri : INF);
    // triangles through the main diagonal
    T diag = vmin<T>(face2(g0, s0x, G.ax, s1yz, G.myz, G.vyz), face2(g0, s0yz, G.myz, s6x, G.ax, G.vyz));
    diag = vmin<T>(diag, vmin<T>(face2(g0, s0y, G.ay, s2xz, G.mxz, G.vxz), face2(g0, s0xz, G.mxz, s5y, G.ay, G.vxz)));
    diag = vmin<T>(diag, vmin<T>(face2(g0, s0z, G.az, s4xy, G.mxy, G.vxy), face2(g0, s0xy, G.mxy, s3z, G.az, G.vxy)));
    // tetrahedra
    T den[6], tv[6];
    tv[0] = face3(g0, s0x, G.ax, s1y, G.ay, s3z, G.az, den[0]);
    tv[1] = face3(g0, s0x, G.ax, s1z, G.az, s5y, G.ay, den[1]);
    tv[2] = face3(g0, s0y, G.ay, s2x, G.ax, s3z, G.az, den[2]);
    tv[3] = face3(g0, s0y, G.ay, s2z, G.az, s6x, G.ax, den[3]);
    tv[4] = face3(g0, s0z, G.az, s4x, G.ax, s5y, G.ay, den[4]);
    tv[5] = face3(g0, s0z, G.az, s4y, G.ay, s6x, G.ax, den[5]);
    uint32_t gmask = 0u;
    if (GMODE != 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) gmask |= (den[k] > den_guard) ? (1u << k) : 0u;
    }
    if (GMODE == 1) ill = ill || (all && gmask != 0u);
    if (GMODE == 2) {
#pragma unroll
        for (int k = 0; k < 6; ++k) tv[k] = ((gmask >> k) & 1u) ? INF : tv[k];
    }
    T tet = vmin<T>(vmin<T>(vmin<T>(tv[0], tv[1]), vmin<T>(tv[2], tv[3])), vmin<T>(tv[4], tv[5]));
    if (GMODE == 2 && all && gmask) {
        // rare: ill-conditioned tetrahedra are projected again in FP64
#pragma nounroll
        for (int k = 0; k < 6; ++k) {
            if ((gmask >> k) & 1u) {
                tet = vmin<T>(tet, (T)tet_fp64(gc, k));
                ++n_fp64;
            }
        }
    }
    diag = vmin<T>(diag, tet);
    best = vmin<T>(best, all ? diag : INF);
    return best;
}


// ---- Ju et al.'s recursion (Sec. 2.1: the branching form of the A1 distance) -------------
//
// The same closed-form chain projections as cell3, organised as the recursion of the
// sequential algorithm: each of the six Kuhn tetrahedra of a cell is projected first, and
// only where a barycentric weight is negative are the facets opposite those vertices
// projected, then their edges, then vertices.  It covers every face of the cell (not only
// the faces the cell owns), so it serves interior cells; cells at the grid faces keep
// cell3.  A chain starts at cube vertex U (bit i: +1 along axis i, x = bit 0) and steps
// through disjoint axis blocks S1, S2, ... that do not meet U.
struct JuCell {
    float g[8];
    float a[3], p[3], p1[3];   // per axis: offset, s^2 a^2, s^2 (a + 1)^2
    Geo<float> G;
    InvS2<float> is;
};
template <int S>
__device__ __forceinline__ float ju_mu(const JuCell& K) {
    static_assert(S >= 1 && S <= 7, "block");
    if constexpr (S == 1) return K.a[0];
    else if constexpr (S == 2) return K.a[1];
    else if constexpr (S == 4) return K.a[2];
    else if constexpr (S == 3) return K.G.mxy;
    else if constexpr (S == 5) return K.G.mxz;
    else if constexpr (S == 6) return K.G.myz;
    else return K.G.mxyz;
}
template <int S>
__device__ __forceinline__ float ju_inv(const JuCell& K) {
    if constexpr (S == 1) return K.is.x;
    else if constexpr (S == 2) return K.is.y;
    else if constexpr (S == 4) return K.is.z;
    else if constexpr (S == 3) return K.is.xy;
    else if constexpr (S == 5) return K.is.xz;
    else if constexpr (S == 6) return K.is.yz;
    else return K.is.xyz;
}
template <int S>
__device__ __forceinline__ float ju_res(const JuCell& K) {
    if constexpr (S == 1 || S == 2 || S == 4) return 0.0f;
    else if constexpr (S == 3) return K.G.vxy;
    else if constexpr (S == 5) return K.G.vxz;
    else if constexpr (S == 6) return K.G.vyz;
    else return K.G.vxyz;
}
// sum of the squared spatial components of vertex U over the axes outside mask S
template <int U, int S>
__device__ __forceinline__ float ju_perp(const JuCell& K) {
    float r = 0.0f;
    if constexpr (!(S & 1)) r += (U & 1) ? K.p1[0] : K.p[0];
    if constexpr (!(S & 2)) r += (U & 2) ? K.p1[1] : K.p[1];
    if constexpr (!(S & 4)) r += (U & 4) ? K.p1[2] : K.p[2];
    return r;
}
template <int U>
__device__ __forceinline__ float ju_vertex(const JuCell& K) {
#pragma clang fp contract(off)
    return fmadd(K.g[U], K.g[U], ju_perp<U, 0>(K));
}
template <int U, int S>
__device__ __forceinline__ Step<float> ju_step(const JuCell& K) {
    static_assert((U & S) == 0, "a chain steps away from its start");
    return mk_step(K.g[U | S], K.g[U], ju_inv<S>(K));
}
// edge from U along block S
template <int U, int S>
__device__ __forceinline__ float ju_edge(const JuCell& K) {
#pragma clang fp contract(off)
    const Step<float> a = ju_step<U, S>(K);
    const float N = n_step(K.g[U], a, ju_mu<S>(K));
    const float L = N * Num<float>::rcp(den_step(1.0f, a));
    const float t = t_step(a, ju_mu<S>(K), L);
    if (t >= 0.0f && t <= 1.0f) return fmadd(N, L, ju_perp<U, S>(K) + ju_res<S>(K));
    return t < 0.0f ? ju_vertex<U>(K) : ju_vertex<U | S>(K);
}
// triangle from U through blocks S1 then S2
template <int U, int S1, int S2>
__device__ __forceinline__ float ju_tri(const JuCell& K) {
#pragma clang fp contract(off)
    const Step<float> a = ju_step<U, S1>(K);
    const Step<float> b = ju_step<U | S1, S2>(K);
    const float N = n_step(n_step(K.g[U], a, ju_mu<S1>(K)), b, ju_mu<S2>(K));
    const float L = N * Num<float>::rcp(den_step(den_step(1.0f, a), b));
    const float t1 = t_step(a, ju_mu<S1>(K), L);
    const float t2 = t_step(b, ju_mu<S2>(K), L);
    const float w0 = 1.0f - t1, w1 = t1 - t2, w2 = t2;
    if (w0 >= 0.0f && w1 >= 0.0f && w2 >= 0.0f)
        return fmadd(N, L, (ju_perp<U, S1 | S2>(K) + ju_res<S1>(K)) + ju_res<S2>(K));
    float best = Num<float>::inf();
    if (w0 < 0.0f) best = vmin<float>(best, ju_edge<U | S1, S2>(K));
    if (w1 < 0.0f) best = vmin<float>(best, ju_edge<U, S1 | S2>(K));
    if (w2 < 0.0f) best = vmin<float>(best, ju_edge<U, S1>(K));
    return best;
}
// tetrahedron v0 -> A -> A+B -> A+B+C (axis masks A, B, C); den: its normal-equation
// denominator (the guard's measure)
template <int A, int B, int C>
__device__ __forceinline__ float ju_tet(const JuCell& K, float& den) {
#pragma clang fp contract(off)
    const Step<float> a = ju_step<0, A>(K);
    const Step<float> b = ju_step<A, B>(K);
    const Step<float> c = ju_step<A | B, C>(K);
    const float N = n_step(n_step(n_step(K.g[0], a, ju_mu<A>(K)), b, ju_mu<B>(K)), c, ju_mu<C>(K));
    den = den3(a, b, c);
    const float L = N * Num<float>::rcp(den);
    const float t1 = t_step(a, ju_mu<A>(K), L);
    const float t2 = t_step(b, ju_mu<B>(K), L);
    const float t3 = t_step(c, ju_mu<C>(K), L);
    const float w0 = 1.0f - t1, w1 = t1 - t2, w2 = t2 - t3, w3 = t3;
    if (w0 >= 0.0f && w1 >= 0.0f && w2 >= 0.0f && w3 >= 0.0f) return N * L;
    float best = Num<float>::inf();
    if (w0 < 0.0f) best = vmin<float>(best, ju_tri<A, B, C>(K));          // drop v0
    if (w1 < 0.0f) best = vmin<float>(best, ju_tri<0, A | B, C>(K));      // drop v0+A
    if (w2 < 0.0f) best = vmin<float>(best, ju_tri<0, A, B | C>(K));      // drop v0+A+B
    if (w3 < 0.0f) best = vmin<float>(best, ju_tri<0, A, B>(K));          // drop v0+A+B+C
    return best;
}
// Interior 3D cell by Ju's recursion: the smallest dist^2 over its six tetrahedra.
// GMODE 1 flags a tetrahedron whose denominator exceeds den_guard (as cell3 does).
template <int GMODE>
__device__ __forceinline__ float cell3_ju(const float* g, const Geo<float>& G, const InvS2<float>& is, float s2x,
                                          float s2y, float s2z, float den_guard, bool& ill) {
    JuCell K;
#pragma unroll
    for (int b = 0; b < 8; ++b) K.g[b] = g[b];
    K.a[0] = G.ax;
    K.a[1] = G.ay;
    K.a[2] = G.az;
    K.p[0] = G.px;
    K.p[1] = G.py;
    K.p[2] = G.pz;
    K.p1[0] = s2x * (G.ax + 1.0f) * (G.ax + 1.0f);
    K.p1[1] = s2y * (G.ay + 1.0f) * (G.ay + 1.0f);
    K.p1[2] = s2z * (G.az + 1.0f) * (G.az + 1.0f);
    K.G = G;
    K.is = is;
    float den = 0.0f;
    bool flag = false;
    float best = ju_tet<1, 2, 4>(K, den);
    flag = flag || den > den_guard;
    best = vmin<float>(best, ju_tet<1, 4, 2>(K, den));
    flag = flag || den > den_guard;
    best = vmin<float>(best, ju_tet<2, 1, 4>(K, den));
    flag = flag || den > den_guard;
    best = vmin<float>(best, ju_tet<2, 4, 1>(K, den));
    flag = flag || den > den_guard;
    best = vmin<float>(best, ju_tet<4, 1, 2>(K, den));
    flag = flag || den > den_guard;
    best = vmin<float>(best, ju_tet<4, 2, 1>(K, den));
    flag = flag || den > den_guard;
    if constexpr (GMODE == 1) ill = ill || flag;
    return best;
}

template <typename T, bool MASKED>
__device__ __forceinline__ T cell2(const T* g, const Geo<T>& G, const InvS2<T>& is, bool okx, bool oky) {
#pragma clang fp contract(off)
    const T INF = Num<T>::inf();
    const T g0 = g[0];
    const Step<T> s0x = mk_step(g[1], g[0], is.x);
    const Step<T> s0y = mk_step(g[2], g[0], is.y);
    const Step<T> s0xy = mk_step(g[3], g[0], is.xy);
    const Step<T> s1y = mk_step(g[3], g[1], is.y);
    const Step<T> s2x = mk_step(g[3], g[2], is.x);
    T best = fmadd(g0, g0, G.px + G.py);
    T e = face1(g0, s0x, G.ax, G.py);
    best = vmin<T>(best, (!MASKED || okx) ? e : INF);
    e = face1(g0, s0y, G.ay, G.px);
    best = vmin<T>(best, (!MASKED || oky) ? e : INF);
    const bool both = !MASKED || (okx && oky);
    e = face1(g0, s0xy, G.mxy, G.vxy);
    e = vmin<T>(e, face2(g0, s0x, G.ax, s1y, G.ay, T(0)));
    e = vmin<T>(e, face2(g0, s0y, G.ay, s2x, G.ax, T(0)));
    best = vmin<T>(best, both ? e : INF);
    return best;
}

// ---------------------------------------------------------------------------------------
// Work passes.
//
// Pass A (zero-key cells, all M nodes in grid order): the 2^d cells with key 0 surround
// every node, so every lane runs the same work and neighbouring lanes read neighbouring
// doses.  The 3^d dose neighbourhood is loaded once (all loads issued before the first
// use) and shared by the 2^d cells.  A node whose bound after these cells is <= the next
// key^2 is finished (the walk would break there); the others are queued for pass B.
//
// Pass B (tail): the queued nodes, sorted by the chosen key (the paper's DD sort:
// gamma0; or the bound after pass A), walk the table from the first non-zero key in
// wave lockstep.
//
// Guard pass (guarded precision): nodes that met an ill-conditioned tetrahedron in A or
// B are redone from the start with those tetrahedra projected in FP64.
// ---------------------------------------------------------------------------------------

// Per-block reduction of the counts, added into one of SUM_BINS partial slots (blocks
// spread over the slots, so no address sees more than a few hundred atomics).
// bins == nullptr: add straight into the map's scalars (`direct`).
__device__ __forceinline__ void block_sums(BlockSums* bins, uint32_t vb, uint32_t npass, uint32_t nborder,
                                           uint32_t nfp64, uint32_t ncells, uint32_t gm,
                                           Scalars* direct = nullptr) {
    __shared__ uint32_t s[5][SEARCH_THREADS / WAVE];
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        npass += (uint32_t)__shfl_xor((int)npass, o);
        nborder += (uint32_t)__shfl_xor((int)nborder, o);
        nfp64 += (uint32_t)__shfl_xor((int)nfp64, o);
        ncells += (uint32_t)__shfl_xor((int)ncells, o);
        gm = max(gm, (uint32_t)__shfl_xor((int)gm, o));
    }
    const int w = threadIdx.x / WAVE;
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        s[0][w] = npass;
        s[1][w] = nborder;
        s[2][w] = nfp64;
        s[3][w] = ncells;
        s[4][w] = gm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long p = 0, b = 0, f = 0, c = 0;
        uint32_t m = 0;
        for (int j = 0; j < SEARCH_THREADS / WAVE; ++j) {
            p += s[0][j];
            b += s[1][j];
            f += s[2][j];
            c += s[3][j];
            m = max(m, s[4][j]);
        }
        if (bins) {
            BlockSums* out = &bins[vb & (SUM_BINS - 1)];
            if (p) atomicAdd(&out->pass, p);
            if (b) atomicAdd(&out->border, b);
            if (f) atomicAdd(&out->fp64, f);
            if (c) atomicAdd(&out->cells, c);
            if (m) atomicMax(&out->maxg2, m);
        } else {
            if (p) atomicAdd(&direct->n_pass, p);
            if (b) atomicAdd(&direct->n_border, b);
            if (f) atomicAdd(&direct->n_fp64, f);
            if (c) atomicAdd(&direct->n_cells, c);
            if (m) atomicMax(&direct->maxg2_bits, m);
        }
    }
}

// Block-aggregated append to a device list: one atomic per block.  Returns the slot of
// this lane (valid where `want`).  All threads of the block must call it.
__device__ __forceinline__ uint32_t block_append(bool want, uint32_t* counter) {
    __shared__ uint32_t s_cnt[SEARCH_THREADS / WAVE];
    __shared__ uint32_t s_base;
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const unsigned long long bal = __ballot(want);
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    if (lane == 0) s_cnt[w] = (uint32_t)__popcll(bal);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0u;
        for (int j = 0; j < SEARCH_THREADS / WAVE; ++j) tot += s_cnt[j];
        s_base = tot ? atomicAdd(counter, tot) : 0u;
    }
    __syncthreads();
    uint32_t off = s_base;
    for (int j = 0; j < w; ++j) off += s_cnt[j];
    __syncthreads();   // s_cnt/s_base may be reused by the next call
    return off + (uint32_t)__popcll(bal & lt);
}

// n / d for n < 2^31 (the host prepares the multiplier; see make_fast_div).
__device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv& d) { return __umulhi(n, d.mul) >> d.shift; }

// Finished node: write gamma, update the per-lane counts.
__device__ __forceinline__ void finish_node(const SearchArgs& a, int node, float F, uint32_t& npass,
                                            uint32_t& nborder, uint32_t& gm) {
    const float gam = sqrtf(F);
    a.gamma[node] = gam;
    npass += gam <= 1.0f;
    nborder += fabsf(gam - 1.0f) <= 1e-5f;
    gm = max(gm, f2u(gam * gam));
}

// Learned radius.  gamma_hat = max(exp(y) - 0.01, 0) from the CNN output y of a tail item;
// the speculative walk takes the bound min(gamma^2, (f * gamma_hat)^2).  The same float
// expression serves the speculative walk and the fallback, so both see the same bound.
__device__ __forceinline__ float pred_gamma(const SearchArgs& a, uint32_t item) {
    return fmaxf(expf(a.yhat[item]) - 0.01f, 0.0f);
}
__device__ __forceinline__ float spec_bound2(const SearchArgs& a, uint32_t item) {
    const float r = a.spec_factor * pred_gamma(a, item);
    return r * r;
}
// Sort key of a queued tail node: gamma0^2 (DD sort) or the bound after the key-0 cells
// (non-negative floats: bit order = numeric order).  The predicted order's keys are
// written afterwards by the network at the tail nodes.
__device__ __forceinline__ uint32_t tail_sort_key(const SearchArgs& a, int node, float F0, float F) {
    (void)node;
    return a.tail_key == 1 ? f2u(F) : f2u(F0);
}
// First table row with key^2 >= r2 (rows are in ascending key order), at least `first`.
// Rows before it either were evaluated by the speculative walk or could not improve it.
__device__ __forceinline__ int resume_row(const TabEntry* tab, int n, int first, float r2) {
    int lo = first, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tab[mid].key2 < r2) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Full cells among the zero-key cells of a node (every one is evaluated for a tail node).
__device__ __forceinline__ uint32_t zero_cells(int DIM, int x, int y, int z, int nx, int ny, int nz) {
    const uint32_t cx = (x > 0) + (x + 1 < nx), cy = (y > 0) + (y + 1 < ny);
    const uint32_t cz = DIM == 3 ? (uint32_t)((z > 0) + (z + 1 < nz)) : 1u;
    return cx * cy * cz;
}

// End of a key-0 pass block (all its threads): a finished node's gamma, the block's counts,
// and the appends of its tail (with the words bound and key) and guard nodes.  The counts of a wave come from ballots (a node
// visits at most 27 cells), the waves' from one barrier, and only a block with tail or guard
// nodes waits for the atomics that give it its slots.  all_cells: the cells of tail nodes are counted
// here too (two grids).  (Two appends and a reduction of five
// counts by shuffles, with eight barriers between them, took 1.7 and 11 us longer in passes of 32
// and 180 us: 391 thousand nodes at 2.5 mm, 3.1 million at 1.25 mm.)
__device__ __forceinline__ void append_tail(const SearchArgs& a, uint32_t pos, int node, uint32_t bound, uint32_t key) {
    a.tail_node[pos] = (uint32_t)node;
    a.tail_f[pos] = bound;
    a.tail_key_arr[pos] = key;
    a.tail_pos[pos] = pos;
}
__device__ __forceinline__ void append_tail(const GridsArgs& a, uint32_t pos, int node, uint32_t bound, uint32_t) {
    a.tail_list[pos] = (uint32_t)node;
    a.tail_f[pos] = u2f(bound);
}
template <typename Args>
__device__ __forceinline__ void zero_epilogue(const Args& a, BlockSums* bins, uint32_t vb, bool live, int node,
                                              float F, uint32_t bound, uint32_t key, uint32_t cells, bool to_tail,
                                              bool to_guard, bool all_cells = false) {
    constexpr int WAVES = SEARCH_THREADS / WAVE;
    __shared__ uint32_t s_n[6][WAVES];   // tail, guard, pass, border, cells, max gamma^2
    __shared__ uint32_t s_base[2];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const bool done = live && !to_tail && !to_guard;
    const float gam = sqrtf(F);
    if (done) a.gamma[node] = gam;
    const unsigned long long tb = __ballot(to_tail), gb = __ballot(to_guard);
    const uint32_t npass = (uint32_t)__popcll(__ballot(done && gam <= 1.0f));
    const uint32_t nborder = (uint32_t)__popcll(__ballot(done && fabsf(gam - 1.0f) <= 1e-5f));
    cells = done || (all_cells && to_tail) ? cells : 0u;
    uint32_t ncells = 0u;
#pragma unroll
    for (int k = 0; k < 5; ++k) ncells += (uint32_t)__popcll(__ballot((cells >> k) & 1u)) << k;
    uint32_t gm = done ? f2u(gam * gam) : 0u;
    for (int o = WAVE / 2; o > 0; o >>= 1) gm = max(gm, (uint32_t)__shfl_xor((int)gm, o));
    if (lane == 0) {
        s_n[0][w] = (uint32_t)__popcll(tb);
        s_n[1][w] = (uint32_t)__popcll(gb);
        s_n[2][w] = npass;
        s_n[3][w] = nborder;
        s_n[4][w] = ncells;
        s_n[5][w] = gm;
    }
    __syncthreads();
    uint32_t tot[2] = {0u, 0u}, off[2] = {0u, 0u};
#pragma unroll
    for (int j = 0; j < WAVES; ++j)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t n = s_n[k][j];
            off[k] += j < w ? n : 0u;
            tot[k] += n;
        }
    if (threadIdx.x == 0) {
        if (tot[0]) s_base[0] = atomicAdd(&a.sc->n_tail, tot[0]);
        if (tot[1]) s_base[1] = atomicAdd(&a.sc->n_guard, tot[1]);
    }
    if (threadIdx.x == WAVE) {
        uint32_t t[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < WAVES; ++j) {
            t[0] += s_n[2][j];
            t[1] += s_n[3][j];
            t[2] += s_n[4][j];
            t[3] = max(t[3], s_n[5][j]);
        }
        BlockSums* out = &bins[vb & (SUM_BINS - 1)];
        if (t[0]) atomicAdd(&out->pass, (unsigned long long)t[0]);
        if (t[1]) atomicAdd(&out->border, (unsigned long long)t[1]);
        if (t[2]) atomicAdd(&out->cells, (unsigned long long)t[2]);
        if (t[3]) atomicMax(&out->maxg2, t[3]);
    }
    if (tot[0] + tot[1] == 0u) return;
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
    if (to_tail) append_tail(a, s_base[0] + off[0] + (uint32_t)__popcll(tb & lt), node, bound, key);
    if (to_guard) a.guard_list[s_base[1] + off[1] + (uint32_t)__popcll(gb & lt)] = (uint32_t)node;
}

// ---- pass A in 3D ------------------------------------------------------------------------
//
// A key-0 cell holds the node at one of its corners (bit i of V: the corner's side along axis
// i, x = 1, y = 2, z = 4), and of the 26 faces it owns only those whose chain steps onto that
// corner hold the node: 75 of the 208 of the eight cells.  For these the spatial constants are
// exact zeros and ones (mu = -1 for the blocks stepped before the node, 0 after it, no
// perpendicular part), so the near faces below are cell3's with the same roundings and
// without its constant terms.
//
// The other 133 faces ("far") keep a distance from the node.  A face that misses corner V has,
// at every point, t_j >= t_i for some axis i in V and j outside it (or, V = 7, some t_i = 0),
// so it lies at least at the distance from the node to the plane t_i = t_j,
// 1 / sqrt(1 / s_i^2 + 1 / s_j^2), or to t_i = 0 (ZeroGeo::far2), and its doses lie in the
// range of the cell's corners.  After the near faces a cell is needed only if that bound is
// below F, with the tail walk's margin of 2^-8 F; the needed cells of a wave (0.3 of 7 per
// node at 2.5 mm 3%/3mm, 0.7-1.9 at 1.25 mm) are queued in LDS and projected 64 at a time as
// in the walk of long tails.  Nodes at the grid's faces queue all of their cells instead.  The
// minimum has the same bits as over all 208 faces.
//
// Bound by VALU issue (1870 instructions of a wave against 3270 over all faces at 2.5 mm) and,
// at 391 thousand nodes, by the two rounds its 1528 blocks take: 40.0 -> 31.6 us there,
// 3.1 million nodes at 1.25 mm 259 -> 174 us (guarded).  Capped at 128 VGPRs for four waves per
// SIMD (uncapped, at 140, 1.07 and 1.13 times as long).

// Chain sums at a block stepped before the node (M = 1: mu = -1) or after it (M = 0: mu = 0).
template <int M, typename T>
__device__ __forceinline__ T near_n(T n, const Step<T>& s) {
#pragma clang fp contract(off)
    return M ? n + s.d : n;
}
template <int M, typename T>
__device__ __forceinline__ T near_t(const Step<T>& s, T L) {
#pragma clang fp contract(off)
    return M ? fmadd(-s.w, L, T(1)) : -(s.w * L);
}
template <int M1, typename T>
__device__ __forceinline__ T near1(T g0, const Step<T>& a) {
#pragma clang fp contract(off)
    const T N = near_n<M1>(g0, a);
    const T L = N * Num<T>::rcp(den_step(T(1), a));
    const T t1 = near_t<M1>(a, L);
    return (t1 >= T(0) && t1 <= T(1)) ? N * L : Num<T>::inf();
}
template <int M1, int M2, typename T>
__device__ __forceinline__ T near2(T g0, const Step<T>& a, const Step<T>& b) {
#pragma clang fp contract(off)
    const T N = near_n<M2>(near_n<M1>(g0, a), b);
    const T L = N * Num<T>::rcp(den_step(den_step(T(1), a), b));
    const T t1 = near_t<M1>(a, L), t2 = near_t<M2>(b, L);
    return (t1 <= T(1) && t1 >= t2 && t2 >= T(0)) ? N * L : Num<T>::inf();
}
template <int M1, int M2, int M3, typename T>
__device__ __forceinline__ T near3(T g0, const Step<T>& a, const Step<T>& b, const Step<T>& c) {
#pragma clang fp contract(off)
    const T N = near_n<M3>(near_n<M2>(near_n<M1>(g0, a), b), c);
    const T L = N * Num<T>::rcp(den3(a, b, c));
    const T t1 = near_t<M1>(a, L), t2 = near_t<M2>(b, L), t3 = near_t<M3>(c, L);
    return (t1 <= T(1) && t1 >= t2 && t2 >= t3 && t3 >= T(0)) ? N * L : Num<T>::inf();
}
template <int S, typename T>
__device__ __forceinline__ T inv_of(const InvS2<T>& is) {
    if constexpr (S == 1) return is.x;
    else if constexpr (S == 2) return is.y;
    else if constexpr (S == 4) return is.z;
    else if constexpr (S == 3) return is.xy;
    else if constexpr (S == 5) return is.xz;
    else if constexpr (S == 6) return is.yz;
    else return is.xyz;
}
// Step from vertex U of the cell along block S.
template <int U, int S, typename T>
__device__ __forceinline__ Step<T> near_step(const T* g, const InvS2<T>& is) {
    static_assert((U & S) == 0, "a chain steps away from its start");
    return mk_step(g[U | S], g[U], inv_of<S>(is));
}
// Smallest dist^2 over the near faces of the cell that holds the node at corner V (V = 0: but
// the node itself).  A, B, C: the axes, V = A, A | B, 7 or 0.
template <int V, int A, int B, int C, typename T>
__device__ __forceinline__ T near_faces(const T* g, const InvS2<T>& is) {
    const T g0 = g[0];
    if constexpr (V == A) {
        const Step<T> a = near_step<0, A>(g, is), ab = near_step<A, B>(g, is), ac = near_step<A, C>(g, is);
        T r = vmin<T>(near1<1>(g0, a), near2<1, 0>(g0, a, near_step<A, (B | C)>(g, is)));
        r = vmin<T>(r, vmin<T>(near2<1, 0>(g0, a, ab), near2<1, 0>(g0, a, ac)));
        return vmin<T>(r, vmin<T>(near3<1, 0, 0>(g0, a, ab, near_step<(A | B), C>(g, is)),
                                          near3<1, 0, 0>(g0, a, ac, near_step<(A | C), B>(g, is))));
    } else if constexpr (V == (A | B)) {
        const Step<T> a = near_step<0, A>(g, is), b = near_step<0, B>(g, is), e = near_step<0, (A | B)>(g, is);
        const Step<T> ab = near_step<A, B>(g, is), ba = near_step<B, A>(g, is), c = near_step<(A | B), C>(g, is);
        T r = vmin<T>(near1<1>(g0, e), near2<1, 0>(g0, e, c));
        r = vmin<T>(r, vmin<T>(near2<1, 1>(g0, a, ab), near2<1, 1>(g0, b, ba)));
        return vmin<T>(r, vmin<T>(near3<1, 1, 0>(g0, a, ab, c), near3<1, 1, 0>(g0, b, ba, c)));
    } else {
        constexpr int M = V == 7 ? 1 : 0;
        const Step<T> x = near_step<0, 1>(g, is), y = near_step<0, 2>(g, is), z = near_step<0, 4>(g, is);
        const Step<T> xy = near_step<0, 3>(g, is), xz = near_step<0, 5>(g, is), yz = near_step<0, 6>(g, is);
        const Step<T> x_y = near_step<1, 2>(g, is), x_z = near_step<1, 4>(g, is), y_x = near_step<2, 1>(g, is);
        const Step<T> y_z = near_step<2, 4>(g, is), z_x = near_step<4, 1>(g, is), z_y = near_step<4, 2>(g, is);
        const Step<T> xy_z = near_step<3, 4>(g, is), xz_y = near_step<5, 2>(g, is), yz_x = near_step<6, 1>(g, is);
        T r = near1<M>(g0, near_step<0, 7>(g, is));
        r = vmin<T>(r, vmin<T>(near2<M, M>(g0, x, near_step<1, 6>(g, is)), near2<M, M>(g0, yz, yz_x)));
        r = vmin<T>(r, vmin<T>(near2<M, M>(g0, y, near_step<2, 5>(g, is)), near2<M, M>(g0, xz, xz_y)));
        r = vmin<T>(r, vmin<T>(near2<M, M>(g0, z, near_step<4, 3>(g, is)), near2<M, M>(g0, xy, xy_z)));
        r = vmin<T>(r, vmin<T>(near3<M, M, M>(g0, x, x_y, xy_z), near3<M, M, M>(g0, x, x_z, xz_y)));
        r = vmin<T>(r, vmin<T>(near3<M, M, M>(g0, y, y_x, xy_z), near3<M, M, M>(g0, y, y_z, yz_x)));
        r = vmin<T>(r, vmin<T>(near3<M, M, M>(g0, z, z_x, xz_y), near3<M, M, M>(g0, z, z_y, yz_x)));
        if constexpr (V == 0) {
            r = vmin<T>(r, vmin<T>(near1<0>(g0, x), vmin<T>(near1<0>(g0, y), near1<0>(g0, z))));
            r = vmin<T>(r, vmin<T>(near1<0>(g0, xy), vmin<T>(near1<0>(g0, xz), near1<0>(g0, yz))));
            r = vmin<T>(r, vmin<T>(near2<0, 0>(g0, x, x_y), near2<0, 0>(g0, y, y_x)));
            r = vmin<T>(r, vmin<T>(near2<0, 0>(g0, x, x_z), near2<0, 0>(g0, z, z_x)));
            r = vmin<T>(r, vmin<T>(near2<0, 0>(g0, y, y_z), near2<0, 0>(g0, z, z_y)));
        }
        return r;
    }
}
// Corners of key-0 cell c = 4 (az + 1) + 2 (ay + 1) + (ax + 1) from the 3 x 3 x 3 neighbourhood.
template <int C, typename T>
__device__ __forceinline__ void zero_corners(const T* g27, T* g) {
#pragma unroll
    for (int b = 0; b < 8; ++b)
        g[b] = g27[((C >> 2) + (b >> 2)) * 9 + (((C >> 1) & 1) + ((b >> 1) & 1)) * 3 + (C & 1) + (b & 1)];
}
template <int C, int V, int A, int B, int CC, typename T>
__device__ __forceinline__ T zero_near(const T* g27, const InvS2<T>& is) {
    static_assert((C ^ 7) == V, "the node's corner");
    T g[8];
    zero_corners<C>(g27, g);
    return near_faces<V, A, B, CC>(g, is);
}

// LDS of the pass: one block of it for every mode of a kernel.  A batch's kernels hold several, and
// with arrays of their own per mode few blocks fit a compute unit: the key-0 phase of 64 mixed
// pairs took 4.24 ms and the tail phase 4.82; they take 3.5 and 1.67.
template <bool FP64>
struct ZeroLds {
    static constexpr int WAVES = SEARCH_THREADS / WAVE;
    float g[WAVES][27][WAVE];          // neighbourhoods of the wave's nodes, normalised (FP64: doses)
    typename std::conditional<FP64, unsigned long long, uint32_t>::type f[WAVES][WAVE];   // their F (non-negative bits)
    float dr[FP64 ? WAVES : 1][WAVE];
    double inv[FP64 ? WAVES : 1][WAVE];
    uint16_t item[WAVES][8 * WAVE];    // queued cells: node's lane | cell << 6
    uint8_t up[WAVES][WAVE];           // bit i: the grid goes on past the node along axis i
    TabEntry zero[8];
};
template <bool FP64>
__device__ __forceinline__ ZeroLds<FP64>& zero_lds() {
    __shared__ ZeroLds<FP64> s;
    return s;
}

// MODE 0: FP32; MODE 1: FP32 and flag ill-conditioned tetrahedra; MODE 3: FP64 (a tail node's
// bound is left as a double in tail_f and tail_key_arr).  vb: the block's index in the node list (256 nodes each).
template <int MODE>
__device__ __forceinline__ void zero3_body(const SearchArgs& a, const ZeroGeo& zg, BlockSums* sums, uint32_t vb) {
    constexpr int GMODE = MODE == 1 ? 1 : 0;
    using T = typename std::conditional<MODE == 3, double, float>::type;
    using U = typename std::conditional<MODE == 3, unsigned long long, uint32_t>::type;
    ZeroLds<MODE == 3>& lds = zero_lds<MODE == 3>();
    auto& s_g = lds.g;
    auto& s_f = lds.f;
    auto& s_dr = lds.dr;
    auto& s_inv = lds.inv;
    auto& s_item = lds.item;
    auto& s_up = lds.up;
    auto& s_zero = lds.zero;
    const uint32_t M = a.sc->n_masked;
    if (vb * SEARCH_THREADS >= M) {   // grids are sized for every grid node; M is on the device
        return;
    }
    if (threadIdx.x < 8) s_zero[threadIdx.x] = zg.row[threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    const uint32_t i = vb * SEARCH_THREADS + threadIdx.x;
    const bool live = i < M;
    const int nx = a.nx, ny = a.ny, nz = a.nz, sxy = nx * ny;
    const int node = live ? (int)a.nodes[i] : 0;
    const uint32_t yz = fast_div((uint32_t)node, a.div_nx);
    const int z = (int)fast_div(yz, a.div_ny), y = (int)yz - z * ny, x = node - (int)yz * nx;
    const float dr = a.ref[node];
    T inv_dd;
    if constexpr (MODE == 3) inv_dd = fp64_inv_dd(a, dr);
    else inv_dd = node_inv_dd(dr, a.sc->inv_dd, a.dd, a.local);
    // neighbourhood offsets, clamped at the grid faces (clamped values feed only cells
    // that do not exist or faces that are masked out)
    const int oxm = x > 0 ? -1 : 0, oxp = x + 1 < nx ? 1 : 0;
    const int oym = y > 0 ? -nx : 0, oyp = y + 1 < ny ? nx : 0;
    const int ozm = z > 0 ? -sxy : 0, ozp = z + 1 < nz ? sxy : 0;
    const int ox[3] = {oxm, 0, oxp}, oy[3] = {oym, 0, oyp}, oz[3] = {ozm, 0, ozp};
    T g27[27];
    {
        float v[27];
#pragma unroll
        for (int k = 0; k < 27; ++k) v[k] = a.ev[node + oz[k / 9] + oy[(k / 3) % 3] + ox[k % 3]];
        if constexpr (MODE == 3) {
#pragma unroll
            for (int k = 0; k < 27; ++k) s_g[wv][k][lane] = v[k];
            s_dr[wv][lane] = dr;
            s_inv[wv][lane] = inv_dd;
        }
#pragma unroll
        for (int k = 0; k < 27; ++k) g27[k] = dose_norm<T>((T)v[k], (T)dr, inv_dd);
    }
    const T F0 = live ? g27[13] * g27[13] : T(0);   // gamma0^2

    const InvS2<T> is = inv_s2_for<T>(a);
    // where the grid goes on from the node: bits 0..2 up along x, y, z, bits 3..5 down (all that
    // is kept of its place: with offsets and coordinates six registers spilled, 186 us at
    // 192x256x256 against 174 now)
    const uint32_t on6 = (oxp ? 1u : 0u) | (oyp ? 2u : 0u) | (ozp ? 4u : 0u) | (oxm ? 8u : 0u) | (oym ? 16u : 0u) | (ozm ? 32u : 0u);
    const bool bnd = on6 != 63u;
    // whether key-0 cell c = 4 (az + 1) + 2 (ay + 1) + (ax + 1) exists, and exists whole
    auto there_of = [&](int c) { return (((on6 >> 3) | (uint32_t)c) & 7u) == 7u; };
    auto whole_of = [&](int c) { return ((on6 | ~(uint32_t)c) & 7u) == 7u; };
    const bool open = live && F0 > T(0);   // a node of dose difference 0 visits no cell
    T F = F0;
    {
        T r = zero_near<7, 0, 1, 2, 4>(g27, is);
        r = vmin<T>(r, zero_near<6, 1, 1, 2, 4>(g27, is));
        r = vmin<T>(r, zero_near<5, 2, 2, 1, 4>(g27, is));
        r = vmin<T>(r, zero_near<3, 4, 4, 1, 2>(g27, is));
        r = vmin<T>(r, zero_near<4, 3, 1, 2, 4>(g27, is));
        r = vmin<T>(r, zero_near<2, 5, 1, 4, 2>(g27, is));
        r = vmin<T>(r, zero_near<1, 6, 2, 4, 1>(g27, is));
        r = vmin<T>(r, zero_near<0, 7, 1, 2, 4>(g27, is));
        F = open && !bnd ? vmin<T>(F, r) : F;
    }
    // a neighbourhood whose doses span less than this holds no ill-conditioned tetrahedron
    bool suspect = false;
    if constexpr (MODE == 1) {
        T lo = g27[0], hi = g27[0];
#pragma unroll
        for (int k = 1; k < 27; ++k) {
            lo = vmin<T>(lo, g27[k]);
            hi = vmax<T>(hi, g27[k]);
        }
        suspect = open && !((hi - lo) * (hi - lo) < a.ill_span2);
    }

    // the cells with far faces that can lower F, or (at the grid's faces) every cell there is
    uint32_t q = 0;
    uint16_t* item = s_item[wv];
    auto push = [&](bool want, int c) {
        const unsigned long long mask = __ballot(want);
        if (want)
            item[q + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] =
                (uint16_t)(lane | (c << 6));
        q += (uint32_t)__popcll(mask);
    };
    const T Fm = F + F * T(0x1p-8);
    const bool edge = open && bnd, inner = open && !bnd;
    if (__ballot(edge || (inner && (T)zg.far2_min < Fm)) != 0ull) {
        // corner ranges of the eight cells, pairs along x, then y, then z
        T lo[18], hi[18];
#pragma unroll
        for (int k = 0; k < 18; ++k) {
            const int r = k >> 1, p = 3 * r + (k & 1);
            lo[k] = vmin<T>(g27[p], g27[p + 1]);
            hi[k] = vmax<T>(g27[p], g27[p + 1]);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int k = ((c >> 2) * 3 + ((c >> 1) & 1)) * 2 + (c & 1);   // pair (z, y, x) of the cell
            const T l = vmin<T>(vmin<T>(lo[k], lo[k + 2]), vmin<T>(lo[k + 6], lo[k + 8]));
            const T h = vmax<T>(vmax<T>(hi[k], hi[k + 2]), vmax<T>(hi[k + 6], hi[k + 8]));
            const T m = vmax<T>(vmax<T>(l, -h), T(0));
            const bool there = there_of(c);
            push((inner && c != 7 && fmadd(m, m, (T)zg.far2[c]) < Fm) || (edge && there), c);
        }
    }
    bool redo = suspect;
    if (q != 0u || __ballot(redo) != 0ull) {
        if constexpr (MODE != 3) {
#pragma unroll
            for (int k = 0; k < 27; ++k) s_g[wv][k][lane] = g27[k];
        }
        s_f[wv][lane] = __builtin_bit_cast(U, F);
        s_up[wv][lane] = (uint8_t)(on6 & 7u);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    uint32_t n_fp64 = 0;
    GuardCtx gc{};
    bool dummy_ill = false;
    // corner doses of cell c of the node of lane nl
    auto cell_doses = [&](int nl, int c, T* g) {
        const float(*gn)[WAVE] = s_g[wv] + (((c >> 2) * 3 + ((c >> 1) & 1)) * 3 + (c & 1));
#pragma unroll
        for (int b = 0; b < 8; ++b) g[b] = gn[(b >> 2) * 9 + ((b >> 1) & 1) * 3 + (b & 1)][nl];
    };
    // its dist^2, all faces it owns
    auto cell_of = [&](int nl, int c, bool mask) -> T {
        T g[8];
        cell_doses(nl, c, g);
        Geo<T> G;
        if constexpr (MODE == 3) {
            const T dn = s_dr[wv][nl], in = s_inv[wv][nl];
#pragma unroll
            for (int b = 0; b < 8; ++b) g[b] = dose_norm<T>(g[b], dn, in);
            G = geo_fp64((c & 1) - 1, ((c >> 1) & 1) - 1, (c >> 2) - 1, a.sx * a.sx, a.sy * a.sy, a.sz * a.sz);
        } else {
            G = geo_from_row(s_zero[c]);
        }
        const uint32_t up = s_up[wv][nl] | ~(uint32_t)c;   // a cell at -1 reaches back to the node
        if (mask)
            return cell3<T, true, 0>(g, G, is, up & 1u, up & 2u, up & 4u, (T)a.den_guard, gc, n_fp64, dummy_ill);
        return cell3<T, false, 0>(g, G, is, true, true, true, (T)a.den_guard, gc, n_fp64, dummy_ill);
    };
    bool ill = false;
    if (q != 0u) {
#pragma unroll 1
        for (uint32_t h = 0; h < q; h += WAVE) {
            const bool on = h + lane < q;
            const uint32_t it = on ? item[h + lane] : 0u;
            const int nl = (int)(it & 63u), c = (int)(it >> 6);
            const bool whole = ((s_up[wv][nl] | ~(uint32_t)c) & 7u) == 7u;
            const bool mask = __ballot(on && !whole) != 0ull;
            if (on) {
                const T v = cell_of(nl, c, mask);
                atomicMin(&s_f[wv][nl], __builtin_bit_cast(U, v));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        F = __builtin_bit_cast(T, s_f[wv][lane]);
    }
    // the whole cells around the node: (goes on up) + (goes on down) per axis, multiplied
    const uint32_t both = on6 & (on6 >> 3), one = (on6 | (on6 >> 3)) & 7u;
    uint32_t cells = open && one == 7u ? 1u << __popc(both & 7u) : 0u;
    // rare: the tetrahedra of a steep neighbourhood's whole cells are judged (their denominators
    // only: projecting the cells again for it, the pass took 58 us at 96x128x128 with the
    // threshold at 100, where every neighbourhood is steep; this takes 38, and 33 where none is),
    // and a node whose F fell to 0 counts the cells up to there, cell by cell in table order
    const bool zero = open && F == T(0);
    if (__ballot(redo || zero) != 0ull) {
        if (q == 0u && __ballot(redo) == 0ull) {
            if constexpr (MODE != 3) {
#pragma unroll
                for (int k = 0; k < 27; ++k) s_g[wv][k][lane] = g27[k];
            }
            s_up[wv][lane] = (uint8_t)(on6 & 7u);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if constexpr (GMODE == 1) {
            if (redo) {
#pragma unroll 1
                for (int c = 0; c < 8 && !ill; ++c) {
                    if (!there_of(c) || !whole_of(c)) continue;
                    T g[8];
                    cell_doses(lane, c, g);
                    ill = tets_ill(g, is, a.den_guard);
                }
            }
        }
        if (zero) {
            F = F0;
            cells = 0u;
#pragma unroll 1
            for (int c = 0; c < 8; ++c) {
                if (!there_of(c)) continue;
                cells += F > T(0) && whole_of(c) ? 1u : 0u;
                F = vmin<T>(F, cell_of(lane, c, true));
            }
        }
    }
    const bool to_guard = MODE == 1 && ill && open;
    const bool to_tail = live && !to_guard && F > (T)a.k1;
    if constexpr (MODE == 3) {
        const unsigned long long fb = __builtin_bit_cast(unsigned long long, F);
        zero_epilogue(a, sums, vb, live, node, (float)F, (uint32_t)fb, (uint32_t)(fb >> 32), cells, to_tail, false);
    } else {
        zero_epilogue(a, sums, vb, live, node, F, f2u(F), tail_sort_key(a, node, F0, F), cells, to_tail, to_guard);
    }
}

__global__ __launch_bounds__(SEARCH_THREADS) void k_zero3_fp64(SearchArgs a, ZeroGeo zg, BlockSums* sums) {
    zero3_body<3>(a, zg, sums, blockIdx.x);
}

template <int MODE>
__global__ __launch_bounds__(SEARCH_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_zero3(SearchArgs a, ZeroGeo zg, BlockSums* sums) {
    zero3_body<MODE>(a, zg, sums, blockIdx.x);
}

// Pass A in 3D with Ju et al.'s recursion (projection = 1): one lane per node, the recursion
// in interior cells, every owned face in the cells of a wave that meets a grid face.
template <int MODE>
__device__ __forceinline__ void zero3_ju_body(const SearchArgs& a, const ZeroGeo& zg, BlockSums* sums, uint32_t vb) {
    constexpr int GMODE = MODE == 1 ? 1 : 0;
    const uint32_t M = a.sc->n_masked;
    if (vb * SEARCH_THREADS >= M) {   // grids are sized for every grid node; M is on the device
        return;
    }
    const uint32_t i = vb * SEARCH_THREADS + threadIdx.x;
    const bool live = i < M;
    const int nx = a.nx, ny = a.ny, nz = a.nz, sxy = nx * ny;
    const int node = live ? (int)a.nodes[i] : 0;
    const int x = node % nx, y = (node / nx) % ny, z = node / sxy;
    const float dr = a.ref[node];
    const float inv_dd = node_inv_dd(dr, a.sc->inv_dd, a.dd, a.local);
    const float F0 = live ? gamma0_sq(a.ev[node], dr, inv_dd) : 0.0f;
    // neighbourhood offsets, clamped at the grid faces (clamped values feed only cells
    // that do not exist or faces that are masked out)
    const int oxm = x > 0 ? -1 : 0, oxp = x + 1 < nx ? 1 : 0;
    const int oym = y > 0 ? -nx : 0, oyp = y + 1 < ny ? nx : 0;
    const int ozm = z > 0 ? -sxy : 0, ozp = z + 1 < nz ? sxy : 0;
    const int ox[3] = {oxm, 0, oxp}, oy[3] = {oym, 0, oyp}, oz[3] = {ozm, 0, ozp};
    float g27[27];
#pragma unroll
    for (int k = 0; k < 27; ++k) g27[k] = a.ev[node + oz[k / 9] + oy[(k / 3) % 3] + ox[k % 3]];
#pragma unroll
    for (int k = 0; k < 27; ++k) g27[k] = (g27[k] - dr) * inv_dd;

    const InvS2<float> is = inv_s2_of(a);
    const bool bnd = x == 0 || x + 1 == nx || y == 0 || y + 1 == ny || z == 0 || z + 1 == nz;
    const bool wave_masked = __ballot(live && bnd) != 0ull;
    float F = F0;
    uint32_t cells = 0, n_fp64 = 0;
    bool ill = false;
    GuardCtx gc{};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        // table order of the zero-key cells: (az, ay, ax) in {-1,0}^3, lexicographic
        const int az = (c >> 2) - 1, ay = ((c >> 1) & 1) - 1, ax = (c & 1) - 1;
        float g[8];
#pragma unroll
        for (int b = 0; b < 8; ++b)
            g[b] = g27[(az + 1 + ((b >> 2) & 1)) * 9 + (ay + 1 + ((b >> 1) & 1)) * 3 + (ax + 1 + (b & 1))];
        const Geo<float> G = geo_from_row(zg.row[c]);
        float v;
        if (wave_masked) {
            const bool exists = (ax == 0 || x > 0) && (ay == 0 || y > 0) && (az == 0 || z > 0);
            const bool okx = ax < 0 || x + 1 < nx, oky = ay < 0 || y + 1 < ny, okz = az < 0 || z + 1 < nz;
            v = cell3<float, true, GMODE>(g, G, is, okx, oky, okz, a.den_guard, gc, n_fp64, ill);
            v = exists ? v : Num<float>::inf();
            cells += (F > 0.0f && exists && okx && oky && okz) ? 1u : 0u;
        } else {
            v = cell3_ju<GMODE>(g, G, is, a.s2x, a.s2y, a.s2z, a.den_guard, ill);
            cells += F > 0.0f ? 1u : 0u;
        }
        F = F0 > 0.0f ? vmin<float>(F, v) : F;
    }
    ill = ill && live && F0 > 0.0f;
    const bool to_guard = MODE == 1 && ill;
    const bool to_tail = live && !to_guard && F > a.k1;
    uint32_t npass = 0, nborder = 0, gm = 0, ncells = 0;
    if (live && !to_guard && !to_tail) {
        finish_node(a, node, F, npass, nborder, gm);
        ncells = cells;
    }
    // queue the tail (one atomic per block), then the guard list
    const uint32_t pos = block_append(to_tail, &a.sc->n_tail);
    if (to_tail) {
        a.tail_node[pos] = (uint32_t)node;
        a.tail_f[pos] = f2u(F);
        a.tail_key_arr[pos] = tail_sort_key(a, node, F0, F);
        a.tail_pos[pos] = pos;
    }
    if (MODE == 1) {
        const uint32_t gpos = block_append(to_guard, &a.sc->n_guard);
        if (to_guard) a.guard_list[gpos] = (uint32_t)node;
    }
    block_sums(sums, vb, npass, nborder, 0u, ncells, gm);
}

template <int MODE>
__global__ __launch_bounds__(SEARCH_THREADS) void k_zero3_ju(SearchArgs a, ZeroGeo zg, BlockSums* sums) {
    zero3_ju_body<MODE>(a, zg, sums, blockIdx.x);
}

// Pass A in 2D (4 zero-key cells, 3x3 neighbourhood).
__device__ __forceinline__ void zero2_body(const SearchArgs& a, const ZeroGeo& zg, BlockSums* sums, uint32_t vb) {
    const uint32_t M = a.sc->n_masked;
    if (vb * SEARCH_THREADS >= M) {
        return;
    }
    const uint32_t i = vb * SEARCH_THREADS + threadIdx.x;
    const bool live = i < M;
    const int nx = a.nx, ny = a.ny;
    const int node = live ? (int)a.nodes[i] : 0;
    const int x = node % nx, y = node / nx;
    const float dr = a.ref[node];
    const float inv_dd = node_inv_dd(dr, a.sc->inv_dd, a.dd, a.local);
    const float F0 = live ? gamma0_sq(a.ev[node], dr, inv_dd) : 0.0f;
    const int ox[3] = {x > 0 ? -1 : 0, 0, x + 1 < nx ? 1 : 0};
    const int oy[3] = {y > 0 ? -nx : 0, 0, y + 1 < ny ? nx : 0};
    float g9[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) g9[k] = a.ev[node + oy[k / 3] + ox[k % 3]];
#pragma unroll
    for (int k = 0; k < 9; ++k) g9[k] = (g9[k] - dr) * inv_dd;
    const InvS2<float> is = inv_s2_of(a);
    const bool bnd = x == 0 || x + 1 == nx || y == 0 || y + 1 == ny;
    const bool wave_masked = __ballot(live && bnd) != 0ull;
    float F = F0;
    uint32_t cells = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int ay = (c >> 1) - 1, ax = (c & 1) - 1;
        float g[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) g[b] = g9[(ay + 1 + ((b >> 1) & 1)) * 3 + (ax + 1 + (b & 1))];
        const Geo<float> G = geo_from_row(zg.row[c]);
        float v;
        if (wave_masked) {
            const bool exists = (ax == 0 || x > 0) && (ay == 0 || y > 0);
            const bool okx = ax < 0 || x + 1 < nx, oky = ay < 0 || y + 1 < ny;
            v = cell2<float, true>(g, G, is, okx, oky);
            v = exists ? v : Num<float>::inf();
            cells += (F > 0.0f && exists && okx && oky) ? 1u : 0u;
        } else {
            v = cell2<float, false>(g, G, is, true, true);
            cells += F > 0.0f ? 1u : 0u;
        }
        F = F0 > 0.0f ? vmin<float>(F, v) : F;
    }
    const bool to_tail = live && F > a.k1;
    uint32_t npass = 0, nborder = 0, gm = 0, ncells = 0;
    if (live && !to_tail) {
        finish_node(a, node, F, npass, nborder, gm);
        ncells = cells;
    }
    const uint32_t pos = block_append(to_tail, &a.sc->n_tail);
    if (to_tail) {
        a.tail_node[pos] = (uint32_t)node;
        a.tail_f[pos] = f2u(F);
        a.tail_key_arr[pos] = tail_sort_key(a, node, F0, F);
        a.tail_pos[pos] = pos;
    }
    block_sums(sums, vb, npass, nborder, 0u, ncells, gm);
}

template <int MODE>
__global__ __launch_bounds__(SEARCH_THREADS) void k_zero2(SearchArgs a, ZeroGeo zg, BlockSums* sums) {
    zero2_body(a, zg, sums, blockIdx.x);
    (void)MODE;
}

// Pass A with one lane per cell: the 2^d lanes of a group share one node (grid order) and
// each takes one of its zero-key cells (table rows 0 .. 2^d-1), then the group takes the
// minimum with shuffles.  Lighter waves than one lane per node (more of them resident, no
// wave-quantisation tail).  Grid-stride over the nodes; MODE 0: FP32, 1: FP32 + flag.
template <int DIM, int MODE>
__global__ __launch_bounds__(SEARCH_THREADS) void k_zero_group(SearchArgs a, ZeroGeo zg, BlockSums* sums) {
    constexpr int G = 1 << DIM;
    constexpr int GROUPS = SEARCH_THREADS / G;
    constexpr int GMODE = (DIM == 3 && MODE == 1) ? 1 : 0;
    const uint32_t M = a.sc->n_masked;
    const int gl = threadIdx.x % G;
    const int nx = a.nx, ny = a.ny, nz = a.nz, sxy = nx * ny;
    const float inv_dd_g = a.sc->inv_dd;
    const InvS2<float> is = inv_s2_of(a);
    const TabEntry row = zg.row[gl];            // this lane's zero-key cell
    const Geo<float> Gm = geo_from_row(row);
    GuardCtx gc{};
    uint32_t dummy_fp64 = 0, cells = 0, gm = 0, npass = 0, nborder = 0;

    for (uint32_t base = blockIdx.x * GROUPS; base < M; base += gridDim.x * GROUPS) {
        const uint32_t i = base + threadIdx.x / G;
        const bool live = i < M;
        const int node = live ? (int)a.nodes[i] : 0;
        const int x = node % nx, y = (node / nx) % ny, z = DIM == 3 ? node / sxy : 0;
        const float dr = a.ref[node];
        const float inv_dd = node_inv_dd(dr, inv_dd_g, a.dd, a.local);
        const float F0 = live ? gamma0_sq(a.ev[node], dr, inv_dd) : 0.0f;
        const int qx = x + row.ax, qy = y + row.ay, qz = z + row.az;
        const bool cin = (unsigned)qx < (unsigned)nx && (unsigned)qy < (unsigned)ny &&
                         (DIM == 2 || (unsigned)qz < (unsigned)nz);
        const bool okx = qx + 1 < nx, oky = qy + 1 < ny, okz = DIM == 2 || qz + 1 < nz;
        const bool work = F0 > 0.0f && cin;
        const bool edge = !(okx && oky && okz);
        const bool wave_masked = __ballot(work && edge) != 0ull;
        float c = Num<float>::inf();
        bool ill = false;
        if (work) {
            const int b0 = (DIM == 3 ? qz * sxy : 0) + qy * nx + qx;
            const int ox = okx ? 1 : 0, oy = oky ? nx : 0, oz = (DIM == 3 && okz) ? sxy : 0;
            if constexpr (DIM == 3) {
                float g[8];
                g[0] = a.ev[b0];
                g[1] = a.ev[b0 + ox];
                g[2] = a.ev[b0 + oy];
                g[3] = a.ev[b0 + oy + ox];
                g[4] = a.ev[b0 + oz];
                g[5] = a.ev[b0 + oz + ox];
                g[6] = a.ev[b0 + oz + oy];
                g[7] = a.ev[b0 + oz + oy + ox];
#pragma unroll
                for (int b = 0; b < 8; ++b) g[b] = (g[b] - dr) * inv_dd;
                if (wave_masked)
                    c = cell3<float, true, GMODE>(g, Gm, is, okx, oky, okz, a.den_guard, gc, dummy_fp64, ill);
                else
                    c = cell3<float, false, GMODE>(g, Gm, is, true, true, true, a.den_guard, gc, dummy_fp64, ill);
            } else {
                float g[4];
                g[0] = a.ev[b0];
                g[1] = a.ev[b0 + ox];
                g[2] = a.ev[b0 + oy];
                g[3] = a.ev[b0 + oy + ox];
#pragma unroll
                for (int b = 0; b < 4; ++b) g[b] = (g[b] - dr) * inv_dd;
                if (wave_masked)
                    c = cell2<float, true>(g, Gm, is, okx, oky);
                else
                    c = cell2<float, false>(g, Gm, is, true, true);
            }
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
            c = vmin<float>(c, __shfl_xor(c, o));
            ill = (__shfl_xor((int)ill, o) != 0) || ill;
        }
        // every lane of the group now holds the same F0, minimum and flag
        const float F = vmin<float>(F0, c);
        const bool node_guard = MODE == 1 && live && ill;
        const bool node_tail = live && !node_guard && F > a.k1;
        // cells are counted by the pass that finishes the node
        if (live && !node_guard && !node_tail && work && !edge) ++cells;
        const bool leader = gl == 0;
        const bool to_guard = leader && node_guard;
        const bool to_tail = leader && node_tail;
        if (leader && live && !node_guard && !node_tail) finish_node(a, node, F, npass, nborder, gm);
        const uint32_t pos = block_append(to_tail, &a.sc->n_tail);
        if (to_tail) {
            a.tail_node[pos] = (uint32_t)node;
            a.tail_f[pos] = f2u(F);
            a.tail_key_arr[pos] = tail_sort_key(a, node, F0, F);
            a.tail_pos[pos] = pos;
        }
        if (MODE == 1) {
            const uint32_t gpos = block_append(to_guard, &a.sc->n_guard);
            if (to_guard) a.guard_list[gpos] = (uint32_t)node;
        }
    }
    block_sums(sums, blockIdx.x, npass, nborder, 0u, cells, gm);
}

// The walk.  TAIL: items are tail positions, the walk starts at row `first` with the bound
// left by pass A; otherwise items are node indices and the walk starts at row 0 with
// gamma0.  MODE 0: FP32; 1: FP32 + flag; 2: FP32 with FP64 re-projection; 3: FP64.
// spec (TAIL only): 0 plain; 1 speculative (bound min(gamma^2, (f gamma_hat)^2); a node
// whose gamma^2 stays above (f gamma_hat)^2 is queued on the fallback list instead of
// finished); 2 fallback (the plain walk from the first row at or beyond f gamma_hat).
// vb / vgrid: the block's index and the number of blocks striding over the list.
template <int DIM, int MODE, bool TAIL>
__device__ __forceinline__ void walk_body(const SearchArgs& a, const TabEntry* __restrict__ tab,
                                          const uint32_t* __restrict__ order, const uint32_t* __restrict__ count,
                                          int first, int spec, BlockSums* sums, uint32_t vb, uint32_t vgrid) {
    using T = typename std::conditional<MODE == 3, double, float>::type;
    constexpr int GMODE = DIM == 3 ? (MODE == 1 ? 1 : (MODE == 2 ? 2 : 0)) : 0;
    const uint32_t M = *count;
    const int lane = threadIdx.x & (WAVE - 1);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int sxy = nx * ny;
    const float inv_dd_g = a.sc->inv_dd;
    const double dmax = (double)ord_to_float(a.sc->dmax_ord);
    const InvS2<T> is = inv_s2<T>(MODE == 3 ? (T)(a.sx * a.sx) : (T)a.s2x,
                                  MODE == 3 ? (T)(a.sy * a.sy) : (T)a.s2y,
                                  DIM == 3 ? (MODE == 3 ? (T)(a.sz * a.sz) : (T)a.s2z) : T(0));
    const double sx2d = a.sx * a.sx, sy2d = a.sy * a.sy, sz2d = a.sz * a.sz;
    const uint32_t stride = vgrid * SEARCH_THREADS;
    uint32_t cells = 0, n_fp64 = 0, gm = 0, npass = 0, nborder = 0;

    // the loop bound is uniform per wave, so every lane reaches the block-wide calls below
    const uint32_t wave0 = vb * SEARCH_THREADS + (threadIdx.x & ~(WAVE - 1));
    const uint32_t iters = wave0 < M ? (M - wave0 + stride - 1) / stride : 0u;
    uint32_t it_max = iters;
    // block-uniform trip count (all waves of a block take part in block_append)
    {
        __shared__ uint32_t s_it[SEARCH_THREADS / WAVE];
        if (lane == 0) s_it[threadIdx.x / WAVE] = iters;
        __syncthreads();
        it_max = 0u;
        for (int j = 0; j < SEARCH_THREADS / WAVE; ++j) it_max = max(it_max, s_it[j]);
        __syncthreads();
    }
    for (uint32_t it = 0; it < it_max; ++it) {
        const uint32_t i = wave0 + it * stride + lane;
        const bool live = i < M;
        const uint32_t item = live ? order[i] : 0u;
        const int node = TAIL ? (live ? (int)a.tail_node[item] : 0) : (int)item;
        const int x = node % nx;
        const int y = (node / nx) % ny;
        const int z = DIM == 3 ? node / sxy : 0;
        const float dr = a.ref[node];
        const float inv_dd = node_inv_dd(dr, inv_dd_g, a.dd, a.local);
        const double inv_dd64 = a.local ? 1.0 / (a.dd64 * (double)dr) : 1.0 / (a.dd64 * dmax);
        T F;
        if constexpr (MODE == 3) {
            const double g0 = ((double)a.ev[node] - (double)dr) * inv_dd64;
            F = g0 * g0;
        } else {
            F = TAIL ? u2f(live ? a.tail_f[item] : 0u) : gamma0_sq(a.ev[node], dr, inv_dd);
        }
        if (!live) F = T(0);
        const T invdd = MODE == 3 ? (T)inv_dd64 : (T)inv_dd;
        const T drT = (T)dr;
        uint32_t lane_cells = 0, lane_fp64 = 0;
        bool ill = false;
        // learned radius: the speculative bound, and the fallback's first row
        const float r2s = (TAIL && spec && live) ? spec_bound2(a, item) : Num<float>::inf();
        int lstart = first;
        if (TAIL && spec == 2 && live) lstart = resume_row(tab, a.tab_len, first, r2s);
        int wstart = lstart;
        if (TAIL && spec == 2) {
            // the wave starts at its smallest row (the rows are wave-uniform loads)
#pragma unroll
            for (int o = WAVE / 2; o > 0; o >>= 1) wstart = min(wstart, __shfl_xor(wstart, o));
        }

        for (int n = wstart; n < a.tab_len; ++n) {
            const TabEntry e = tab[n];
            const T bound = (TAIL && spec == 1) ? vmin<T>(F, (T)r2s) : F;
            const bool act = live && n >= lstart && ((T)e.key2 < bound);
            if (__ballot(live && ((T)e.key2 < bound)) == 0ull) break;
            const int qx = x + e.ax, qy = y + e.ay, qz = z + e.az;
            const bool cin = (unsigned)qx < (unsigned)nx && (unsigned)qy < (unsigned)ny &&
                             (DIM == 2 || (unsigned)qz < (unsigned)nz);
            const bool okx = qx + 1 < nx, oky = qy + 1 < ny, okz = DIM == 2 || qz + 1 < nz;
            const bool work = act && cin;
            const bool edge = !(okx && oky && okz);
            const bool wave_masked = __ballot(work && edge) != 0ull;
            if (!work) continue;
            lane_cells += edge ? 0u : 1u;   // full grid cells, the unit of the work count
            const int base = (DIM == 3 ? qz * sxy : 0) + qy * nx + qx;
            const int ox = okx ? 1 : 0, oy = oky ? nx : 0, oz = (DIM == 3 && okz) ? sxy : 0;
            Geo<T> G;
            if constexpr (MODE == 3) {
                G = geo_fp64(e.ax, e.ay, e.az, sx2d, sy2d, DIM == 3 ? sz2d : 0.0);
            } else {
                G = geo_from_row(e);
            }
            if constexpr (DIM == 3) {
                float v[8];
                v[0] = a.ev[base];
                v[1] = a.ev[base + ox];
                v[2] = a.ev[base + oy];
                v[3] = a.ev[base + oy + ox];
                v[4] = a.ev[base + oz];
                v[5] = a.ev[base + oz + ox];
                v[6] = a.ev[base + oz + oy];
                v[7] = a.ev[base + oz + oy + ox];
                T g[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) g[b] = dose_norm<T>((T)v[b], drT, invdd);
                GuardCtx gc{};
                if constexpr (GMODE == 2) {
                    gc = GuardCtx{a.ev, base, ox, oy, oz, dr, inv_dd64, e.ax, e.ay, e.az, sx2d, sy2d, sz2d};
                }
                T c;
                if (wave_masked)
                    c = cell3<T, true, GMODE>(g, G, is, okx, oky, okz, (T)a.den_guard, gc, lane_fp64, ill);
                else
                    c = cell3<T, false, GMODE>(g, G, is, true, true, true, (T)a.den_guard, gc, lane_fp64, ill);
                F = vmin<T>(F, c);
            } else {
                float v[4];
                v[0] = a.ev[base];
                v[1] = a.ev[base + ox];
                v[2] = a.ev[base + oy];
                v[3] = a.ev[base + oy + ox];
                T g[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) g[b] = dose_norm<T>((T)v[b], drT, invdd);
                T c;
                if (wave_masked)
                    c = cell2<T, true>(g, G, is, okx, oky);
                else
                    c = cell2<T, false>(g, G, is, true, true);
                F = vmin<T>(F, c);
            }
        }

        const bool to_guard = MODE == 1 && live && ill;
        const bool to_fb = TAIL && spec == 1 && live && !to_guard && (float)F > r2s;
        if (live && !to_guard && !to_fb) {
            finish_node(a, node, (float)F, npass, nborder, gm);
            cells += lane_cells + (TAIL ? zero_cells(DIM, x, y, z, nx, ny, nz) : 0u);
            n_fp64 += lane_fp64;
        }
        if (to_fb) cells += lane_cells;
        if (MODE == 1) {
            const uint32_t gpos = block_append(to_guard, &a.sc->n_guard);
            if (to_guard) a.guard_list[gpos] = (uint32_t)node;
        }
        if (TAIL && spec == 1) {
            const uint32_t fpos = block_append(to_fb, &a.sc->n_fallback);
            if (to_fb) {
                a.fb_list[fpos] = item;
                a.tail_f[item] = f2u((float)F);
            }
        }
    }
    block_sums(sums, vb, npass, nborder, n_fp64, cells, gm, a.sc);
}

template <int DIM, int MODE, bool TAIL>
__global__ __launch_bounds__(SEARCH_THREADS) void k_walk(SearchArgs a, const TabEntry* __restrict__ tab,
                                                         const uint32_t* __restrict__ order,
                                                         const uint32_t* __restrict__ count, int first,
                                                         int spec, BlockSums* sums) {
    walk_body<DIM, MODE, TAIL>(a, tab, order, count, first, spec, sums, blockIdx.x, gridDim.x);
}

// Pass B with G lanes per node: the G lanes of a group take G consecutive table rows of
// one node at once (independent loads, so the gathers of G cells overlap instead of
// forming one dependent chain), then take the minimum over the group and move to the next
// G rows while the first of them still has key^2 < gamma^2.  Every row the sequential walk
// would evaluate is evaluated; up to G-1 rows past its break may be too.
// MODE 0: FP32; 1: FP32 + flag ill-conditioned tetrahedra (3D).
// g_req: lanes per node (8..64), or <= 0 to pick it from the tail length on the device:
// about 2^19 lanes in flight fill the GPU, so a short tail gets wide groups (latency) and a
// long one narrow groups (fewer rows past the break), but never fewer than -g_req (when
// negative) lanes: a tail whose longest walks are long needs wide groups whatever its
// length, since the kernel lasts as long as its longest walk.
// spec: as in k_walk (1 speculative, 2 fallback from the first row at or beyond f gamma_hat).
template <int DIM, int MODE>
__device__ __forceinline__ void tail_group_body(const SearchArgs& a, const TabEntry* __restrict__ tab,
                                                const uint32_t* __restrict__ order,
                                                const uint32_t* __restrict__ count, int first, int g_req,
                                                int spec, BlockSums* sums, uint32_t vb, uint32_t vgrid) {
    constexpr int GMODE = (DIM == 3 && MODE == 1) ? 1 : 0;
    const uint32_t M = *count;
    int G = g_req;
    if (G <= 0) {
        // automatic: -g_req (if given) is the least width, raised for lists whose longest
        // walks would otherwise take many dependent steps
        const int gmin = G < 0 ? -G : 8;
        G = 64;
        while (G > gmin && (uint64_t)M * (uint64_t)G > (1ull << 19)) G >>= 1;
    }
    const int GROUPS = SEARCH_THREADS / G;
    const int gl = threadIdx.x % G;               // lane within the group
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int sxy = nx * ny;
    const float inv_dd_g = a.sc->inv_dd;
    const InvS2<float> is = inv_s2_of(a);
    uint32_t cells = 0, gm = 0, npass = 0, nborder = 0, nfb = 0;
    GuardCtx gc{};
    uint32_t dummy_fp64 = 0;

    // block-uniform trip count
    for (uint64_t base = (uint64_t)vb * GROUPS; base < M; base += (uint64_t)vgrid * GROUPS) {
        const uint32_t i = (uint32_t)base + threadIdx.x / G;
        const bool live = i < M;
        const uint32_t item = !live ? 0u : (order ? order[i] : i);
        const int node = live ? (int)a.tail_node[item] : 0;
        const int x = node % nx;
        const int y = (node / nx) % ny;
        const int z = DIM == 3 ? node / sxy : 0;
        const float dr = a.ref[node];
        const float inv_dd = node_inv_dd(dr, inv_dd_g, a.dd, a.local);
        float F = live ? u2f(a.tail_f[item]) : 0.0f;
        uint32_t lane_cells = 0;
        bool ill = false;
        const float r2s = (spec && live) ? spec_bound2(a, item) : Num<float>::inf();
        // the fallback resumes at the first row the speculative bound cut off, which the
        // speculative launch stored in the (by then unused) sort-key slot of the item
        const int start = (spec == 2 && live) ? (int)a.tail_key_arr[item] : first;
        // The first batch's row (a listed node always takes part in it), in flight with the node's
        // loads: a short list is a chain of dependent loads.  With the list position not
        // loaded where the list is unsorted, 11.7 -> 10.9 us at 96x128x128, 9.3 -> 8.5 at 64x64.
        TabEntry e = tab[min(start + gl, a.tab_len - 1)];
        uint32_t steps = 0;   // batches of G rows this group walked
        int last_n0 = -1;     // first row of the group's last batch (speculative walk)

        for (int n0 = start; n0 < a.tab_len; n0 += G) {
            const float k_first = tab[n0].key2;       // uniform per group
            const float bound = spec == 1 ? vmin<float>(F, r2s) : F;
            const bool grp_act = live && k_first < bound;
            if (__ballot(grp_act) == 0ull) break;
            steps += grp_act ? 1u : 0u;
            last_n0 = grp_act ? n0 : last_n0;
            const int n = n0 + gl;
            bool act = false;
            if (grp_act && n < a.tab_len) {
                if (n0 != start) e = tab[n];
                act = e.key2 < bound;
            }
            int qx = 0, qy = 0, qz = 0;
            if (act) {
                qx = x + e.ax;
                qy = y + e.ay;
                qz = z + e.az;
            }
            const bool cin = (unsigned)qx < (unsigned)nx && (unsigned)qy < (unsigned)ny &&
                             (DIM == 2 || (unsigned)qz < (unsigned)nz);
            const bool okx = qx + 1 < nx, oky = qy + 1 < ny, okz = DIM == 2 || qz + 1 < nz;
            const bool work = act && cin;
            const bool edge = !(okx && oky && okz);
            const bool wave_masked = __ballot(work && edge) != 0ull;
            float c = Num<float>::inf();
            constexpr int NV = DIM == 3 ? 8 : 4;
            float g[NV];
            // Dose bound: the PL dose inside the cell lies between its vertex values, so a
            // cell whose vertex differences share a sign is at least key^2 + (smallest
            // |difference|)^2 from the node; at or above F it cannot lower F and is skipped
            // (still counted as visited).  A lane's decision is its own, so the result does
            // not depend on which nodes share the wave.
            bool need = false;
            if (work) {
                lane_cells += edge ? 0u : 1u;
                const int base_i = (DIM == 3 ? qz * sxy : 0) + qy * nx + qx;
                const int ox = okx ? 1 : 0, oy = oky ? nx : 0, oz = (DIM == 3 && okz) ? sxy : 0;
                g[0] = a.ev[base_i];
                g[1] = a.ev[base_i + ox];
                g[2] = a.ev[base_i + oy];
                g[3] = a.ev[base_i + oy + ox];
                if constexpr (DIM == 3) {
                    g[4] = a.ev[base_i + oz];
                    g[5] = a.ev[base_i + oz + ox];
                    g[6] = a.ev[base_i + oz + oy];
                    g[7] = a.ev[base_i + oz + oy + ox];
                }
                float gmin = Num<float>::inf(), gmax = -Num<float>::inf();
#pragma unroll
                for (int b = 0; b < NV; ++b) {
                    g[b] = dose_norm<float>(g[b], dr, inv_dd);
                    gmin = vmin<float>(gmin, g[b]);
                    gmax = __builtin_fmaxf(gmax, g[b]);
                }
                const float m = gmin > 0.0f ? gmin : (gmax < 0.0f ? -gmax : 0.0f);
                // margin 2^-8 F: far above the rounding of the projections, so a skipped
                // cell's projected value could not have been below F either, and F, the
                // walk and the result are bit for bit those of the unpruned walk
                need = e.key2 + m * m < F + F * 0x1p-8f;
                // the guard still judges a skipped cell's tetrahedra (whether a node is
                // redone in FP64 must not depend on the pruning)
                if constexpr (GMODE == 1)
                    if (!need && okx && oky && okz) ill = ill || tets_ill(g, is, a.den_guard);
            }
            // the whole projection only where some lane of the wave needs it
            if (__ballot(need) != 0ull && need) {
                const Geo<float> Gm = geo_from_row(e);
                if constexpr (DIM == 3) {
                    if (wave_masked)
                        c = cell3<float, true, GMODE>(g, Gm, is, okx, oky, okz, a.den_guard, gc, dummy_fp64, ill);
                    else
                        c = cell3<float, false, GMODE>(g, Gm, is, true, true, true, a.den_guard, gc, dummy_fp64,
                                                       ill);
                } else {
                    if (wave_masked)
                        c = cell2<float, true>(g, Gm, is, okx, oky);
                    else
                        c = cell2<float, false>(g, Gm, is, true, true);
                }
            }
            // group minimum (the group is G consecutive lanes of the wave)
#pragma unroll
            for (int o = G / 2; o > 0; o >>= 1) c = vmin<float>(c, __shfl_xor(c, o));
            F = vmin<float>(F, c);
        }
        // reduce the group's flags and cell counts onto its first lane
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
            lane_cells += (uint32_t)__shfl_xor((int)lane_cells, o);
            ill = (__shfl_xor((int)ill, o) != 0) || ill;
        }
        // record a long walk (rare): the next map of this context widens its groups
        {
            uint32_t rows = (live && gl == 0) ? steps * (uint32_t)G : 0u;
            if (__ballot(rows > LONG_WALK_ROWS) != 0ull) {
                for (int o = WAVE / 2; o > 0; o >>= 1) rows = max(rows, (uint32_t)__shfl_xor((int)rows, o));
                if ((threadIdx.x & (WAVE - 1)) == 0) atomicMax(&a.sc->long_rows, rows);
            }
        }
        const bool leader = live && gl == 0;
        const bool to_guard = MODE == 1 && leader && ill;
        const bool to_fb = spec == 1 && leader && !to_guard && F > r2s;
        // a short tail walks with the plain bound; the nodes the prediction would not have
        // certified (F above its bound) are counted as its fallbacks, except those the guard
        // redoes (as the speculative walk does)
        if (spec == 3) nfb += (leader && !to_guard && F > r2s) ? 1u : 0u;
        if (leader && !to_guard && !to_fb) {
            finish_node(a, node, F, npass, nborder, gm);
            cells += lane_cells + zero_cells(DIM, x, y, z, nx, ny, nz);
        }
        if (to_fb) cells += lane_cells;
        if (MODE == 1) {
            const uint32_t gpos = block_append(to_guard, &a.sc->n_guard);
            if (to_guard) a.guard_list[gpos] = (uint32_t)node;
        }
        if (spec == 1) {
            // the first row the speculative bound cut off.  A node sent to the fallback kept
            // F above r2s, so its bound was r2s throughout: it walked every row before its
            // last batch and, in that batch, the rows below r2s (a prefix: rows are in key
            // order); with no batch walked it is the first row
            const int rr = last_n0 + gl;
            const bool below = last_n0 >= 0 && rr < a.tab_len && tab[rr].key2 < r2s;
            const unsigned long long bm = __ballot(below);
            const int lane = (int)(threadIdx.x & (WAVE - 1));
            const unsigned long long gmask = G >= WAVE ? ~0ull : (((1ull << G) - 1ull) << (lane & ~(G - 1)));
            const int cut = last_n0 < 0 ? start : last_n0 + (int)__popcll(bm & gmask);
            const uint32_t fpos = block_append(to_fb, &a.sc->n_fallback);
            if (to_fb) {
                a.fb_list[fpos] = item;
                a.tail_f[item] = f2u(F);
                a.tail_key_arr[item] = (uint32_t)cut;
            }
        }
    }
    if (spec == 3) {
        // one atomic per block (one per wave on a single address serialises)
        __shared__ uint32_t s_fb[SEARCH_THREADS / WAVE];
        for (int o = WAVE / 2; o > 0; o >>= 1) nfb += (uint32_t)__shfl_xor((int)nfb, o);
        if ((threadIdx.x & (WAVE - 1)) == 0) s_fb[threadIdx.x / WAVE] = nfb;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = 0u;
            for (int j = 0; j < SEARCH_THREADS / WAVE; ++j) t += s_fb[j];
            if (t) atomicAdd(&a.sc->n_fallback_inline, t);
        }
    }
    block_sums(sums, vb, npass, nborder, 0u, cells, gm);
}

template <int DIM, int MODE>
__global__ __launch_bounds__(SEARCH_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_tail_group(SearchArgs a, const TabEntry* __restrict__ tab,
                                                               const uint32_t* __restrict__ order,
                                                               const uint32_t* __restrict__ count, int first,
                                                               int g_req, int spec, BlockSums* sums) {
    tail_group_body<DIM, MODE>(a, tab, order, count, first, g_req, spec, sums, blockIdx.x, gridDim.x);
}

// Pass B for long tails (plain radius, automatic layout).  The walk of a node is split into a
// cheap scan and the projections:
//   scan  a group of 8 lanes tests 32 rows of its node per step (4 per lane, their loads in
//         flight together); a row whose cell can still lower F, by the dose bound, goes to
//         the wave's queue in LDS;
//   eval  when 64 cells are queued, whichever nodes they belong to, the wave projects them, one
//         per lane, and each takes its node's F down with an LDS minimum.  A queued cell whose
//         bound F has passed meanwhile is dropped.
// A group that finishes a node takes its next one without waiting for the other groups, and
// past TQ_LONG rows a node is scanned by the whole wave (its walk would outlast the others').
// The groups of a wave take neighbouring list entries, whose cells share cache lines, or
// (spread) entries far apart, since long walks lie together in the list and a wave walks its own
// one after the other.
//
// Why: a projection costs about ten times a test.  A tail node visits about 30 cells (158 at a
// 5 % dose error) of which 11 (23) can lower F, and walking 8 rows of a node at a time
// projected all 64 of the wave's whenever one could.  Measured, walking 8 rows at a time against
// this: 482535 nodes at 192x256x256 410 -> 204 us; 349353 nodes under local normalisation
// (walks up to 1440 rows) 407 -> 168 us; 1.25 M nodes at 160x200x200 with a 5 % dose error
// 4.3 -> 1.54 ms.  Bound by VALU issue (80 % of it: 191 instructions of a wave per node, of
// which the 11 projections are 74).
//
// A projection's or test's arithmetic is that of tail_group_body, the minimum does not depend
// on its order and a dropped or untested cell cannot lower F, so F has the same bits.  The
// sequential walk visits exactly the rows whose key is below the final F (every row up to the
// one that gives F has a smaller key), so the visited cells and the ill-conditioned
// tetrahedra are judged by the final F: which nodes share a wave changes no count.
//
// The test needs the range of a cell's corner doses.  For a tail worth it (range_min nodes),
// k_cell_range has written every cell's range beforehand: one 8-byte load per row instead of
// eight gathers.
constexpr int TQ_LANES = 8, TQ_ROWS = 4, TQ_STEP = TQ_LANES * TQ_ROWS;
constexpr int TQ_GROUPS = SEARCH_THREADS / TQ_LANES;   // of a workgroup
constexpr int TQ_LONG = 256;   // rows after which a walk goes on in steps of the whole wave
constexpr int TQ_FEW = 2;      // groups with rows left at which a partial batch is projected
constexpr int TQ_TAB = 192;    // table rows staged in LDS
constexpr int TQ_RING = 512;   // queue slots of a wave: 63 left over and a step of 8 groups fit
static_assert(TQ_TAB <= SEARCH_THREADS, "two grids: a thread per staged row");
static_assert(WAVE - 1 + WAVE * TQ_ROWS <= TQ_RING && (TQ_RING & (TQ_RING - 1)) == 0, "queue ring");

// Sum over the 8 lanes of a group by data-parallel primitives (no LDS round trip): lanes 1
// and 2 apart within a quad, then the mirrored lane of the group's other quad.
template <int CTRL>
__device__ __forceinline__ int dpp8(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false); }
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141;
__device__ __forceinline__ uint32_t sum8(uint32_t v) {
    v += (uint32_t)dpp8<DPP_XOR1>((int)v);
    v += (uint32_t)dpp8<DPP_XOR2>((int)v);
    return v + (uint32_t)dpp8<DPP_HALF_MIRROR>((int)v);
}

// Smallest and largest corner dose of a cell.
template <int DIM>
__device__ __forceinline__ void corner_range(const float* __restrict__ ev, int b0, int ox, int oy, int oz, float& lo,
                                             float& hi) {
    const float v0 = ev[b0], v1 = ev[b0 + ox], v2 = ev[b0 + oy], v3 = ev[b0 + oy + ox];
    lo = vmin<float>(vmin<float>(v0, v1), vmin<float>(v2, v3));
    hi = __builtin_fmaxf(__builtin_fmaxf(v0, v1), __builtin_fmaxf(v2, v3));
    if constexpr (DIM == 3) {
        const float v4 = ev[b0 + oz], v5 = ev[b0 + oz + ox], v6 = ev[b0 + oz + oy], v7 = ev[b0 + oz + oy + ox];
        lo = vmin<float>(lo, vmin<float>(vmin<float>(v4, v5), vmin<float>(v6, v7)));
        hi = __builtin_fmaxf(hi, __builtin_fmaxf(__builtin_fmaxf(v4, v5), __builtin_fmaxf(v6, v7)));
    }
}

// Range of the corner doses of every cell (index of its lower corner; corners past the grid
// count as the last node, as in the walk).  A thread takes one column of RANGE_Z planes and
// carries the range of a plane's four corners to the next cell.
constexpr int RANGE_Z = 8;
__global__ __launch_bounds__(SEARCH_THREADS) void k_cell_range(const float* __restrict__ ev, int nx, int ny, int nz,
                                                               const uint32_t* __restrict__ count, uint32_t least,
                                                               float2* __restrict__ range) {
    if (*count < least) return;
    const int64_t sxy = (int64_t)nx * ny;
    const uint32_t cols = (uint32_t)((sxy + SEARCH_THREADS - 1) / SEARCH_THREADS);
    const uint32_t zb = blockIdx.x / cols;
    const int64_t c = (int64_t)(blockIdx.x - zb * cols) * SEARCH_THREADS + threadIdx.x;
    if (c >= sxy) return;
    const int x = (int)(c % nx), y = (int)(c / nx);
    const int ox = x + 1 < nx ? 1 : 0, oy = y + 1 < ny ? nx : 0;
    const int z0 = (int)zb * RANGE_Z;
    float v[RANGE_Z + 1][4];
#pragma unroll
    for (int k = 0; k <= RANGE_Z; ++k) {
        const int zz = z0 + k < nz ? z0 + k : nz - 1;
        const float* p = ev + zz * sxy + c;
        v[k][0] = p[0];
        v[k][1] = p[ox];
        v[k][2] = p[oy];
        v[k][3] = p[oy + ox];
    }
    float lo[RANGE_Z + 1], hi[RANGE_Z + 1];
#pragma unroll
    for (int k = 0; k <= RANGE_Z; ++k) {
        lo[k] = vmin<float>(vmin<float>(v[k][0], v[k][1]), vmin<float>(v[k][2], v[k][3]));
        hi[k] = __builtin_fmaxf(__builtin_fmaxf(v[k][0], v[k][1]), __builtin_fmaxf(v[k][2], v[k][3]));
    }
#pragma unroll
    for (int k = 0; k < RANGE_Z; ++k)
        if (z0 + k < nz)
            range[(z0 + k) * sxy + c] = make_float2(vmin<float>(lo[k], lo[k + 1]), __builtin_fmaxf(hi[k], hi[k + 1]));
}

// List entries of the queued walk's groups.  Of a list of TQ_OPEN_ROUNDS entries per group or
// more, the first TQ_DEALT sixteenths are dealt out in strides of the whole grid (an entry per
// group and round); the rest lie in up to TQ_POOLS pools and are claimed TQ_CLAIM at a time by
// the waves of the pool's blocks that get there first, since the cost of a node varies and
// waves with cheap nodes ran dry long before the last one (a wave lived 80 % of the launch on
// average).  Dealt out / claimed: 1908 / 1540 us for 1.25 M nodes with a 5 % dose error, 213 /
// 204 for 482535 nodes at 192x256x256, 175 / 168 for 349353 under local normalisation.  (Dealing
// 1/4, 5/8 or 3/4 of the list, 16 to 64 pools and claims of 16 differ by less than 5 %; one pool
// for all took 360 us for the second: atomics on one address take about 8 ns each.)
constexpr uint32_t TQ_OPEN_ROUNDS = 8, TQ_DEALT = 6;
constexpr uint32_t TQ_CLAIM = 8;
constexpr uint32_t TQ_POOLS = 64;   // of 64 waves each in a full grid
static_assert(TQ_POOLS * 4 <= SUM_BINS, "a partial slot per pool, four apart");
static_assert(TQ_CLAIM >= WAVE / TQ_LANES, "one claim serves every group of a wave");
static_assert(TQ_OPEN_ROUNDS * TQ_DEALT / 16u >= 2u, "the entries in flight at the start are dealt ones");
// The dealt part of a list of M entries (whole rounds of `stride`).
__device__ __forceinline__ uint32_t tq_split(uint32_t M, uint32_t stride) {
    return M / stride < TQ_OPEN_ROUNDS ? M : (uint32_t)((uint64_t)M * TQ_DEALT / 16u) / stride * stride;
}
// The next open entry of every group with `want` (the same in the lanes of a group).  st: the
// wave's claim (its next entry and end; in LDS, since the walk has no registers to spare).
__device__ __forceinline__ uint32_t tq_claim(bool want, int lane, uint32_t split, uint32_t vb, uint32_t vgrid,
                                             BlockSums* sums, uint2* st) {
    const unsigned long long m = __ballot(want && (lane & (TQ_LANES - 1)) == 0);
    const uint32_t next = (uint32_t)__builtin_amdgcn_readfirstlane((int)st->x);
    const uint32_t c = (uint32_t)__popcll(m), left = (uint32_t)__builtin_amdgcn_readfirstlane((int)st->y) - next;
    const uint32_t rank = (uint32_t)__popcll(m & ((1ull << (lane & ~(TQ_LANES - 1))) - 1ull));
    uint32_t i = next + rank;
    if (c <= left) {
        if (lane == 0) st->x = next + c;
        return i;
    }
    const uint32_t pools = min(vgrid, TQ_POOLS), pool = vb % pools;
    uint32_t v = 0u;
    if (lane == 0) v = atomicAdd(&sums[4u * pool].claims, 1u);
    const uint32_t base = split + ((uint32_t)__builtin_amdgcn_readfirstlane((int)v) * pools + pool) * TQ_CLAIM;
    if (rank >= left) i = base + (rank - left);
    if (lane == 0) *st = make_uint2(base + (c - left), base + TQ_CLAIM);
    return i;
}

// The node of a group, read by the group's scan and by the lanes that project its cells.
struct alignas(16) TqNode {
    int x, y, z, node;
    float dr, inv_dd;
    uint32_t f;      // F (non-negative float bits: an unsigned minimum is the float minimum; FP64:
                     // rounded up, which every float key is below exactly when it is below F)
    uint32_t inner;  // every cell with key below F lies inside the grid, whole
};

// What a group has finished.  In LDS: kept in registers, these and the last step's keys made the
// walk spill twelve, and a reload waits for the loads in flight (178 -> 171 us for 349353
// nodes under local normalisation).
struct TqCounts {
    uint32_t pass, border, cells, maxg2, long_rows;
};

// LDS of the walk, one block of it for every form of a kernel.
template <bool FP64>
struct TqLds {
    TabEntry tab[TQ_TAB];
    TqNode node[TQ_GROUPS];
    uint2 queue[SEARCH_THREADS / WAVE][TQ_RING];        // row | group of the wave << 28, bound
    uint2 head[TQ_TAB];                                 // key^2, offset in nodes
    unsigned long long f64[FP64 ? TQ_GROUPS : 1];       // FP64: F and 1 / dD of a group's node
    double inv64[FP64 ? TQ_GROUPS : 1];
    uint2 claim[SEARCH_THREADS / WAVE];
    TqCounts counts[TQ_GROUPS];
};
template <bool FP64>
__device__ __forceinline__ TqLds<FP64>& tq_lds() {
    __shared__ TqLds<FP64> s;
    return s;
}

template <int DIM, int MODE>
__device__ __forceinline__ void tail_queue_body(const SearchArgs& a, const TabEntry* __restrict__ tab,
                                                const uint32_t* __restrict__ order, uint32_t M, int first,
                                                BlockSums* sums, uint32_t vb, uint32_t vgrid) {
    constexpr int NV = DIM == 3 ? 8 : 4;
    constexpr bool FP64 = MODE == 3;
    using T = typename std::conditional<FP64, double, float>::type;
    TqLds<FP64>& lds = tq_lds<FP64>();
    auto& s_node = lds.node;
    auto& s_counts = lds.counts;
    auto& s_claim = lds.claim;
    auto& s_f64 = lds.f64;
    auto& s_inv64 = lds.inv64;
    auto& s_queue = lds.queue;
    auto& s_tab = lds.tab;
    auto& s_head = lds.head;
    const int lane = threadIdx.x & (WAVE - 1), gl = lane & (TQ_LANES - 1), gsh = lane & ~(TQ_LANES - 1);
    uint2* queue = s_queue[threadIdx.x / WAVE];
    TqNode* wnode = s_node + (threadIdx.x / WAVE) * (WAVE / TQ_LANES);
    TqNode& self = wnode[lane / TQ_LANES];
    TqCounts& counts = s_counts[threadIdx.x / TQ_LANES];   // kept by the group's first lane
    const int nx = a.nx, ny = a.ny, nz = a.nz, sxy = nx * ny;
    const float inv_dd_g = a.sc->inv_dd;
    const InvS2<T> is = inv_s2_for<T>(a);
    const int wgrp = FP64 ? (threadIdx.x / WAVE) * (WAVE / TQ_LANES) : 0;   // first group of the wave
    const bool ranges = a.range != nullptr && M >= a.range_min;   // (N < 2^29: byte offsets fit 32 bits)
    GuardCtx gc{};
    uint32_t dummy_fp64 = 0;
    bool dummy_ill = false;

    // the first rows of the walk, which every node visits, in LDS
    const int tab_len = a.tab_len - first, tab_lds = min(tab_len, TQ_TAB);
    tab += first;
    for (int u = threadIdx.x; u < tab_lds * 4; u += SEARCH_THREADS)
        reinterpret_cast<uint4*>(s_tab)[u] = reinterpret_cast<const uint4*>(tab)[u];
    // (a group that never gets a node still reads one in the steps of the others: node 0)
    if (gl == 0) {
        self = TqNode{};
        counts = TqCounts{};
    }
    if (lane == 0) s_claim[threadIdx.x / WAVE] = make_uint2(0u, 0u);
    for (int u = threadIdx.x; u < tab_lds; u += SEARCH_THREADS) {
        const TabEntry& e = tab[u];
        s_head[u] = make_uint2(f2u(e.key2), (uint32_t)((e.az * ny + e.ay) * nx + e.ax));
    }
    __syncthreads();
    // key^2 (infinite past the table) and offset of row n
    auto row_head = [&](int n) -> int4 {
        int4 e = make_int4(0x7F800000, 0, 0, 0);
        if (n < tab_lds) e = *reinterpret_cast<const int4*>(&s_tab[n]);
        else if (n < tab_len) e = *reinterpret_cast<const int4*>(&tab[n]);
        return e;
    };

    const uint32_t waves = vgrid * (SEARCH_THREADS / WAVE), wave = vb * (SEARCH_THREADS / WAVE) + threadIdx.x / WAVE;
    const uint32_t grp = (uint32_t)(lane / TQ_LANES);
    uint32_t i = a.spread ? grp * waves + wave : wave * (WAVE / TQ_LANES) + grp;
    const uint32_t stride = vgrid * TQ_GROUPS, split = tq_split(M, stride);
    bool have = false, done = false;
    int n0 = 0;                           // the node's next row
    uint32_t q_head = 0, q_tail = 0;      // of the wave's queue (uniform)
    uint32_t q_last = 0;                  // the node's last queued cell lies before this position
    uint32_t lane_cells = 0, whole = 0;   // whole cells of this lane's rows; of the last step only
    float ill_key = Num<float>::inf();    // smallest key of a cell with an ill-conditioned tetrahedron
    // the group's next node, loaded while the current one is walked: its dose one iteration
    // after its index, so that no load waits for another
    int p_node = 0;
    uint32_t p_hi = 0;   // FP64: high word of the bound
    float p_f = 0.0f, p_dr = 0.0f;
    bool p_have = i < M, p_fresh = true;
    if (p_have) {
        const uint32_t item = order ? order[i] : i;
        p_node = (int)a.tail_node[item];
        p_f = u2f(a.tail_f[item]);
        if constexpr (FP64) p_hi = a.tail_key_arr[item];
    }
    i += stride;   // (the entry after next from here on)

    // One scan step.  KIND 0: each group its own node's rows, all in LDS and every cell inside
    // the grid; 1: the same without those conditions; 2: the whole wave the rows of group wg's
    // node (KIND 0, 1: wg is the lane's own group).  row0: this lane's first row.
    auto scan_step = [&](auto kind, int wg, int row0) {
        constexpr int KIND = decltype(kind)::value;
        constexpr int RSTEP = KIND == 2 ? WAVE : TQ_LANES;
        const bool scan = KIND == 2 || (have && !done), mine = KIND == 2 ? lane / TQ_LANES == wg : scan;
        const TqNode nd = wnode[wg];
        const float F = u2f(nd.f), Fm = F + F * 0x1p-8f;
        bool past = false;   // a row of the step at or past F (or past the table): the rows end here
        if (mine) {
            lane_cells += __popc(whole);   // the step before held no row past F
            whole = 0u;
        }
        float kk[TQ_ROWS], lo[TQ_ROWS], hi[TQ_ROWS];   // keys, range of each row's corner doses
        int b0[TQ_ROWS];
        uint32_t work = 0u, full = 0u;
#pragma unroll
        for (int k = 0; k < TQ_ROWS; ++k) {
            kk[k] = lo[k] = hi[k] = 0.0f;
            b0[k] = nd.node;
            if constexpr (KIND == 0) {
                // (a lane that does not scan reads row 0, whose cell exists for its node)
                const uint2 e = s_head[scan ? row0 + k * RSTEP : 0];
                kk[k] = u2f(e.x);
                const bool in = scan && kk[k] < F;
                past = past || !in;
                work |= in ? 1u << k : 0u;
                b0[k] += in ? (int)e.y : 0;
            } else if (scan) {
                const int4 e = row_head(row0 + k * RSTEP);
                kk[k] = __builtin_bit_cast(float, e.x);
                const int qx = nd.x + e.y, qy = nd.y + e.z, qz = nd.z + e.w;
                const bool in = (unsigned)qx < (unsigned)nx && (unsigned)qy < (unsigned)ny &&
                                (DIM == 2 || (unsigned)qz < (unsigned)nz) && kk[k] < F;
                const bool okx = qx + 1 < nx, oky = qy + 1 < ny, okz = DIM == 2 || qz + 1 < nz;
                past = past || !(kk[k] < F);
                if (in) {
                    work |= 1u << k;
                    full |= okx && oky && okz ? (1u << k) : 0u;
                    b0[k] = (DIM == 3 ? qz * sxy : 0) + qy * nx + qx;
                    if (!ranges)
                        corner_range<DIM>(a.ev, b0[k], okx ? 1 : 0, oky ? nx : 0, (DIM == 3 && okz) ? sxy : 0, lo[k], hi[k]);
                }
            }
        }
        if constexpr (KIND == 0) full = work;
        if (ranges) {
#pragma unroll
            for (int k = 0; k < TQ_ROWS; ++k) {
                // (a row without work reads its node's own cell; byte offsets fit 32 bits)
                const float2 r = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(a.range) + (uint32_t)b0[k] * 8u);
                lo[k] = r.x;
                hi[k] = r.y;
            }
        } else if constexpr (KIND == 0) {
#pragma unroll
            for (int k = 0; k < TQ_ROWS; ++k)
                if ((work >> k) & 1u) corner_range<DIM>(a.ev, b0[k], 1, nx, DIM == 3 ? sxy : 0, lo[k], hi[k]);
        }
        const uint32_t before = q_tail;
        float bad_key = Num<float>::inf();
        uint32_t wide_cells = 0u;
        bool suspect = false;   // a whole cell whose corners span enough for an ill-conditioned tetrahedron
#pragma unroll
        for (int k = 0; k < TQ_ROWS; ++k) {
            // the normalisation is monotone, so the range of the normalised corners is the
            // normalised range, bit for bit
            const float glo = dose_norm<float>(lo[k], nd.dr, nd.inv_dd), ghi = dose_norm<float>(hi[k], nd.dr, nd.inv_dd);
            const float m = __builtin_fmaxf(__builtin_fmaxf(glo, -ghi), 0.0f);
            float lb = fmadd(m, m, kk[k]);
            // FP64: a bound past the float range (doses below 1e-37 under local normalisation) says nothing
            if constexpr (FP64) lb = lb < Num<float>::inf() ? lb : 0.0f;
            const bool need = ((work >> k) & 1u) && lb < Fm;
            if constexpr (DIM == 3 && MODE == 1) suspect = suspect || !((ghi - glo) * (ghi - glo) < a.ill_span2);
            const unsigned long long mask = __ballot(need);
            if (need)
                queue[(q_tail + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))) &
                      (TQ_RING - 1)] = make_uint2((uint32_t)(row0 + k * RSTEP) | ((uint32_t)wg << 28), f2u(lb));
            q_tail += (uint32_t)__popcll(mask);
            if constexpr (KIND == 2) wide_cells += (uint32_t)__popcll(__ballot((full >> k) & 1u));
        }
        if constexpr (DIM == 3 && MODE == 1) {
            if (__ballot(suspect && full != 0u) != 0ull) {   // rare
#pragma nounroll
                for (int k = 0; k < TQ_ROWS; ++k) {
                    if (!((full >> k) & 1u)) continue;
                    const int4 e = row_head(row0 + k * RSTEP);
                    const int c0 = ((nd.z + e.w) * ny + nd.y + e.z) * nx + nd.x + e.y;
                    float g[8];
#pragma unroll
                    for (int b = 0; b < 8; ++b)
                        g[b] = dose_norm<float>(a.ev[c0 + (b & 1) + ((b >> 1) & 1) * nx + ((b >> 2) & 1) * sxy], nd.dr,
                                                nd.inv_dd);
                    if (tets_ill(g, inv_s2_of(a), a.den_guard)) bad_key = vmin<float>(bad_key, __builtin_bit_cast(float, e.x));
                }
                if (KIND == 2)
                    for (int o = WAVE / 2; o > 0; o >>= 1) bad_key = vmin<float>(bad_key, __shfl_xor(bad_key, o));
                if (mine) ill_key = vmin<float>(ill_key, bad_key);
            }
        }
        const unsigned long long pb = __ballot(past);
        if (mine) {
            if constexpr (KIND == 2) {
                lane_cells += gl == 0 ? wide_cells : 0u;
                n0 += WAVE * TQ_ROWS;
            } else {
                whole = full;
                n0 += TQ_STEP;
                done = ((pb >> gsh) & ((1ull << TQ_LANES) - 1ull)) != 0ull;
            }
            if (q_tail != before) q_last = q_tail;
        }
    };

    for (;;) {
        if (p_fresh) {
            p_dr = a.ref[p_node];
            p_fresh = false;
        }
        bool want = false;
        if (!have && p_have) {
            const uint32_t row = fast_div((uint32_t)p_node, a.div_nx);
            const int z = DIM == 3 ? (int)fast_div(row, a.div_ny) : 0;
            if (gl == 0) {
                const int x = p_node - (int)row * nx, y = (int)row - z * ny;
                // a cell of key below F starts at most sqrt(F) / s past the node's own cells:
                // all are whole while sqrt(F) stays below s times the cells left on either side
                const int cx = min(nx - 2 - x, x - 1), cy = min(ny - 2 - y, y - 1);
                const int cz = DIM == 3 ? min(nz - 2 - z, z - 1) : cx;
                const float fx = (float)cx, fy = (float)cy, fz = (float)cz;
                const float lim = vmin<float>(a.s2x * (fx * fx), vmin<float>(a.s2y * (fy * fy), DIM == 3 ? a.s2z * (fz * fz) : Num<float>::inf()));
                if constexpr (FP64) {
                    const unsigned long long fb = ((unsigned long long)p_hi << 32) | f2u(p_f);
                    s_f64[wgrp + lane / TQ_LANES] = fb;
                    s_inv64[wgrp + lane / TQ_LANES] = fp64_inv_dd(a, p_dr);
                    p_f = __double2float_ru(__builtin_bit_cast(double, fb));
                }
                const bool inner = cx > 0 && cy > 0 && cz > 0 && p_f < lim * 0.999f;
                self = TqNode{x, y, z, p_node, p_dr, node_inv_dd(p_dr, inv_dd_g, a.dd, a.local), f2u(p_f), inner ? 1u : 0u};
            }
            n0 = 0;
            q_last = q_head;
            lane_cells = whole = 0u;
            ill_key = Num<float>::inf();
            have = true;
            done = false;
            p_have = i < M;
            if (p_have) {
                const uint32_t item = order ? order[i] : i;
                p_node = (int)a.tail_node[item];
                p_f = u2f(a.tail_f[item]);
                if constexpr (FP64) p_hi = a.tail_key_arr[item];
                p_fresh = true;
            }
            i += stride;
            want = i >= split;
        }
        if (split < M && __ballot(want) != 0ull) {
            const uint32_t k = tq_claim(want, lane, split, vb, vgrid, sums, &s_claim[threadIdx.x / WAVE]);
            if (want) i = k;
        }
        if (__ballot(have) == 0ull) break;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

        // scan
        bool flush = false;
        if (q_tail - q_head < WAVE && __ballot(have && !done) != 0ull) {
            // a long walk goes on in steps of 256 rows by the whole wave, while all of them lie
            // below F with its queued cells projected (the rest of its rows, and its end, again
            // by the group)
            bool far = have && !done && n0 >= TQ_LONG;
            unsigned long long fb = __ballot(far);
            if (fb != 0ull) {
                if (far) far = __builtin_bit_cast(float, row_head(n0 + WAVE * TQ_ROWS - 1).x) < u2f(self.f);
                fb = __ballot(far);
            }
            if (fb != 0ull) {
                const int wg = (__ffsll(fb) - 1) / TQ_LANES, wl = __builtin_amdgcn_readfirstlane(wg * TQ_LANES);
                flush = (int32_t)(q_head - (uint32_t)__builtin_amdgcn_readlane((int)q_last, wl)) < 0;
                if (!flush) scan_step(std::integral_constant<int, 2>{}, wg, __builtin_amdgcn_readlane(n0, wl) + lane);
            } else if (__ballot(have && !done && (self.inner == 0u || n0 + TQ_STEP > tab_lds)) == 0ull) {
                scan_step(std::integral_constant<int, 0>{}, lane / TQ_LANES, n0 + gl);
            } else {
                scan_step(std::integral_constant<int, 1>{}, lane / TQ_LANES, n0 + gl);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

        // project: 64 cells, or what is queued once few groups have rows left to scan
        const uint32_t queued = q_tail - q_head;
        if (queued >= WAVE || flush || (queued > 0u && __popcll(__ballot(have && !done)) <= TQ_FEW * TQ_LANES)) {
            const uint32_t take = queued < WAVE ? queued : WAVE;
            const uint2 it = queue[(q_head + lane) & (TQ_RING - 1)];
            TqNode* owner = &wnode[(it.x >> 28) & 7u];
            const TqNode nd = *owner;
            const float F = u2f(nd.f);
            const bool proj = (uint32_t)lane < take && u2f(it.y) < F + F * 0x1p-8f;
            TabEntry e{};
            if (proj) {
                const int n = (int)(it.x & 0x0FFFFFFFu);
                if (n < tab_lds) e = s_tab[n];
                else e = tab[n];
            }
            const int qx = nd.x + e.ax, qy = nd.y + e.ay, qz = nd.z + e.az;
            const bool okx = qx + 1 < nx, oky = qy + 1 < ny, okz = DIM == 2 || qz + 1 < nz;
            const bool wave_masked = __ballot(proj && !(okx && oky && okz)) != 0ull;
            if (proj) {
                const int b0 = (DIM == 3 ? qz * sxy : 0) + qy * nx + qx;
                const int ox = okx ? 1 : 0, oy = oky ? nx : 0, oz = (DIM == 3 && okz) ? sxy : 0;
                float v[NV];
                v[0] = a.ev[b0];
                v[1] = a.ev[b0 + ox];
                v[2] = a.ev[b0 + oy];
                v[3] = a.ev[b0 + oy + ox];
                if constexpr (DIM == 3) {
                    v[4] = a.ev[b0 + oz];
                    v[5] = a.ev[b0 + oz + ox];
                    v[6] = a.ev[b0 + oz + oy];
                    v[7] = a.ev[b0 + oz + oy + ox];
                }
                T inv = nd.inv_dd;
                Geo<T> Gm;
                if constexpr (FP64) {
                    inv = s_inv64[wgrp + (int)((it.x >> 28) & 7u)];
                    Gm = geo_fp64(e.ax, e.ay, e.az, a.sx * a.sx, a.sy * a.sy, DIM == 3 ? a.sz * a.sz : 0.0);
                } else {
                    Gm = geo_from_row(e);
                }
                T g[NV];
#pragma unroll
                for (int b = 0; b < NV; ++b) g[b] = dose_norm<T>((T)v[b], (T)nd.dr, inv);
                T c;
                if constexpr (DIM == 3) {
                    if (wave_masked)
                        c = cell3<T, true, 0>(g, Gm, is, okx, oky, okz, (T)a.den_guard, gc, dummy_fp64, dummy_ill);
                    else
                        c = cell3<T, false, 0>(g, Gm, is, true, true, true, (T)a.den_guard, gc, dummy_fp64, dummy_ill);
                } else {
                    if (wave_masked)
                        c = cell2<T, true>(g, Gm, is, okx, oky);
                    else
                        c = cell2<T, false>(g, Gm, is, true, true);
                }
                if constexpr (FP64) {
                    atomicMin(&s_f64[wgrp + (int)((it.x >> 28) & 7u)], __builtin_bit_cast(unsigned long long, c));
                    atomicMin(&owner->f, f2u(__double2float_ru(c)));
                } else if (c < F) {
                    atomicMin(&owner->f, f2u(c));
                }
            }
            q_head += take;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }

        // finish the nodes whose rows are scanned and whose queued cells are projected
        const bool fin = have && done && (int32_t)(q_head - q_last) >= 0;
        if (__ballot(fin) != 0ull) {
            const TqNode nd = self;
            const float F = u2f(nd.f);
            if (fin) {
#pragma unroll
                for (int k = 0; k < TQ_ROWS; ++k)
                    if ((whole >> k) & 1u)
                        lane_cells += __builtin_bit_cast(float, row_head(n0 - TQ_STEP + k * TQ_LANES + gl).x) < F ? 1u : 0u;
                // steps before the last whose rows the projections have since put past F (rare)
                for (int s0 = n0 - TQ_STEP;
                     s0 > 0 && !(__builtin_bit_cast(float, row_head(s0 - 1).x) < F); s0 -= TQ_STEP) {
#pragma unroll
                    for (int k = 0; k < TQ_ROWS; ++k) {
                        const int4 e = row_head(s0 - TQ_STEP + k * TQ_LANES + gl);
                        const int qx = nd.x + e.y, qy = nd.y + e.z, qz = nd.z + e.w;
                        const bool w = qx >= 0 && qx + 1 < nx && qy >= 0 && qy + 1 < ny &&
                                       (DIM == 2 || (qz >= 0 && qz + 1 < nz));
                        lane_cells -= w && !(__builtin_bit_cast(float, e.x) < F) ? 1u : 0u;
                    }
                }
            }
            const uint32_t sum = sum8(lane_cells);
            bool to_guard = false;
            if constexpr (MODE == 1)
                to_guard = ((__ballot(fin && ill_key < F) >> gsh) & ((1ull << TQ_LANES) - 1ull)) != 0ull;
            if (fin) {
                if (gl == 0) {
                    TqCounts c = counts;
                    if (n0 > (int)LONG_WALK_ROWS && (uint32_t)n0 > c.long_rows)   // (it has at most n0 rows)
                        c.long_rows = max(c.long_rows, (uint32_t)resume_row(tab, tab_len, 0, F));
                    if (!to_guard) {
                        const float Ff = FP64 ? (float)__builtin_bit_cast(double, s_f64[FP64 ? wgrp + lane / TQ_LANES : 0]) : F;
                        finish_node(a, nd.node, Ff, c.pass, c.border, c.maxg2);
                        c.cells += sum + zero_cells(DIM, nd.x, nd.y, nd.z, nx, ny, nz);
                    }
                    counts = c;
                }
                have = false;
            }
            if constexpr (MODE == 1) {
                const bool put = fin && to_guard && gl == 0;
                const unsigned long long gb = __ballot(put);
                if (gb != 0ull) {   // rare: one atomic per wave
                    uint32_t base = 0u;
                    if (lane == 0) base = atomicAdd(&a.sc->n_guard, (uint32_t)__popcll(gb));
                    base = (uint32_t)__shfl((int)base, 0);
                    if (put) a.guard_list[base + (uint32_t)__popcll(gb & ((1ull << lane) - 1ull))] = (uint32_t)nd.node;
                }
            }
        }
    }
    TqCounts c{};
    if (gl == 0) c = counts;
    uint32_t long_rows = c.long_rows;
    if (__ballot(long_rows > LONG_WALK_ROWS) != 0ull) {
        for (int o = WAVE / 2; o > 0; o >>= 1) long_rows = max(long_rows, (uint32_t)__shfl_xor((int)long_rows, o));
        if (lane == 0) atomicMax(&a.sc->long_rows, long_rows);
    }
    block_sums(sums, vb, c.pass, c.border, 0u, c.cells, c.maxg2);
}

// The walk of the automatic layout (vb / vgrid: this block and the number of blocks).
template <int DIM, int MODE>
__device__ __forceinline__ void tail_auto_body(const SearchArgs& a, const uint32_t* __restrict__ order, bool sorted,
                                               const uint32_t* __restrict__ count, int first, int g_req, BlockSums* sums,
                                               uint32_t vb, uint32_t vgrid) {
    if (*count >= QUEUED_TAIL)
        tail_queue_body<DIM, MODE>(a, a.tab, sorted ? order : nullptr, *count, first, sums, vb, vgrid);
    else
        tail_group_body<DIM, MODE>(a, a.tab, sorted ? order : nullptr, count, first, g_req, 0, sums, vb, vgrid);
}

__global__ __launch_bounds__(SEARCH_THREADS) void k_tail_fp64(SearchArgs a, int first, BlockSums* sums) {
    tail_queue_body<3, 3>(a, a.tab, nullptr, a.sc->n_tail, first, sums, blockIdx.x, gridDim.x);
}

template <int DIM, int MODE>
__global__ __launch_bounds__(SEARCH_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_tail_auto(
    SearchArgs a, const uint32_t* __restrict__ order, int sorted, const uint32_t* __restrict__ count, int first, int g_req,
    BlockSums* sums) {
    tail_auto_body<DIM, MODE>(a, order, sorted != 0, count, first, g_req, sums, blockIdx.x, gridDim.x);
}

// One block: sum the per-block partial counts into the scalars, and flag a cell table
// that does not reach the search radius (the host then rebuilds it and runs again).
// ADD: add the sums into the scalars (which the prep zeroed) instead of storing them, so
// that other blocks may add theirs at the same time.
template <bool ADD = false>
__device__ __forceinline__ void finalize_body(const BlockSums* __restrict__ sums, int n, Scalars* sc,
                                              float r2_cap) {
    unsigned long long p = 0, b = 0, f = 0, c = 0;
    uint32_t m = 0, r2 = 0, bad = 0;
    for (int j = threadIdx.x; j < n; j += SEARCH_THREADS) {
        p += sums[j].pass;
        b += sums[j].border;
        f += sums[j].fp64;
        c += sums[j].cells;
        m = max(m, sums[j].maxg2);
        r2 = max(r2, sums[j].prep & ~PREP_BAD);
        bad |= sums[j].prep & PREP_BAD;
    }
    __shared__ unsigned long long s[4][SEARCH_THREADS];
    __shared__ uint32_t sm[SEARCH_THREADS], sr[SEARCH_THREADS];
    bad = (uint32_t)__syncthreads_or((int)bad);
    s[0][threadIdx.x] = p;
    s[1][threadIdx.x] = b;
    s[2][threadIdx.x] = f;
    s[3][threadIdx.x] = c;
    sm[threadIdx.x] = m;
    sr[threadIdx.x] = r2;
    __syncthreads();
    for (int h = SEARCH_THREADS / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            for (int k = 0; k < 4; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + h];
            sm[threadIdx.x] = max(sm[threadIdx.x], sm[threadIdx.x + h]);
            sr[threadIdx.x] = max(sr[threadIdx.x], sr[threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (sr[0] > sc->r2_bits) sc->r2_bits = sr[0];
        if (bad != 0u) sc->flags |= FLAG_NONFINITE;
        if (u2f(sc->r2_bits) > r2_cap && sc->n_masked > 0) sc->flags |= FLAG_TABLE_SHORT;
        if (ADD) {
            if (s[0][0]) atomicAdd(&sc->n_pass, s[0][0]);
            if (s[1][0]) atomicAdd(&sc->n_border, s[1][0]);
            if (s[2][0]) atomicAdd(&sc->n_fp64, s[2][0]);
            if (s[3][0]) atomicAdd(&sc->n_cells, s[3][0]);
            if (sm[0]) atomicMax(&sc->maxg2_bits, sm[0]);
        } else {
            sc->n_pass = s[0][0];
            sc->n_border = s[1][0];
            sc->n_fp64 = s[2][0];
            sc->n_cells = s[3][0];
            sc->maxg2_bits = sm[0];
        }
    }
}

// The map's scalars into the pinned ring at the slot of the device map counter, made visible
// at system scope before the kernel ends; then the counter moves on.  src: global memory
// (read at device scope: other blocks' atomics put the counts there) or LDS.
template <bool LDS>
__device__ __forceinline__ void publish_scalars(const uint32_t* src, uint32_t* seq, Scalars* ring) {
    constexpr int W = (int)(sizeof(Scalars) / sizeof(uint32_t));
    static_assert(sizeof(Scalars) % sizeof(uint32_t) == 0 && W <= WAVE, "Scalars fits one wave's words");
    if (threadIdx.x >= WAVE) return;
    const uint32_t k = *seq;   // (every lane reads the counter before lane 0 moves it on)
    Scalars* dst = ring + (k % SCALAR_RING);
    const int t = threadIdx.x;
    if (t < W)
        reinterpret_cast<volatile uint32_t*>(dst)[t] =
            LDS ? src[t] : __hip_atomic_load(src + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == 0) *seq = k + 1u;
    __threadfence_system();
}

// One block: the partial slots added to the scalars, then the scalars published.
__device__ __forceinline__ void finish_counts(const BlockSums* __restrict__ sums, Scalars* sc, float r2_cap,
                                              uint32_t* seq, Scalars* ring) {
    constexpr int W = (int)(sizeof(Scalars) / sizeof(uint32_t));
    __shared__ __align__(8) uint32_t s_sc[W];
    unsigned long long p = 0, b = 0, f = 0, c = 0;
    uint32_t m = 0, r2 = 0, bad = 0;
    if (threadIdx.x < SUM_BINS) {
        const BlockSums v = sums[threadIdx.x];
        p = v.pass;
        b = v.border;
        f = v.fp64;
        c = v.cells;
        m = v.maxg2;
        r2 = v.prep & ~PREP_BAD;
        bad = v.prep & PREP_BAD;
    }
    if (threadIdx.x < W) s_sc[threadIdx.x] = reinterpret_cast<const uint32_t*>(sc)[threadIdx.x];
    __shared__ unsigned long long s[4][SEARCH_THREADS / WAVE];
    __shared__ uint32_t sm[SEARCH_THREADS / WAVE], sr[SEARCH_THREADS / WAVE];
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        p += (unsigned long long)__shfl_xor((long long)p, o);
        b += (unsigned long long)__shfl_xor((long long)b, o);
        f += (unsigned long long)__shfl_xor((long long)f, o);
        c += (unsigned long long)__shfl_xor((long long)c, o);
        m = max(m, (uint32_t)__shfl_xor((int)m, o));
        r2 = max(r2, (uint32_t)__shfl_xor((int)r2, o));
    }
    bad = __ballot(bad != 0u) != 0ull ? PREP_BAD : 0u;
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        const int w = threadIdx.x / WAVE;
        s[0][w] = p;
        s[1][w] = b;
        s[2][w] = f;
        s[3][w] = c;
        sm[w] = m;
        sr[w] = r2 | bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        Scalars* l = reinterpret_cast<Scalars*>(s_sc);
        for (int w = 0; w < SEARCH_THREADS / WAVE; ++w) {
            l->r2_bits = max(l->r2_bits, sr[w] & ~PREP_BAD);
            if (sr[w] & PREP_BAD) l->flags |= FLAG_NONFINITE;
        }
        if (u2f(l->r2_bits) > r2_cap && l->n_masked > 0) l->flags |= FLAG_TABLE_SHORT;
        for (int w = 0; w < SEARCH_THREADS / WAVE; ++w) {
            l->n_pass += s[0][w];
            l->n_border += s[1][w];
            l->n_fp64 += s[2][w];
            l->n_cells += s[3][w];
            l->maxg2_bits = max(l->maxg2_bits, sm[w]);
        }
    }
    __syncthreads();
    if (threadIdx.x < W) reinterpret_cast<uint32_t*>(sc)[threadIdx.x] = s_sc[threadIdx.x];
    if (ring) publish_scalars<true>(s_sc, seq, ring);
}
// End of a map in one launch: the partial slots of the passes are added to the scalars, the
// nodes with an ill-conditioned tetrahedron are redone in FP64-guarded precision (GUARD: 3D,
// guarded), and the scalars are published (ring: null where the caller reads them itself).
// With no node to redo, block 0 does it all and the others return; else every block takes a
// ticket after its share, and the last one publishes.  (A count reduction with the guard and
// a publishing kernel behind it were two launches of 4.5 and 3.9 us at the end of every map;
// this one takes 4.4.)
template <bool GUARD>
__global__ __launch_bounds__(SEARCH_THREADS) void k_finish(SearchArgs a, const BlockSums* __restrict__ sums,
                                                           uint32_t* seq, Scalars* ring) {
    __shared__ uint32_t s_last;
    Scalars* sc = a.sc;
    if (GUARD && sc->n_guard != 0u) {
        if (blockIdx.x == 0) finalize_body<true>(sums, SUM_BINS, sc, a.r2_cap);
        walk_body<3, 2, false>(a, a.tab, a.guard_list, &sc->n_guard, 0, 0, nullptr, blockIdx.x, gridDim.x);
        if (!ring) return;
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) s_last = atomicAdd(&sc->ticket, 1u) == gridDim.x - 1u ? 1u : 0u;
        __syncthreads();
        if (s_last != 0u) publish_scalars<false>(reinterpret_cast<const uint32_t*>(sc), seq, ring);
        return;
    }
    if (blockIdx.x == 0) finish_counts(sums, sc, a.r2_cap, seq, ring);
}

// The counts and the publication alone (two grids).
__global__ __launch_bounds__(SEARCH_THREADS) void k_finish_counts(const BlockSums* __restrict__ sums, Scalars* sc,
                                                                  uint32_t* seq, Scalars* ring) {
    finish_counts(sums, sc, Num<float>::inf(), seq, ring);
}
static_assert(SUM_BINS <= SEARCH_THREADS, "one partial slot per thread");

constexpr unsigned kTailBlocks = 1024;   // grid-stride blocks of the tail walk
constexpr unsigned kGuardBlocks = 64;    // grid-stride blocks of the guard pass
constexpr unsigned kZeroGroupBlocks = 8192;   // grid-stride blocks of pass A, one lane per cell

unsigned blocks_for(uint32_t m) { return (m + SEARCH_THREADS - 1) / SEARCH_THREADS; }

template <int DIM, int MODE, bool TAIL>
void walk(const SearchArgs& a, const uint32_t* order, const uint32_t* count, int first, unsigned blocks,
          BlockSums* sums, hipStream_t s, int spec = 0) {
    hipLaunchKernelGGL((k_walk<DIM, MODE, TAIL>), dim3(blocks), dim3(SEARCH_THREADS), 0, s, a, a.tab, order,
                       count, first, spec, sums);
}

template <int DIM, int MODE>
void tail_group_g(const SearchArgs& a, const uint32_t* order, const uint32_t* count, int G, int first,
                  unsigned blocks, int spec, BlockSums* sums, hipStream_t s) {
    hipLaunchKernelGGL((k_tail_group<DIM, MODE>), dim3(blocks), dim3(SEARCH_THREADS), 0, s, a, a.tab, order, count,
                       first, G, spec, sums);
}

void tail_group(const SearchArgs& a, const uint32_t* order, const uint32_t* count, int ndim, int mode, int G,
                int first, unsigned blocks, int spec, BlockSums* sums, hipStream_t s) {
    if (ndim == 3) {
        if (mode == 1) tail_group_g<3, 1>(a, order, count, G, first, blocks, spec, sums, s);
        else tail_group_g<3, 0>(a, order, count, G, first, blocks, spec, sums, s);
    } else {
        tail_group_g<2, 0>(a, order, count, G, first, blocks, spec, sums, s);
    }
}

// The cell ranges that the queued walk of `count` nodes reads, where the map has them (every
// launch of that walk comes after this).
void cell_ranges(const SearchArgs& a, const uint32_t* count, hipStream_t s) {
    if (!a.range) return;
    const unsigned cols = (unsigned)(((int64_t)a.nx * a.ny + SEARCH_THREADS - 1) / SEARCH_THREADS);
    hipLaunchKernelGGL(k_cell_range, dim3(cols * (unsigned)((a.nz + RANGE_Z - 1) / RANGE_Z)), dim3(SEARCH_THREADS), 0, s, a.ev,
                       a.nx, a.ny, a.nz, count, a.range_min, a.range);
}

// Pass B over `order` (count on the device): one lane per node (G == 1) or G lanes.
void tail_pass(const SearchArgs& a, const SearchPlan& p, const uint32_t* order, const uint32_t* count,
               int first, bool guarded, int spec, unsigned tb, BlockSums* sums, hipStream_t s) {
    // 0: chosen on the device from the list length; negative: the same with a least width
    const int G = p.tail_lanes ? p.tail_lanes : -(p.tail_min_lanes > 8 ? p.tail_min_lanes : 8);
    if (G == 1) {
        if (p.ndim == 3) {
            if (guarded) walk<3, 1, true>(a, order, count, first, tb, sums, s, spec);
            else walk<3, 0, true>(a, order, count, first, tb, sums, s, spec);
        } else {
            walk<2, 0, true>(a, order, count, first, tb, sums, s, spec);
        }
        return;
    }
    const unsigned groups = SEARCH_THREADS / (unsigned)(G > 0 ? G : -G);
    unsigned gb = (p.M + groups - 1) / groups;
    if (gb > kTailBlocks) gb = kTailBlocks;
    if (G < 0 && spec == 0) {
        cell_ranges(a, count, s);
        const int sorted = p.hist != nullptr;
        if (p.ndim == 3) {
            if (guarded) hipLaunchKernelGGL((k_tail_auto<3, 1>), dim3(gb), dim3(SEARCH_THREADS), 0, s, a, order, sorted, count, first, G, sums);
            else hipLaunchKernelGGL((k_tail_auto<3, 0>), dim3(gb), dim3(SEARCH_THREADS), 0, s, a, order, sorted, count, first, G, sums);
        } else {
            hipLaunchKernelGGL((k_tail_auto<2, 0>), dim3(gb), dim3(SEARCH_THREADS), 0, s, a, order, sorted, count, first, G, sums);
        }
        return;
    }
    tail_group(a, order, count, p.ndim, guarded ? 1 : 0, G, first, gb, spec, sums, s);
}

// ---- batches ------------------------------------------------------------------------

// The key-0 pass of every pair of a batch: block b takes item b = (pair, block of 256 nodes)
// and runs that pair's pass over those nodes, as the pair's own kernel would (a block past
// the pair's M returns at once).
__global__ __launch_bounds__(SEARCH_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_batch_key0(const BatchPair* __restrict__ pairs,
                                                               const uint2* __restrict__ items) {
    const uint2 w = items[blockIdx.x];
    const BatchPair& P = pairs[w.x];
    const SearchArgs& sa = P.sa;
    if (P.ndim == 3) {
        if (P.guarded) zero3_body<1>(sa, P.zg, sa.sums, w.y);
        else zero3_body<0>(sa, P.zg, sa.sums, w.y);
    } else {
        zero2_body(sa, P.zg, sa.sums, w.y);
    }
}

// The tail walk of every pair (no sort, plain radius): block b takes item (pair, tail block).
__global__ __launch_bounds__(SEARCH_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_batch_tail(
    const BatchPair* __restrict__ pairs, const uint2* __restrict__ items) {
    const uint2 w = items[blockIdx.x];
    const BatchPair& P = pairs[w.x];
    const SearchArgs& sa = P.sa;
    const uint32_t* n = &sa.sc->n_tail;
    const uint32_t nb = (uint32_t)P.tail_blocks;
    if (P.g_req < 0) {
        if (P.ndim == 3) {
            if (P.guarded) tail_auto_body<3, 1>(sa, sa.tail_pos, false, n, P.first, P.g_req, sa.sums, w.y, nb);
            else tail_auto_body<3, 0>(sa, sa.tail_pos, false, n, P.first, P.g_req, sa.sums, w.y, nb);
        } else {
            tail_auto_body<2, 0>(sa, sa.tail_pos, false, n, P.first, P.g_req, sa.sums, w.y, nb);
        }
    } else if (P.ndim == 3) {
        if (P.guarded) tail_group_body<3, 1>(sa, sa.tab, sa.tail_pos, n, P.first, P.g_req, 0, sa.sums, w.y, nb);
        else tail_group_body<3, 0>(sa, sa.tab, sa.tail_pos, n, P.first, P.g_req, 0, sa.sums, w.y, nb);
    } else {
        tail_group_body<2, 0>(sa, sa.tab, sa.tail_pos, n, P.first, P.g_req, 0, sa.sums, w.y, nb);
    }
}

// Every pair's guard pass with its count reduction, or the count reduction alone; block 0 of
// each pair then stamps its completion.
__global__ __launch_bounds__(SEARCH_THREADS) void k_batch_finish(const BatchPair* __restrict__ pairs,
                                                                 const uint2* __restrict__ items) {
    const uint2 w = items[blockIdx.x];
    const BatchPair& P = pairs[w.x];
    if (P.guarded) {
        if (w.y == 0) finalize_body<true>(P.sa.sums, SUM_BINS, P.sa.sc, P.sa.r2_cap);
        walk_body<3, 2, false>(P.sa, P.sa.tab, P.sa.guard_list, &P.sa.sc->n_guard, 0, 0, nullptr, w.y, kGuardBlocks);
    } else {
        finalize_body(P.sa.sums, SUM_BINS, P.sa.sc, P.sa.r2_cap);
    }
    if (w.y == 0 && threadIdx.x == 0) *P.done = wall_clock64();
}

__global__ void k_stamp(unsigned long long* t) {
    if (threadIdx.x == 0) *t = wall_clock64();
}

// ---- two grids (the evaluation dose on a grid of its own, 3D) ---------------------------

// Evaluation-grid position of reference node r: u = (k * rh - eo) / eh per axis (z, y, x).
__device__ __forceinline__ void grids_pos(const GridsArgs& a, int r, double u[3], bool& inside) {
    const int x = r % a.rn[2], y = (r / a.rn[2]) % a.rn[1], z = r / (a.rn[2] * a.rn[1]);
    const int k[3] = {z, y, x};
    inside = true;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        u[i] = ((double)k[i] * a.rh[i] - a.eo[i]) / a.eh[i];
        inside = inside && u[i] >= 0.0 && u[i] <= (double)(a.en[i] - 1);
    }
}

// Holding cell (lower corner c0, clamped so that the cell exists) and the node's position f
// inside it, in [0, 1] per axis.
template <typename T>
__device__ __forceinline__ void grids_cell(const GridsArgs& a, const double u[3], int c0[3], T f[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        int c = (int)floor(u[i]);
        c = c > a.en[i] - 2 ? a.en[i] - 2 : (c < 0 ? 0 : c);
        c0[i] = c;
        f[i] = (T)(u[i] - (double)c);
    }
}

// Spatial constants of the cell at offset (a - f) from the node, in evaluation-grid units
// (the per-row constants of the one-grid table, for a node off the grid's nodes).
// (is: the reciprocals of the block sums of s^2, so no division per cell)
template <typename T>
__device__ __forceinline__ Geo<T> geo_frac(T ax, T ay, T az, T sx2, T sy2, T sz2, const InvS2<T>& is) {
    Geo<T> g;
    g.ax = ax; g.ay = ay; g.az = az;
    g.px = sx2 * ax * ax; g.py = sy2 * ay * ay; g.pz = sz2 * az * az;
    const T dxy = ax - ay, dxz = ax - az, dyz = ay - az;
    g.vxy = sx2 * sy2 * dxy * dxy * is.xy;
    g.vxz = sx2 * sz2 * dxz * dxz * is.xz;
    g.vyz = sy2 * sz2 * dyz * dyz * is.yz;
    g.vxyz = (sx2 * sy2 * dxy * dxy + sx2 * sz2 * dxz * dxz + sy2 * sz2 * dyz * dyz) * is.xyz;
    g.mxy = (sx2 * ax + sy2 * ay) * is.xy;
    g.mxz = (sx2 * ax + sz2 * az) * is.xz;
    g.myz = (sy2 * ay + sz2 * az) * is.yz;
    g.mxyz = (sx2 * ax + sy2 * ay + sz2 * az) * is.xyz;
    return g;
}

__device__ __forceinline__ float grids_thr(const GridsArgs& a, float dmax) { return a.thr * dmax; }

// First bound of a node: the nearest of the 8 vertices of its holding cell.
template <typename T>
__device__ __forceinline__ T grids_f0(const GridsArgs& a, const int c0[3], const T f[3], T dr, T inv_dd) {
    const T s2[3] = {(T)(a.eh[0] / a.dta) * (T)(a.eh[0] / a.dta), (T)(a.eh[1] / a.dta) * (T)(a.eh[1] / a.dta),
                     (T)(a.eh[2] / a.dta) * (T)(a.eh[2] / a.dta)};
    T best = Num<T>::inf();
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const int bz = (b >> 2) & 1, by = (b >> 1) & 1, bx = b & 1;
        const T dz = (T)bz - f[0], dy = (T)by - f[1], dx = (T)bx - f[2];
        const int64_t j = ((int64_t)(c0[0] + bz) * a.en[1] + (c0[1] + by)) * a.en[2] + (c0[2] + bx);
        const T gv = ((T)a.ev[j] - dr) * inv_dd;
        best = vmin<T>(best, s2[0] * dz * dz + s2[1] * dy * dy + s2[2] * dx * dx + gv * gv);
    }
    return best;
}

constexpr int GRIDS_MAX_ITEMS = 8;
__global__ __launch_bounds__(256) void k_grids_max(GridsArgs a, int64_t nr, int64_t ne) {
    float m = -Num<float>::inf();
    bool bad = false;
    const int64_t n = nr > ne ? nr : ne;
    // GRIDS_MAX_ITEMS nodes of each volume per thread and step, every load of a step issued
    // before the first use (indices clamped to the last node: the copies change neither the
    // maximum nor the finiteness check)
    constexpr int K = GRIDS_MAX_ITEMS;
    const int64_t step = (int64_t)gridDim.x * 256 * K;
    for (int64_t b0 = (int64_t)blockIdx.x * 256 * K; b0 < n; b0 += step) {
        float r[K], e[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t i = b0 + (int64_t)k * 256 + threadIdx.x;
            r[k] = a.ref[i < nr ? i : nr - 1];
            e[k] = a.ev[i < ne ? i : ne - 1];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            bad = bad || !isfinite(r[k]) || !isfinite(e[k]);
            m = fmaxf(m, r[k]);
        }
    }
    // one partial per block (an atomic maximum per wave on one address serialises: it took
    // 30-80 us); the listing kernel reduces the partials
    __shared__ uint32_t s_m[4];
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    __shared__ uint32_t s_bad[4];
    const bool wbad = __ballot(bad) != 0ull;
    if ((threadIdx.x & 63) == 0) {
        s_m[threadIdx.x >> 6] = m > -Num<float>::inf() ? float_to_ord(m) : 0u;
        s_bad[threadIdx.x >> 6] = wbad ? 1u : 0u;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.part[blockIdx.x] = max(max(s_m[0], s_m[1]), max(s_m[2], s_m[3]));
        a.part[MAX_BLOCKS + blockIdx.x] = s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3];
    }
    // the map's scalars and partial counts start at 0 (no other block touches them here)
    if (blockIdx.x == 0) {
        if (threadIdx.x < sizeof(Scalars) / sizeof(uint32_t)) reinterpret_cast<uint32_t*>(a.sc)[threadIdx.x] = 0u;
        for (int j = threadIdx.x; j < SUM_BINS; j += 256) a.sums[j] = BlockSums{};
    }
}

// Listing in chunks of 16 nodes per thread (4096 per block): one atomic per chunk on the
// list counter (one per 256 nodes would serialise on that address).
constexpr int GRIDS_PER_THREAD = 16;
__global__ __launch_bounds__(256) void k_grids_list(GridsArgs a, int64_t nr, int nb_max) {
    static_assert(GRIDS_PER_THREAD * 4 == 64, "one lane per (item, wave) count");
    __shared__ uint32_t s_wsum[4];
    __shared__ uint32_t s_cnt[64];
    // the dose maximum from k_grids_max's partials (every block reduces them itself)
    uint32_t dm = 0u, nonfinite = 0u;
    for (int j = threadIdx.x; j < nb_max; j += 256) {
        dm = max(dm, a.part[j]);
        nonfinite |= a.part[MAX_BLOCKS + j];
    }
    for (int o = 32; o > 0; o >>= 1) dm = max(dm, (uint32_t)__shfl_xor((int)dm, o));
    if ((threadIdx.x & 63) == 0) s_wsum[threadIdx.x >> 6] = dm;
    if (blockIdx.x == 0 && nonfinite != 0u) atomicOr(&a.sc->flags, FLAG_NONFINITE);
    __syncthreads();
    dm = max(max(s_wsum[0], s_wsum[1]), max(s_wsum[2], s_wsum[3]));
    __syncthreads();   // s_wsum is reused below
    const float dmax = ord_to_float(dm);
    const float thr_val = grids_thr(a, dmax);
    const float inv_dd_g = 1.0f / ((float)a.dd * dmax);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.sc->dmax_ord = dm;
        a.sc->thr_val = thr_val;
        a.sc->inv_dd = inv_dd_g;
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t chunk = 256 * GRIDS_PER_THREAD;
    // block-uniform trip count, so that every thread reaches the barriers
    for (int64_t b0 = (int64_t)blockIdx.x * chunk; b0 < nr; b0 += (int64_t)gridDim.x * chunk) {
        float F0[GRIDS_PER_THREAD], drs[GRIDS_PER_THREAD];
        uint32_t takes = 0u;
        // every reference load first, and the gamma = -1 stores after the chunk's loads: a
        // store between them (gamma may alias the doses, as far as the compiler knows) kept
        // each node's loads waiting for the previous node's
#pragma unroll
        for (int k = 0; k < GRIDS_PER_THREAD; ++k) {
            const int64_t r = b0 + threadIdx.x + 256 * k;
            drs[k] = a.ref[r < nr ? r : nr - 1];
        }
#pragma unroll
        for (int k = 0; k < GRIDS_PER_THREAD; ++k) {
            const int64_t r = b0 + threadIdx.x + 256 * k;
            F0[k] = 0.0f;
            if (r < nr) {
                const float dr = drs[k];
                double u[3];
                bool inside;
                grids_pos(a, (int)r, u, inside);
                if (dr >= thr_val && (!a.local || dr > 0.0f) && inside) {
                    int c0[3];
                    float f[3];
                    grids_cell<float>(a, u, c0, f);
                    F0[k] = grids_f0<float>(a, c0, f, dr, node_inv_dd(dr, inv_dd_g, (float)a.dd, a.local));
                    takes |= 1u << k;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < GRIDS_PER_THREAD; ++k) {
            const int64_t r = b0 + threadIdx.x + 256 * k;
            if (r < nr) a.gamma[r] = -1.0f;
        }
        // the chunk's nodes in grid order (neighbouring lanes of the later kernels then read
        // neighbouring doses): counts per (item, wave), their exclusive prefix, one atomic.
        // Listed thread by thread, neighbouring entries lay 256 nodes apart and a load of the
        // key-0 pass touched 52 cache lines: that pass 86 us, 70 in grid order.
#pragma unroll
        for (int k = 0; k < GRIDS_PER_THREAD; ++k) {
            const unsigned long long bal = __ballot((takes >> k) & 1u);
            if (lane == 0) s_cnt[k * 4 + w] = (uint32_t)__popcll(bal);
        }
        __syncthreads();
        if (w == 0) {
            const uint32_t c = s_cnt[lane];
            uint32_t incl = c;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t up = (uint32_t)__shfl_up((int)incl, o);
                if (lane >= o) incl += up;
            }
            uint32_t base = 0u;
            if (lane == 63 && incl != 0u) base = atomicAdd(&a.sc->n_masked, incl);
            base = (uint32_t)__shfl((int)base, 63);
            s_cnt[lane] = base + incl - c;
        }
        __syncthreads();
        uint32_t fb = 0u;
#pragma unroll
        for (int k = 0; k < GRIDS_PER_THREAD; ++k) {
            const unsigned long long bal = __ballot((takes >> k) & 1u);
            if ((takes >> k) & 1u) {
                const uint32_t pos = s_cnt[k * 4 + w] + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
                a.list[pos] = (uint32_t)(b0 + threadIdx.x + 256 * k);
                a.f0[pos] = F0[k];
                fb = max(fb, f2u(F0[k]));
            }
        }
        // the largest first bound: one atomic per block and chunk, only while it can raise it
        for (int o = 32; o > 0; o >>= 1) fb = max(fb, (uint32_t)__shfl_xor((int)fb, o));
        if (lane == 0) s_wsum[w] = fb;
        __syncthreads();
        if (threadIdx.x == 0) {
            fb = max(max(s_wsum[0], s_wsum[1]), max(s_wsum[2], s_wsum[3]));
            if (fb > __atomic_load_n(&a.sc->r2_bits, __ATOMIC_RELAXED)) atomicMax(&a.sc->r2_bits, fb);
        }
        __syncthreads();   // s_wsum is reused by the next chunk
    }
}

// Whether the cell at offset (ax, ay, az) from the holding cell can still lower F.  The node
// (at f inside the holding cell) is at least the cell's geometric distance from it, and the
// PL dose inside the cell lies between its vertex values, so when those share a sign the
// cell is at least dist^2 + (smallest |g|)^2 away.  A cell at or above F (1 + 2^-8) is
// skipped: the margin is far above the rounding of the projections, so it could not have
// lowered F either.  The bound needs no projection, so the guard judges only the cells that
// are projected: a skipped cell's conditioning cannot change the result.
__device__ __forceinline__ bool grids_need(const float* g, float ax, float ay, float az, const float* f, float sx2,
                                           float sy2, float sz2, float F) {
    float gmin = g[0], gmax = g[0];
#pragma unroll
    for (int b = 1; b < 8; ++b) {
        gmin = vmin<float>(gmin, g[b]);
        gmax = __builtin_fmaxf(gmax, g[b]);
    }
    const float m = gmin > 0.0f ? gmin : (gmax < 0.0f ? -gmax : 0.0f);
    // distance from f to the interval [a, a + 1], per axis
    const float dx = __builtin_fmaxf(__builtin_fmaxf(0.0f, ax - f[2]), f[2] - ax - 1.0f);
    const float dy = __builtin_fmaxf(__builtin_fmaxf(0.0f, ay - f[1]), f[1] - ay - 1.0f);
    const float dz = __builtin_fmaxf(__builtin_fmaxf(0.0f, az - f[0]), f[0] - az - 1.0f);
    const float lb = ((sx2 * dx * dx + sy2 * dy * dy) + sz2 * dz * dz) + m * m;
    return lb < F + F * 0x1p-8f;
}

// The counts of a block of 256 threads (every thread calls): summed over its waves in LDS and
// added with one atomic per count.  An atomic per wave on these few addresses serialises.
__device__ __forceinline__ void grids_counts(Scalars* sc, uint32_t npass, uint32_t nborder, unsigned long long cells,
                                             uint32_t gm) {
    __shared__ unsigned long long s_c[4];
    __shared__ uint32_t s_p[4], s_b[4], s_g[4];
    for (int o = 32; o > 0; o >>= 1) {
        npass += (uint32_t)__shfl_xor((int)npass, o);
        nborder += (uint32_t)__shfl_xor((int)nborder, o);
        gm = max(gm, (uint32_t)__shfl_xor((int)gm, o));
        cells += (unsigned long long)__shfl_xor((long long)cells, o);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_p[w] = npass;
        s_b[w] = nborder;
        s_g[w] = gm;
        s_c[w] = cells;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        npass = s_p[0] + s_p[1] + s_p[2] + s_p[3];
        nborder = s_b[0] + s_b[1] + s_b[2] + s_b[3];
        gm = max(max(s_g[0], s_g[1]), max(s_g[2], s_g[3]));
        cells = s_c[0] + s_c[1] + s_c[2] + s_c[3];
        if (npass) atomicAdd(&sc->n_pass, (unsigned long long)npass);
        if (nborder) atomicAdd(&sc->n_border, (unsigned long long)nborder);
        if (cells) atomicAdd(&sc->n_cells, cells);
        if (gm) atomicMax(&sc->maxg2_bits, gm);
    }
}

// A listed node as the lanes that project its cells read it.
struct alignas(16) GridsNode {
    int cz, cy, cx, r;       // holding cell, reference node
    float fz, fy, fx, dr;    // position in that cell, reference dose
    float inv_dd;
    uint32_t f;              // F (non-negative float bits)
    float f_start;           // and what the pass began with
    uint32_t pad;
};
// The evaluation grid's normalised spacings squared and their chain-block reciprocals.
struct GridsGeo {
    float sx2, sy2, sz2;
    InvS2<float> is;
};
__device__ __forceinline__ GridsGeo grids_geo(const GridsArgs& a) {
    GridsGeo q;
    q.sx2 = (float)((a.eh[2] / a.dta) * (a.eh[2] / a.dta));
    q.sy2 = (float)((a.eh[1] / a.dta) * (a.eh[1] / a.dta));
    q.sz2 = (float)((a.eh[0] / a.dta) * (a.eh[0] / a.dta));
    q.is = inv_s2<float>(q.sx2, q.sy2, q.sz2);
    return q;
}
__device__ __forceinline__ GridsNode grids_node(const GridsArgs& a, int r, float dr, float F, float inv_dd_g) {
    double u[3];
    bool inside;
    grids_pos(a, r, u, inside);
    int c0[3];
    float f[3];
    grids_cell<float>(a, u, c0, f);
    return GridsNode{c0[0], c0[1], c0[2], r, f[0], f[1], f[2], dr, node_inv_dd(dr, inv_dd_g, (float)a.dd, a.local), f2u(F),
                     F, 0u};
}
// dist^2 to the faces of the cell at offset (az, ay, ax) from the node's holding cell (a cell
// whose lower corner lies on the grid; mask: some lane's cell is cut by the grid's faces).
__device__ __forceinline__ float grids_project(const GridsArgs& a, const GridsGeo& q, const GridsNode& n, int az, int ay,
                                               int ax, bool okx, bool oky, bool okz, bool mask) {
    const int enx = a.en[2], esxy = enx * a.en[1];
    const int64_t b = (int64_t)(n.cz + az) * esxy + (int64_t)(n.cy + ay) * enx + (n.cx + ax);
    float g[8];
    cell_corners<3>(a.ev, b, okx, oky ? enx : 0, okz ? esxy : 0, g);
#pragma unroll
    for (int k = 0; k < 8; ++k) g[k] = dose_norm<float>(g[k], n.dr, n.inv_dd);
    const Geo<float> G = geo_frac<float>((float)ax - n.fx, (float)ay - n.fy, (float)az - n.fz, q.sx2, q.sy2, q.sz2, q.is);
    GuardCtx gc{};
    uint32_t n_fp64 = 0;
    bool ill = false;
    if (mask) return cell3<float, true, 0>(g, G, q.is, okx, oky, okz, a.den_guard, gc, n_fp64, ill);
    return cell3<float, false, 0>(g, G, q.is, true, true, true, a.den_guard, gc, n_fp64, ill);
}
// Whether the whole cell with lower corner (cz, cy, cx) holds an ill-conditioned tetrahedron.
__device__ __forceinline__ bool grids_ill(const GridsArgs& a, const GridsGeo& q, const GridsNode& n, int cz, int cy, int cx) {
    const int enx = a.en[2], esxy = enx * a.en[1];
    const int64_t b = (int64_t)cz * esxy + (int64_t)cy * enx + cx;
    float g[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        g[k] = dose_norm<float>(a.ev[b + (k & 1) + ((k >> 1) & 1) * enx + (k >> 2) * esxy], n.dr, n.inv_dd);
    return tets_ill(g, q.is, a.den_guard);
}

// The queued passes below project a node's cells in another order than one lane per node (or a
// group of lanes, batch by batch) would, and more or fewer of them, depending on which nodes
// share the wave; so a node that met an ill-conditioned tetrahedron in any whole cell (rare) is
// judged by that order again.
// The cell at offset (az, ay, ax) in it: dist^2 to its faces if it can still lower F (its
// tetrahedra are judged then), else infinity.
__device__ __forceinline__ float grids_judge(const GridsArgs& a, const GridsGeo& q, const GridsNode& n, int az, int ay,
                                             int ax, float F, bool& ill) {
    const int enx = a.en[2], eny = a.en[1], enz = a.en[0], esxy = enx * eny;
    const int cz = n.cz + az, cy = n.cy + ay, cx = n.cx + ax;
    if ((unsigned)cx >= (unsigned)enx || (unsigned)cy >= (unsigned)eny || (unsigned)cz >= (unsigned)enz)
        return Num<float>::inf();
    const bool okx = cx + 1 < enx, oky = cy + 1 < eny, okz = cz + 1 < enz;
    float g[8];
    cell_corners<3>(a.ev, (int64_t)cz * esxy + (int64_t)cy * enx + cx, okx, oky ? enx : 0, okz ? esxy : 0, g);
#pragma unroll
    for (int k = 0; k < 8; ++k) g[k] = dose_norm<float>(g[k], n.dr, n.inv_dd);
    const float f[3] = {n.fz, n.fy, n.fx};
    if (!grids_need(g, (float)ax, (float)ay, (float)az, f, q.sx2, q.sy2, q.sz2, F)) return Num<float>::inf();
    const Geo<float> G = geo_frac<float>((float)ax - n.fx, (float)ay - n.fy, (float)az - n.fz, q.sx2, q.sy2, q.sz2, q.is);
    GuardCtx gc{};
    uint32_t n_fp64 = 0;
    return cell3<float, true, 1>(g, G, q.is, okx, oky, okz, a.den_guard, gc, n_fp64, ill);
}
// The walk past the key-0 cells by batches of 16 rows (the 8 lanes of a group, two rows each).
__device__ __forceinline__ bool grids_judge_walk(const GridsArgs& a, const GridsGeo& q, const GridsNode& n, float F,
                                                 int first, int gl) {
    bool ill = false;
#pragma unroll 1
    for (int n0 = first; n0 < a.tab_len && a.tab[n0].key2 < F; n0 += 16) {
        float c = Num<float>::inf();
#pragma unroll 1
        for (int r = n0 + gl; r < n0 + 16 && r < a.tab_len; r += 8) {
            const int4 e = *reinterpret_cast<const int4*>(&a.tab[r]);   // key^2 and offset
            if (__builtin_bit_cast(float, e.x) < F) c = vmin<float>(c, grids_judge(a, q, n, e.w, e.z, e.y, F, ill));
        }
        for (int o = 4; o > 0; o >>= 1) c = vmin<float>(c, __shfl_xor(c, o));
        F = vmin<float>(F, c);
    }
    for (int o = 4; o > 0; o >>= 1) ill = (__shfl_xor((int)ill, o) != 0) || ill;
    return ill;
}

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// The 27 key-0 cells (offsets a in {-1,0,1}^3 from the holding cell) of every listed node, one
// lane per node: the holding cell is projected first; the others are tested by their exact
// distance and the range of their corner doses (from the 4 x 4 x 4 evaluation neighbourhood,
// read plane by plane, clamped at the grid's faces), and those that can still lower F are
// queued in LDS and projected 64 at a time, whichever nodes they belong to.  A node whose
// bound is then at most k1 is finished; the others go to the tail list.  Which of a wave's 64
// nodes need a cell differs, so projecting it whenever one does took the 27 cells' time for
// the few that each node needs: 434 thousand nodes on a grid of half the spacing 129 us, now
// 66-72 (4200 instructions of a wave, half of its time; three waves per SIMD, which four with
// 52 spilled registers do not beat: 95 against 86 us before the list was in grid order).
//
// A neighbourhood whose doses span too little for an ill-conditioned tetrahedron needs no
// judgement, nor does one whose whole cells hold none; the others are judged cell by cell.
//
// FAR: the first bound of some node may have overflowed (doses more than 1e19 dD apart, as tails of a
// dose under local normalisation without a threshold).  Projections of such doses mean little, so which
// of a node's cells are projected shows: nodes with such a bound or neighbourhood take them one
// after the other, while they can still lower F.
template <int GMODE, bool FAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_grids_zero(GridsArgs a) {
    __shared__ GridsNode s_node[256];
    __shared__ uint16_t s_item[4][26 * 64];   // queued cells: node's lane | cell << 6
    const uint32_t M = a.sc->n_masked;
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x * 256 >= M) return;   // uniform
    const bool live = i < M;
    const int lane = threadIdx.x & 63;
    const int r = (int)a.list[live ? i : 0u];
    GridsNode* wnode = s_node + (threadIdx.x & ~63u);
    uint16_t* item = s_item[threadIdx.x >> 6];
    const GridsGeo q = grids_geo(a);
    GridsNode n = grids_node(a, r, a.ref[r], live ? a.f0[i] : 0.0f, a.sc->inv_dd);
    const int enx = a.en[2], eny = a.en[1], enz = a.en[0];
    // per axis: does the cell at -1 exist, is the cell at +1 whole
    const bool lox = n.cx > 0, loy = n.cy > 0, loz = n.cz > 0;
    const bool hix = n.cx + 2 < enx, hiy = n.cy + 2 < eny, hiz = n.cz + 2 < enz;
    bool far = FAR && live && !(n.f_start < Num<float>::inf());
    {
        const float c = grids_project(a, q, n, 0, 0, 0, true, true, true, false);
        n.f = f2u(live && !far ? vmin<float>(u2f(n.f), c) : u2f(n.f));
    }
    wnode[lane] = n;
    const float Fm = u2f(n.f) + u2f(n.f) * 0x1p-8f;

    // squared distance of the cells at -1 and +1 per axis
    const float dxl = q.sx2 * (n.fx * n.fx), dxh = q.sx2 * ((1.0f - n.fx) * (1.0f - n.fx));
    const float dyl = q.sy2 * (n.fy * n.fy), dyh = q.sy2 * ((1.0f - n.fy) * (1.0f - n.fy));
    const float dzl = q.sz2 * (n.fz * n.fz), dzh = q.sz2 * ((1.0f - n.fz) * (1.0f - n.fz));
    auto cl = [](int v, int m) { return v < 0 ? 0 : (v > m - 1 ? m - 1 : v); };
    const bool rows4 = __ballot(!(lox && hix)) == 0ull;   // no lane's row is clamped along x
    uint32_t nq = 0;
    float all_lo = Num<float>::inf(), all_hi = -Num<float>::inf();
    float plo[9], phi[9];   // ranges of the 3 x 3 squares of the plane before
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float v[16];
        const int64_t zb = (int64_t)cl(n.cz - 1 + p, enz) * eny;
        if (rows4) {   // a row's four doses in one load
#pragma unroll
            for (int dy = 0; dy < 4; ++dy) {
                const f32x4u t = *reinterpret_cast<const f32x4u*>(a.ev + (zb + cl(n.cy - 1 + dy, eny)) * enx + (n.cx - 1));
                v[dy * 4] = t.x;
                v[dy * 4 + 1] = t.y;
                v[dy * 4 + 2] = t.z;
                v[dy * 4 + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int dy = 0; dy < 4; ++dy)
#pragma unroll
                for (int dx = 0; dx < 4; ++dx)
                    v[dy * 4 + dx] = a.ev[(zb + cl(n.cy - 1 + dy, eny)) * enx + cl(n.cx - 1 + dx, enx)];
        }
        float clo[9], chi[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int b = (k / 3) * 4 + k % 3;
            clo[k] = vmin<float>(vmin<float>(v[b], v[b + 1]), vmin<float>(v[b + 4], v[b + 5]));
            chi[k] = vmax<float>(vmax<float>(v[b], v[b + 1]), vmax<float>(v[b + 4], v[b + 5]));
        }
        if (p > 0) {
            const int az = p - 2;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int ay = k / 3 - 1, ax = k % 3 - 1;
                if (az == 0 && ay == 0 && ax == 0) continue;
                const float lo = dose_norm<float>(vmin<float>(plo[k], clo[k]), n.dr, n.inv_dd);
                const float hi = dose_norm<float>(vmax<float>(phi[k], chi[k]), n.dr, n.inv_dd);
                if (GMODE == 1 || FAR) {
                    all_lo = vmin<float>(all_lo, lo);
                    all_hi = vmax<float>(all_hi, hi);
                }
                const float m = vmax<float>(vmax<float>(lo, -hi), 0.0f);
                const float d = (ax < 0 ? dxl : (ax > 0 ? dxh : 0.0f)) + (ay < 0 ? dyl : (ay > 0 ? dyh : 0.0f)) +
                                (az < 0 ? dzl : (az > 0 ? dzh : 0.0f));
                const bool there = (ax >= 0 || lox) && (ay >= 0 || loy) && (az >= 0 || loz);
                const bool need = live && !far && there && fmadd(m, m, d) < Fm;
                const unsigned long long mask = __ballot(need);
                if (need)
                    item[nq + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] =
                        (uint16_t)(lane | (((az + 1) * 9 + k) << 6));
                nq += (uint32_t)__popcll(mask);
            }
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            plo[k] = clo[k];
            phi[k] = chi[k];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
    for (uint32_t h = 0; h < nq; h += 64) {
        const bool on = h + lane < nq;
        const uint32_t it = on ? item[h + lane] : (uint32_t)(13u << 6);
        const GridsNode o = wnode[it & 63u];
        const int c = (int)(it >> 6), az = c / 9 - 1, ay = (c / 3) % 3 - 1, ax = c % 3 - 1;
        const bool okx = o.cx + ax + 1 < enx, oky = o.cy + ay + 1 < eny, okz = o.cz + az + 1 < enz;
        const bool mask = __ballot(on && !(okx && oky && okz)) != 0ull;
        if (on) {
            const float v = grids_project(a, q, o, az, ay, ax, okx, oky, okz, mask);
            atomicMin(&wnode[it & 63u].f, f2u(v));
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float F = u2f(wnode[lane].f);
    bool ill = false;
    if constexpr (FAR) {
        far = far || (live && !((all_hi - all_lo) * (all_hi - all_lo) * ((q.is.x + q.is.y) + q.is.z) < Num<float>::inf()));
        if (far) {
            const GridsNode o = wnode[lane];
            F = o.f_start;
#pragma unroll 1
            for (int c = 0; c < 27; ++c)
                F = vmin<float>(F, grids_judge(a, q, o, c / 9 - 1, (c / 3) % 3 - 1, c % 3 - 1, F, ill));
        }
    }
    if (GMODE == 1) {
        const bool suspect = live && !far && !((all_hi - all_lo) * (all_hi - all_lo) <
                                       (a.den_guard * 0.999f - 1.0f) / ((q.is.x + q.is.y) + q.is.z));
        if (__ballot(suspect) != 0ull && suspect) {   // rare
            const GridsNode o = wnode[lane];   // (read again: the node's registers are free by now)
            bool any = false;
#pragma unroll 1
            for (int c = 0; c < 27 && !any; ++c) {
                const int cz = o.cz + c / 9 - 1, cy = o.cy + (c / 3) % 3 - 1, cx = o.cx + c % 3 - 1;
                if (cz >= 0 && cy >= 0 && cx >= 0 && cz + 1 < enz && cy + 1 < eny && cx + 1 < enx)
                    any = grids_ill(a, q, o, cz, cy, cx);
            }
            float f = o.f_start;
#pragma unroll 1
            for (int c = 0; c < 27 && any; ++c)
                f = vmin<float>(f, grids_judge(a, q, o, c / 9 - 1, (c / 3) % 3 - 1, c % 3 - 1, f, ill));
        }
    }
    const bool to_guard = GMODE == 1 && ill;
    const bool to_tail = live && !to_guard && F > a.k1;
    const uint32_t cells = (1u + lox + hix) * (1u + loy + hiy) * (1u + loz + hiz);
    zero_epilogue(a, a.sums, blockIdx.x, live, r, F, f2u(F), 0u, cells, to_tail, to_guard, true);
}

// The walk of the tail list in the automatic layout: the scan, pooled projections and finish of
// tail_queue_body, for nodes between the evaluation grid's nodes.  A row's test takes the exact
// distance of its cell (the key is its least over the holding cell) and the range of its
// corner doses; visited cells are those of the rows below the final F.  40 us at 36 thousand
// nodes where 16 lanes per node take 68 (46 with the table in memory and the finished counts in
// registers).  It is taken where grids_queued says so: its steps are heavier, so one long walk
// outlasts 16 lanes.
template <int GMODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_grids_tail(GridsArgs a) {
    constexpr int FIRST = 27;   // rows of the key-0 cells
    __shared__ GridsNode s_node[TQ_GROUPS];
    __shared__ TqCounts s_counts[TQ_GROUPS];   // kept by the group's first lane
    __shared__ uint2 s_queue[4][TQ_RING];      // row | group of the wave << 28, bound
    __shared__ int4 s_head[TQ_TAB];            // key^2 and offset of the first rows of a walk
    const uint32_t M = a.sc->n_tail;
    const int lane = threadIdx.x & 63, gl = lane & (TQ_LANES - 1), gsh = lane & ~(TQ_LANES - 1);
    const unsigned long long gmask = (1ull << TQ_LANES) - 1ull;
    uint2* queue = s_queue[threadIdx.x >> 6];
    GridsNode* wnode = s_node + (threadIdx.x >> 6) * (WAVE / TQ_LANES);
    GridsNode& self = wnode[lane / TQ_LANES];
    TqCounts& counts = s_counts[threadIdx.x / TQ_LANES];
    const float inv_dd_g = a.sc->inv_dd;
    const GridsGeo q = grids_geo(a);
    const int enx = a.en[2], eny = a.en[1], enz = a.en[0];
    const float ill_span2 = (a.den_guard * 0.999f - 1.0f) / ((q.is.x + q.is.y) + q.is.z);
    auto row_head = [&](int n) -> int4 {   // key^2 (infinite past the table) and offset
        if (n < FIRST + TQ_TAB) return s_head[n - FIRST];
        return n < a.tab_len ? *reinterpret_cast<const int4*>(&a.tab[n]) : make_int4(0x7F800000, 0, 0, 0);
    };
    uint32_t i = blockIdx.x * TQ_GROUPS + threadIdx.x / TQ_LANES;
    const uint32_t stride = gridDim.x * TQ_GROUPS;
    if (blockIdx.x * TQ_GROUPS >= M) return;   // uniform
    if (gl == 0) {
        self = GridsNode{};
        counts = TqCounts{};
    }
    if (threadIdx.x < TQ_TAB) {
        const int n = FIRST + (int)threadIdx.x;
        s_head[threadIdx.x] = n < a.tab_len ? *reinterpret_cast<const int4*>(&a.tab[n]) : make_int4(0x7F800000, 0, 0, 0);
    }
    __syncthreads();
    bool have = false, done = false;
    int n0 = FIRST;
    uint32_t q_head = 0, q_tail = 0, q_last = 0, lane_cells = 0, whole = 0;
    bool steep = false;   // a whole cell of this lane's rows holds an ill-conditioned tetrahedron

    for (;;) {
        if (!have && i < M) {
            const int r = (int)a.tail_list[i];
            const float f = a.tail_f[i], dr = a.ref[r];
            if (gl == 0) self = grids_node(a, r, dr, f, inv_dd_g);
            n0 = FIRST;
            q_last = q_head;
            lane_cells = whole = 0u;
            steep = false;
            have = true;
            done = false;
            i += stride;
        }
        if (__ballot(have) == 0ull) break;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

        // scan
        if (q_tail - q_head < WAVE && __ballot(have && !done) != 0ull) {
            const bool scan = have && !done;
            const GridsNode nd = self;
            const float F = u2f(nd.f), Fm = F + F * 0x1p-8f;
            bool past = false;
            if (scan) {
                lane_cells += __popc(whole);
                whole = 0u;
            }
            float lb[TQ_ROWS];
            uint32_t work = 0u, before = q_tail;
            bool suspect = false;
            float v[TQ_ROWS][8];
#pragma unroll
            for (int k = 0; k < TQ_ROWS; ++k) {
                lb[k] = 0.0f;
#pragma unroll
                for (int b = 0; b < 8; ++b) v[k][b] = 0.0f;
                if (scan) {
                    const int4 e = row_head(n0 + k * TQ_LANES + gl);
                    const float key = __builtin_bit_cast(float, e.x);
                    const int cx = nd.cx + e.y, cy = nd.cy + e.z, cz = nd.cz + e.w;
                    const bool in = (unsigned)cx < (unsigned)enx && (unsigned)cy < (unsigned)eny &&
                                    (unsigned)cz < (unsigned)enz && key < F;
                    const bool okx = cx + 1 < enx, oky = cy + 1 < eny, okz = cz + 1 < enz;
                    past = past || !(key < F);
                    if (in) {
                        work |= 1u << k;
                        whole |= okx && oky && okz ? (1u << k) : 0u;
                        const int64_t b = ((int64_t)cz * eny + cy) * enx + cx;
                        cell_corners<3>(a.ev, b, okx, oky ? enx : 0, okz ? enx * eny : 0, v[k]);
                        const float x = (float)e.y - nd.fx, y = (float)e.z - nd.fy, z = (float)e.w - nd.fz;
                        const float dx = vmax<float>(vmax<float>(x, -x - 1.0f), 0.0f);
                        const float dy = vmax<float>(vmax<float>(y, -y - 1.0f), 0.0f);
                        const float dz = vmax<float>(vmax<float>(z, -z - 1.0f), 0.0f);
                        lb[k] = (q.sx2 * (dx * dx) + q.sy2 * (dy * dy)) + q.sz2 * (dz * dz);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < TQ_ROWS; ++k) {
                float lo = v[k][0], hi = v[k][0];
#pragma unroll
                for (int b = 1; b < 8; ++b) {
                    lo = vmin<float>(lo, v[k][b]);
                    hi = vmax<float>(hi, v[k][b]);
                }
                lo = dose_norm<float>(lo, nd.dr, nd.inv_dd);
                hi = dose_norm<float>(hi, nd.dr, nd.inv_dd);
                const float m = vmax<float>(vmax<float>(lo, -hi), 0.0f);
                lb[k] = fmadd(m, m, lb[k]);
                const bool need = ((work >> k) & 1u) && lb[k] < Fm;
                if (GMODE == 1) suspect = suspect || (((whole >> k) & 1u) && !((hi - lo) * (hi - lo) < ill_span2));
                const unsigned long long mask = __ballot(need);
                if (need)
                    queue[(q_tail + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))) &
                          (TQ_RING - 1)] =
                        make_uint2((uint32_t)(n0 + k * TQ_LANES + gl) | ((uint32_t)(lane / TQ_LANES) << 28), f2u(lb[k]));
                q_tail += (uint32_t)__popcll(mask);
            }
            if (GMODE == 1 && __ballot(scan && suspect) != 0ull && scan) {   // rare
#pragma nounroll
                for (int k = 0; k < TQ_ROWS; ++k) {
                    if (!((whole >> k) & 1u)) continue;
                    const int4 e = row_head(n0 + k * TQ_LANES + gl);
                    steep = steep || grids_ill(a, q, nd, nd.cz + e.w, nd.cy + e.z, nd.cx + e.y);
                }
            }
            const unsigned long long pb = __ballot(past);
            if (scan) {
                n0 += TQ_STEP;
                done = ((pb >> gsh) & gmask) != 0ull;
                if (q_tail != before) q_last = q_tail;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

        // project
        const uint32_t queued = q_tail - q_head;
        if (queued >= WAVE || (queued > 0u && __popcll(__ballot(have && !done)) <= TQ_FEW * TQ_LANES)) {
            const uint32_t take = queued < WAVE ? queued : WAVE;
            const uint2 it = queue[(q_head + lane) & (TQ_RING - 1)];
            GridsNode* owner = &wnode[(it.x >> 28) & 7u];
            const GridsNode nd = *owner;
            const float F = u2f(nd.f);
            const bool proj = (uint32_t)lane < take && u2f(it.y) < F + F * 0x1p-8f;
            const int4 e = row_head(proj ? (int)(it.x & 0x0FFFFFFFu) : FIRST);
            const bool okx = nd.cx + e.y + 1 < enx, oky = nd.cy + e.z + 1 < eny, okz = nd.cz + e.w + 1 < enz;
            const bool mask = __ballot(proj && !(okx && oky && okz)) != 0ull;
            if (proj) atomicMin(&owner->f, f2u(grids_project(a, q, nd, e.w, e.z, e.y, okx, oky, okz, mask)));
            q_head += take;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }

        // finish
        const bool fin = have && done && (int32_t)(q_head - q_last) >= 0;
        if (__ballot(fin) != 0ull) {
            const GridsNode nd = self;
            const float F = u2f(nd.f);
            if (fin) {
#pragma unroll
                for (int k = 0; k < TQ_ROWS; ++k)
                    if ((whole >> k) & 1u)
                        lane_cells += __builtin_bit_cast(float, row_head(n0 - TQ_STEP + k * TQ_LANES + gl).x) < F ? 1u : 0u;
                for (int s0 = n0 - TQ_STEP;
                     s0 > FIRST && !(__builtin_bit_cast(float, row_head(s0 - 1).x) < F); s0 -= TQ_STEP) {
#pragma unroll
                    for (int k = 0; k < TQ_ROWS; ++k) {
                        const int4 e = row_head(s0 - TQ_STEP + k * TQ_LANES + gl);
                        const int cx = nd.cx + e.y, cy = nd.cy + e.z, cz = nd.cz + e.w;
                        const bool w = cx >= 0 && cx + 1 < enx && cy >= 0 && cy + 1 < eny && cz >= 0 && cz + 1 < enz;
                        lane_cells -= w && !(__builtin_bit_cast(float, e.x) < F) ? 1u : 0u;
                    }
                }
            }
            const uint32_t sum = sum8(lane_cells);
            bool to_guard = false;
            if (GMODE == 1) {
                const unsigned long long sb = __ballot(fin && steep);
                if (sb != 0ull && ((sb >> gsh) & gmask) != 0ull)   // rare
                    to_guard = grids_judge_walk(a, q, nd, nd.f_start, FIRST, gl);
            }
            const bool put = fin && to_guard && gl == 0;
            if (fin) {
                if (gl == 0 && !to_guard) {
                    const float gam = sqrtf(F);
                    a.gamma[nd.r] = gam;
                    TqCounts c = counts;
                    c.pass += gam <= 1.0f;
                    c.border += fabsf(gam - 1.0f) <= 1e-5f;
                    c.maxg2 = max(c.maxg2, f2u(gam * gam));
                    c.cells += sum;
                    counts = c;
                }
                have = false;
            }
            if (GMODE == 1) {
                const unsigned long long gb = __ballot(put);
                if (gb != 0ull) {   // rare: one atomic per wave
                    uint32_t base = 0u;
                    if (lane == 0) base = atomicAdd(&a.sc->n_guard, (uint32_t)__popcll(gb));
                    base = (uint32_t)__shfl((int)base, 0);
                    if (put) a.guard_list[base + (uint32_t)__popcll(gb & ((1ull << lane) - 1ull))] = (uint32_t)nd.r;
                }
            }
        }
    }
    TqCounts c{};
    if (gl == 0) c = counts;
    // the longest walk of the wave, where long: the context's next map chooses its layout by it
    if (FIRST + (int)LONG_WALK_ROWS < a.tab_len) {
        uint32_t f = c.maxg2;
        for (int o = WAVE / 2; o > 0; o >>= 1) f = max(f, (uint32_t)__shfl_xor((int)f, o));
        if (lane == 0 && a.tab[FIRST + LONG_WALK_ROWS].key2 < u2f(f))
            atomicMax(&a.sc->long_rows, (uint32_t)(resume_row(a.tab, a.tab_len, FIRST, u2f(f)) - FIRST));
    }
    block_sums(a.sums, blockIdx.x, c.pass, c.border, 0u, c.cells, c.maxg2);
}

// G lanes per node walk the lower-key table of the evaluation grid.  LIST 0: the listed nodes
// from row 0 (FP64 maps); 1: the guard list (FP64) from row 0; 2: the tail list of the key-0
// pass from the first row past the key-0 cells.  below: count the visited cells below the final
// F (as the queued walk does: the automatic layout's count does not depend on which of the two it
// takes), not those that the node's last batch visited past it.
template <typename T, int GMODE, int LIST>
__global__ __launch_bounds__(256) void k_grids_walk(GridsArgs a, int G, bool below) {
    static_assert((LIST == 2) == (sizeof(T) == 4), "FP32 walks the tail list, FP64 the others");
    const uint32_t M = LIST == 1 ? a.sc->n_guard : (LIST == 2 ? a.sc->n_tail : a.sc->n_masked);
    if (M == 0u) return;   // (the guard list, as a rule)
    const uint32_t* list = LIST == 1 ? a.guard_list : (LIST == 2 ? a.tail_list : a.list);
    const int first = LIST == 2 ? 27 : 0;
    const int GROUPS = 256 / G;
    const int gl = threadIdx.x % G;
    const double dmax = (double)ord_to_float(a.sc->dmax_ord);
    const float inv_dd_g = a.sc->inv_dd;
    const T sx2 = (T)((a.eh[2] / a.dta) * (a.eh[2] / a.dta)), sy2 = (T)((a.eh[1] / a.dta) * (a.eh[1] / a.dta)),
            sz2 = (T)((a.eh[0] / a.dta) * (a.eh[0] / a.dta));
    const InvS2<T> is = inv_s2<T>(sx2, sy2, sz2);
    const int enx = a.en[2], eny = a.en[1], enz = a.en[0], esxy = enx * eny;
    uint32_t npass = 0, nborder = 0, gm = 0, n_fp64 = 0;
    unsigned long long cells = 0;
    GuardCtx gc{};
    for (uint64_t base = (uint64_t)blockIdx.x * GROUPS; base < M; base += (uint64_t)gridDim.x * GROUPS) {
        const uint32_t i = (uint32_t)base + threadIdx.x / G;
        const bool live = i < M;
        const int r = live ? (int)list[i] : 0;
        double u[3];
        bool inside;
        grids_pos(a, r, u, inside);
        int c0[3];
        T f[3];
        grids_cell<T>(a, u, c0, f);
        const float dr32 = a.ref[r];
        const T dr = (T)dr32;
        T inv_dd;
        if constexpr (sizeof(T) == 8)
            inv_dd = a.local ? (T)(1.0 / (a.dd * (double)dr32)) : (T)(1.0 / (a.dd * dmax));
        else
            inv_dd = (T)node_inv_dd(dr32, inv_dd_g, (float)a.dd, a.local);
        T F = T(0);
        if (live) {
            if constexpr (LIST == 2) F = (T)a.tail_f[i];
            else F = grids_f0<T>(a, c0, f, dr, inv_dd);
        }
        uint32_t lane_cells = 0, rows = 0;
        T last_key = T(0);   // of this lane's last whole cell: its only one that may lie past the final F
        bool ill = false;
        for (int n0 = first; n0 < a.tab_len; n0 += G) {
            const bool grp_act = live && (T)a.tab[n0].key2 < F;
            if (__ballot(grp_act) == 0ull) break;
            if constexpr (LIST == 2) rows += grp_act ? (uint32_t)G : 0u;
            const int n = n0 + gl;
            TabEntry e;
            bool act = false;
            if (grp_act && n < a.tab_len) {
                e = a.tab[n];
                act = (T)e.key2 < F;
            }
            int cz = 0, cy = 0, cx = 0;
            if (act) {
                cz = c0[0] + e.az;
                cy = c0[1] + e.ay;
                cx = c0[2] + e.ax;
            }
            const bool cin = (unsigned)cx < (unsigned)enx && (unsigned)cy < (unsigned)eny && (unsigned)cz < (unsigned)enz;
            const bool okx = cx + 1 < enx, oky = cy + 1 < eny, okz = cz + 1 < enz;
            const bool work = act && cin;
            const bool edge = !(okx && oky && okz);
            const bool wave_masked = __ballot(work && edge) != 0ull;
            T c = Num<T>::inf();
            T g[8];
            bool need = false;
            if (work) {
                lane_cells += edge ? 0u : 1u;
                if constexpr (LIST == 2) last_key = edge ? last_key : (T)e.key2;
                const int64_t b = (int64_t)cz * esxy + (int64_t)cy * enx + cx;
                const int ox = okx ? 1 : 0, oy = oky ? enx : 0, oz = okz ? esxy : 0;
                g[0] = dose_norm<T>((T)a.ev[b], dr, inv_dd);
                g[1] = dose_norm<T>((T)a.ev[b + ox], dr, inv_dd);
                g[2] = dose_norm<T>((T)a.ev[b + oy], dr, inv_dd);
                g[3] = dose_norm<T>((T)a.ev[b + oy + ox], dr, inv_dd);
                g[4] = dose_norm<T>((T)a.ev[b + oz], dr, inv_dd);
                g[5] = dose_norm<T>((T)a.ev[b + oz + ox], dr, inv_dd);
                g[6] = dose_norm<T>((T)a.ev[b + oz + oy], dr, inv_dd);
                g[7] = dose_norm<T>((T)a.ev[b + oz + oy + ox], dr, inv_dd);
                need = true;
                if constexpr (sizeof(T) == 4) need = grids_need(g, (float)e.ax, (float)e.ay, (float)e.az, f, sx2, sy2, sz2, F);
            }
            if (__ballot(need) != 0ull && need) {
                const Geo<T> Gm = geo_frac<T>((T)e.ax - f[2], (T)e.ay - f[1], (T)e.az - f[0], sx2, sy2, sz2, is);
                if (wave_masked)
                    c = cell3<T, true, GMODE>(g, Gm, is, okx, oky, okz, (T)a.den_guard, gc, n_fp64, ill);
                else
                    c = cell3<T, false, GMODE>(g, Gm, is, true, true, true, (T)a.den_guard, gc, n_fp64, ill);
            }
            for (int o = G / 2; o > 0; o >>= 1) c = vmin<T>(c, __shfl_xor(c, o));
            F = vmin<T>(F, c);
        }
        if constexpr (LIST == 2) {
            lane_cells -= below && lane_cells != 0u && !(last_key < F) ? 1u : 0u;
            // the longest walk: the context's next map chooses its layout by it
            if (__ballot(rows > LONG_WALK_ROWS) != 0ull) {
                for (int o = WAVE / 2; o > 0; o >>= 1) rows = max(rows, (uint32_t)__shfl_xor((int)rows, o));
                if ((threadIdx.x & (WAVE - 1)) == 0) atomicMax(&a.sc->long_rows, rows);
            }
        }
        for (int o = G / 2; o > 0; o >>= 1) {
            lane_cells += (uint32_t)__shfl_xor((int)lane_cells, o);
            ill = (__shfl_xor((int)ill, o) != 0) || ill;
        }
        const bool leader = live && gl == 0;
        const bool to_guard = GMODE == 1 && leader && ill;
        if (leader && !to_guard) {
            const float gam = (float)sqrt((double)F);
            a.gamma[r] = gam;
            npass += gam <= 1.0f;
            nborder += fabsf(gam - 1.0f) <= 1e-5f;
            gm = max(gm, f2u(gam * gam));
            cells += lane_cells;
        }
        if (GMODE == 1) {
            const uint32_t gpos = block_append(to_guard, &a.sc->n_guard);
            if (to_guard) a.guard_list[gpos] = (uint32_t)r;
        }
    }
    grids_counts(a.sc, npass, nborder, cells, gm);
}

}  // namespace

hipError_t launch_batch_key0(const BatchPair* pairs, const uint2* items, int n_items, hipStream_t s) {
    if (n_items > 0)
        hipLaunchKernelGGL(k_batch_key0, dim3((unsigned)n_items), dim3(SEARCH_THREADS), 0, s, pairs, items);
    return hipGetLastError();
}

hipError_t launch_batch_tail(const BatchPair* pairs, const uint2* items, int n_items, hipStream_t s) {
    if (n_items > 0)
        hipLaunchKernelGGL(k_batch_tail, dim3((unsigned)n_items), dim3(SEARCH_THREADS), 0, s, pairs, items);
    return hipGetLastError();
}

hipError_t launch_batch_finish(const BatchPair* pairs, const uint2* items, int n_items, hipStream_t s) {
    if (n_items > 0)
        hipLaunchKernelGGL(k_batch_finish, dim3((unsigned)n_items), dim3(SEARCH_THREADS), 0, s, pairs, items);
    return hipGetLastError();
}

unsigned tail_grid_blocks(uint32_t m_bound, int g) {
    // as tail_pass: groups of |g| lanes (automatic: the least width), at most kTailBlocks
    const unsigned groups = SEARCH_THREADS / (unsigned)(g > 0 ? g : -g);
    unsigned gb = (m_bound + groups - 1) / groups;
    return gb > kTailBlocks ? kTailBlocks : gb;
}

unsigned guard_grid_blocks() { return kGuardBlocks; }

hipError_t launch_stamp(unsigned long long* t, hipStream_t s) {
    hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, s, t);
    return hipGetLastError();
}

int64_t search_sums_needed(uint32_t) { return SUM_BINS; }

hipError_t launch_search(const SearchArgs& a, const SearchPlan& p, hipStream_t s) {
    const unsigned nb = blocks_for(p.M);
    if (nb == 0) return hipSuccess;
    const unsigned tb = nb < kTailBlocks ? nb : kTailBlocks;
    BlockSums* sums = a.sums;
    if (p.precision == 2) {
        // FP64 throughout.  3D: the key-0 pass and the queued walk as in FP32, whatever the
        // tail's length and layout request (391 thousand nodes at 2.5 mm: one lane per node from
        // row 0 took 145-400 us by the longest walk of each wave, this 63 + 16); 2D: one walk over all nodes from the
        // first row
        if (p.ndim == 3) hipLaunchKernelGGL(k_zero3_fp64, dim3(nb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
        else walk<2, 3, false>(a, a.nodes, &a.sc->n_masked, 0, nb, sums, s);
        if (p.ev_shell_end) (void)hipEventRecord(p.ev_shell_end, s);
        if (p.ev_sort_end) (void)hipEventRecord(p.ev_sort_end, s);
        if (p.ndim == 3 && a.tab_len > 8) {
            const unsigned gb = (p.M + TQ_GROUPS - 1) / TQ_GROUPS;
            cell_ranges(a, &a.sc->n_tail, s);
            hipLaunchKernelGGL(k_tail_fp64, dim3(gb < kTailBlocks ? gb : kTailBlocks), dim3(SEARCH_THREADS), 0, s, a, 8, sums);
        }
        if (p.ev_tail_end) (void)hipEventRecord(p.ev_tail_end, s);
    } else {
        const bool guarded = p.precision == 1 && p.ndim == 3;
        const int first = p.ndim == 3 ? 8 : 4;
        // pass A (unless a batch queued it for every pair in one launch)
        if (p.skip_zero) {
        } else if (p.zero_lanes) {
            // one lane per zero-key cell, grid-stride over the nodes
            const unsigned lanes = p.ndim == 3 ? 8u : 4u;
            uint64_t want = ((uint64_t)p.M * lanes + SEARCH_THREADS - 1) / SEARCH_THREADS;
            const unsigned zb = (unsigned)(want < kZeroGroupBlocks ? want : kZeroGroupBlocks);
            if (p.ndim == 3) {
                if (guarded) hipLaunchKernelGGL((k_zero_group<3, 1>), dim3(zb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
                else hipLaunchKernelGGL((k_zero_group<3, 0>), dim3(zb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
            } else {
                hipLaunchKernelGGL((k_zero_group<2, 0>), dim3(zb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
            }
        } else if (p.ndim == 3 && p.projection == 1) {
            // Ju's recursion in the key-0 pass (interior cells)
            if (guarded) hipLaunchKernelGGL(k_zero3_ju<1>, dim3(nb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
            else hipLaunchKernelGGL(k_zero3_ju<0>, dim3(nb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
        } else if (p.ndim == 3) {
            if (guarded) hipLaunchKernelGGL(k_zero3<1>, dim3(nb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
            else hipLaunchKernelGGL(k_zero3<0>, dim3(nb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
        } else {
            hipLaunchKernelGGL(k_zero2<0>, dim3(nb), dim3(SEARCH_THREADS), 0, s, a, p.zero, sums);
        }
        if (p.ev_shell_end) (void)hipEventRecord(p.ev_shell_end, s);
        if (p.after_zero) {
            hipError_t e = p.after_zero(p.after_zero_user, s);
            if (e != hipSuccess) return e;
        }
        // tail sort (count read on the device).  The order only groups similar walks into a
        // wave (every order gives the same map), so long tails are sorted by the keys' top 16
        // bits: two radix passes instead of four
        if (p.hist) {
            hipError_t e = p.small_sort
                               ? sort_order_small(a.tail_key_arr, a.tail_pos, &a.sc->n_tail, &a.sc->sort_overflow, s)
                               : radix_sort_pairs(a.tail_key_arr, a.tail_pos, p.tmp_keys, p.tmp_vals, p.M,
                                                  &a.sc->n_tail, p.hist, s, 16);
            if (e != hipSuccess) return e;
        }
        if (p.ev_sort_end) (void)hipEventRecord(p.ev_sort_end, s);
        // pass B (with the learned radius: the speculative walk, then the plain walk of the
        // nodes it could not certify, resumed where the speculative bound cut them off)
        if (a.tab_len > first) {
            const int spec = p.spec;
            tail_pass(a, p, a.tail_pos, &a.sc->n_tail, first, guarded, spec, tb, sums, s);
            if (spec == 1)
                tail_pass(a, p, a.fb_list, &a.sc->n_fallback, first, guarded, 2, tb, sums, s);
        }
        if (p.ev_tail_end) (void)hipEventRecord(p.ev_tail_end, s);
        // guard pass, count reduction and publication in one launch
        if (guarded) {
            hipLaunchKernelGGL(k_finish<true>, dim3(kGuardBlocks), dim3(SEARCH_THREADS), 0, s, a, sums, p.seq, p.ring);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL(k_finish<false>, dim3(1), dim3(SEARCH_THREADS), 0, s, a, sums, p.seq, p.ring);
    return hipGetLastError();
}


hipError_t launch_grids_prep(const GridsArgs& a, hipStream_t s) {
    const int64_t nr = (int64_t)a.rn[0] * a.rn[1] * a.rn[2];
    const int64_t ne = (int64_t)a.en[0] * a.en[1] * a.en[2];
    const int64_t n = nr > ne ? nr : ne;
    constexpr int64_t kMaxBlocks = MAX_BLOCKS;   // partials each listing block reduces
    const int64_t nb1 = (n + 256 * GRIDS_MAX_ITEMS - 1) / (256 * GRIDS_MAX_ITEMS);
    const unsigned b1 = (unsigned)(nb1 < kMaxBlocks ? nb1 : kMaxBlocks);
    hipLaunchKernelGGL(k_grids_max, dim3(b1), dim3(256), 0, s, a, nr, ne);
    const int64_t chunks = (nr + 256 * GRIDS_PER_THREAD - 1) / (256 * GRIDS_PER_THREAD);
    const unsigned b2 = (unsigned)(chunks < 4096 ? chunks : 4096);
    hipLaunchKernelGGL(k_grids_list, dim3(b2), dim3(256), 0, s, a, nr, (int)b1);
    return hipGetLastError();
}

hipError_t launch_grids_fp64(const GridsArgs& a, bool guard, int lanes, hipStream_t s) {
    if (guard) hipLaunchKernelGGL((k_grids_walk<double, 0, 1>), dim3(512), dim3(256), 0, s, a, lanes, false);
    else hipLaunchKernelGGL((k_grids_walk<double, 0, 0>), dim3(2048), dim3(256), 0, s, a, lanes, false);
    return hipGetLastError();
}

hipError_t launch_grids_finish(const GridsArgs& a, uint32_t* seq, Scalars* ring, hipStream_t s) {
    hipLaunchKernelGGL(k_finish_counts, dim3(1), dim3(SEARCH_THREADS), 0, s, a.sums, a.sc, seq, ring);
    return hipGetLastError();
}

hipError_t launch_grids_zero(const GridsArgs& a, int precision, bool far, hipStream_t s) {
    const int64_t nr = (int64_t)a.rn[0] * a.rn[1] * a.rn[2];   // the list holds at most nr nodes
    const unsigned nb = (unsigned)((nr + 255) / 256);
    if (precision == 1) {
        if (far) hipLaunchKernelGGL((k_grids_zero<1, true>), dim3(nb), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_grids_zero<1, false>), dim3(nb), dim3(256), 0, s, a);
    } else {
        if (far) hipLaunchKernelGGL((k_grids_zero<0, true>), dim3(nb), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_grids_zero<0, false>), dim3(nb), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_grids_tail(const GridsArgs& a, int precision, int lanes, bool queued, hipStream_t s) {
    if (lanes == 0 && queued) {
        const int64_t nr = (int64_t)a.rn[0] * a.rn[1] * a.rn[2];
        const int64_t nb = (nr + TQ_GROUPS - 1) / TQ_GROUPS;
        const dim3 g((unsigned)(nb < kTailBlocks ? nb : kTailBlocks)), b(SEARCH_THREADS);
        if (precision == 1) hipLaunchKernelGGL(k_grids_tail<1>, g, b, 0, s, a);
        else hipLaunchKernelGGL(k_grids_tail<0>, g, b, 0, s, a);
        return hipGetLastError();
    }
    const dim3 grid(2048), block(256);
    const int G = lanes > 0 ? lanes : GRIDS_LANES;
    if (precision == 1) hipLaunchKernelGGL((k_grids_walk<float, 1, 2>), grid, block, 0, s, a, G, lanes == 0);
    else hipLaunchKernelGGL((k_grids_walk<float, 0, 2>), grid, block, 0, s, a, G, lanes == 0);
    return hipGetLastError();
}

}  // namespace gammax
