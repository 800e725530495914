// Device helpers of libneb: vector math, Philox, BSDFs, plane-box area,
// octree addressing and queries, BVH traversal.  gfx950 only.
#pragma once
#include "neb_bvh.h"
#include "neb_internal.h"

namespace neb {

#define NEB_PI 3.14159265358979323846f

struct f3 {
    float x, y, z;
};
__device__ __forceinline__ f3 mk3(float x, float y, float z) { return f3{x, y, z}; }
__device__ __forceinline__ f3 operator+(f3 a, f3 b) { return mk3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ __forceinline__ f3 operator-(f3 a, f3 b) { return mk3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ f3 operator-(f3 a) { return mk3(-a.x, -a.y, -a.z); }
__device__ __forceinline__ f3 operator*(f3 a, float s) { return mk3(a.x * s, a.y * s, a.z * s); }
__device__ __forceinline__ f3 operator*(f3 a, f3 b) { return mk3(a.x * b.x, a.y * b.y, a.z * b.z); }
__device__ __forceinline__ float dot3(f3 a, f3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ f3 cross3(f3 a, f3 b) {
    return mk3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ f3 normalize3(f3 a) { return a * rsqrtf(dot3(a, a)); }
__device__ __forceinline__ f3 xyz(float4 v) { return mk3(v.x, v.y, v.z); }
__device__ __forceinline__ float4 f4(f3 a, float w) { return make_float4(a.x, a.y, a.z, w); }
__device__ __forceinline__ float get3(f3 a, int i) { return i == 0 ? a.x : (i == 1 ? a.y : a.z); }
__device__ __forceinline__ bool is_zero3(f3 a) { return a.x == 0.f && a.y == 0.f && a.z == 0.f; }
__device__ __forceinline__ f3 load3(const float* p) { return mk3(p[0], p[1], p[2]); }

// ---------------------------------------------------------------------------
// Philox-4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
// 32x32->64 multiplications with Weyl-sequence key schedule.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t m0 = 0xD2511F53u, m1 = 0xCD9E8D57u;
        uint32_t hi0 = __umulhi(m0, c.x), lo0 = m0 * c.x;
        uint32_t hi1 = __umulhi(m1, c.z), lo1 = m1 * c.z;
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

struct U4 {
    float u[4];
};
// four uniforms in [0,1): the top 24 bits of each output, exact in FP32
__device__ __forceinline__ U4 uniforms(uint32_t k0, uint32_t k1, uint32_t a, uint32_t b, uint32_t c,
                                       uint32_t tag) {
    uint4 x = philox10(make_uint4(a, b, c, tag), k0, k1);
    const float s = 1.0f / 16777216.0f;
    U4 r;
    r.u[0] = (float)(x.x >> 8) * s;
    r.u[1] = (float)(x.y >> 8) * s;
    r.u[2] = (float)(x.z >> 8) * s;
    r.u[3] = (float)(x.w >> 8) * s;
    return r;
}

// branchless orthonormal basis around n (Duff et al., JCGT 6(1), 2017)
__device__ __forceinline__ void basis(f3 n, f3& t1, f3& t2) {
    float sg = copysignf(1.0f, n.z);
    float a = -1.0f / (sg + n.z);
    float b = n.x * n.y * a;
    t1 = mk3(1.0f + sg * n.x * n.x * a, sg * b, -sg * n.x);
    t2 = mk3(b, sg + n.y * n.y * a, -n.y);
}

// ---------------------------------------------------------------------------
// BSDFs.  Geometric normal only; wi = direction the path arrived from, wo =
// direction it leaves to, both pointing away from the surface.  Delta lobes
// report their discrete selection probability as pdf.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool mat_delta(int type) { return type == NEB_MAT_MIRROR || type == NEB_MAT_DIELECTRIC; }
__device__ __forceinline__ bool mat_black(const neb_material& m) {
    return m.albedo[0] == 0.f && m.albedo[1] == 0.f && m.albedo[2] == 0.f;
}
__device__ __forceinline__ bool mat_emits(const neb_material& m) {
    return m.emission[0] + m.emission[1] + m.emission[2] > 0.f;
}

__device__ __forceinline__ float fresnel(float cos_i, float eta) {
    float s2 = eta * eta * (1.0f - cos_i * cos_i);
    if (s2 >= 1.0f) return 1.0f;
    float ct = sqrtf(1.0f - s2);
    float rs = (eta * cos_i - ct) / (eta * cos_i + ct);
    float rp = (cos_i - eta * ct) / (cos_i + eta * ct);
    return 0.5f * (rs * rs + rp * rp);
}

__device__ __forceinline__ float ggx_d(float a, float c) {
    if (c <= 0.f) return 0.f;
    float a2 = a * a;
    float t = c * c * (a2 - 1.0f) + 1.0f;
    return a2 / (NEB_PI * t * t);
}
__device__ __forceinline__ float ggx_g1(float a, float c) {
    float c2 = c * c;
    return 2.0f / (1.0f + sqrtf(1.0f + a * a * (1.0f - c2) / c2));
}

__device__ __forceinline__ float bsdf_pdf(const neb_material& m, f3 n, f3 wi, f3 wo) {
    float ci = dot3(n, wi), co = dot3(n, wo);
    bool same = ci * co > 0.f;
    switch (m.type) {
    case NEB_MAT_LAMBERT: return same ? fabsf(co) * (1.0f / NEB_PI) : 0.f;
    case NEB_MAT_MIRROR: return same ? 1.f : 0.f;
    case NEB_MAT_DIELECTRIC: {
        float F = fresnel(fabsf(ci), ci > 0.f ? 1.0f / m.ior : m.ior);
        return same ? F : 1.0f - F;
    }
    case NEB_MAT_GGX: {
        if (!same) return 0.f;
        f3 ns = ci > 0.f ? n : -n;
        f3 h = normalize3(wi + wo);
        float cm = dot3(h, ns);
        return ggx_d(m.alpha, cm) * cm / (4.0f * fabsf(dot3(wo, h)));
    }
    }
    return 0.f;
}

__device__ __forceinline__ f3 bsdf_f(const neb_material& m, f3 n, f3 wi, f3 wo) {
    float ci = dot3(n, wi), co = dot3(n, wo);
    f3 alb = load3(m.albedo);
    if (ci * co <= 0.f) return mk3(0.f, 0.f, 0.f);
    if (m.type == NEB_MAT_LAMBERT) return alb * (1.0f / NEB_PI);
    if (m.type == NEB_MAT_GGX) {
        f3 ns = ci > 0.f ? n : -n;
        f3 h = normalize3(wi + wo);
        float D = ggx_d(m.alpha, dot3(h, ns));
        float G = ggx_g1(m.alpha, fabsf(ci)) * ggx_g1(m.alpha, fabsf(co));
        return alb * (D * G / (4.0f * fabsf(ci) * fabsf(co)));
    }
    return mk3(0.f, 0.f, 0.f);
}

struct Sample {
    f3 dir, w;
    float pdf;
    int ev;      // 1 scatter, 2 reflect, 3 refract, 0 failed
};

// bsdf_f and the densities of both directions, of wo given wi and of wi given
// wo, of a material that is not specular: one half vector and one normal
// distribution for the three
__device__ __forceinline__ f3 bsdf_both(const neb_material& m, f3 n, f3 wi, f3 wo, float& p_wo, float& p_wi) {
    const float ci = dot3(n, wi), co = dot3(n, wo);
    const f3 alb = load3(m.albedo);
    p_wo = p_wi = 0.f;
    if (ci * co <= 0.f) return mk3(0.f, 0.f, 0.f);
    if (m.type == NEB_MAT_LAMBERT) {
        p_wo = fabsf(co) * (1.0f / NEB_PI);
        p_wi = fabsf(ci) * (1.0f / NEB_PI);
        return alb * (1.0f / NEB_PI);
    }
    if (m.type == NEB_MAT_GGX) {
        const f3 ns = ci > 0.f ? n : -n;
        const f3 h = normalize3(wi + wo);
        const float cm = dot3(h, ns), D = ggx_d(m.alpha, cm);
        p_wo = D * cm / (4.0f * fabsf(dot3(wo, h)));
        p_wi = D * cm / (4.0f * fabsf(dot3(wi, h)));
        const float G = ggx_g1(m.alpha, fabsf(ci)) * ggx_g1(m.alpha, fabsf(co));
        return alb * (D * G / (4.0f * fabsf(ci) * fabsf(co)));
    }
    return mk3(0.f, 0.f, 0.f);
}
__device__ __forceinline__ Sample bsdf_sample(const neb_material& m, f3 n, f3 wi, const U4& u) {
    Sample s;
    s.ev = 0;
    s.pdf = 0.f;
    s.w = mk3(0.f, 0.f, 0.f);
    s.dir = mk3(0.f, 0.f, 1.f);
    float ci = dot3(n, wi);
    if (ci == 0.f) return s;
    f3 ns = ci > 0.f ? n : -n;
    f3 alb = load3(m.albedo);
    if (m.type == NEB_MAT_LAMBERT) {
        f3 t1, t2;
        basis(ns, t1, t2);
        float r = sqrtf(u.u[1]);
        float sp, cp;
        sincosf(2.0f * NEB_PI * u.u[2], &sp, &cp);
        float z = sqrtf(fmaxf(0.f, 1.0f - u.u[1]));
        s.dir = normalize3(t1 * (r * cp) + t2 * (r * sp) + ns * z);
        float co = dot3(s.dir, ns);
        if (co <= 0.f) return s;
        s.pdf = co * (1.0f / NEB_PI);
        s.w = alb;
        s.ev = 1;
    } else if (m.type == NEB_MAT_MIRROR) {
        float c = dot3(wi, ns);
        s.dir = ns * (2.0f * c) - wi;
        s.pdf = 1.0f;
        s.w = alb;
        s.ev = 2;
    } else if (m.type == NEB_MAT_DIELECTRIC) {
        float c = dot3(wi, ns);
        float eta = ci > 0.f ? 1.0f / m.ior : m.ior;
        float F = fresnel(c, eta);
        if (u.u[0] < F) {
            s.dir = ns * (2.0f * c) - wi;
            s.pdf = F;
            s.ev = 2;
        } else {
            float ct = sqrtf(fmaxf(0.f, 1.0f - eta * eta * (1.0f - c * c)));
            s.dir = normalize3(ns * (eta * c - ct) - wi * eta);
            s.pdf = 1.0f - F;
            s.ev = 3;
        }
        s.w = alb;
    } else if (m.type == NEB_MAT_GGX) {
        float a = m.alpha;
        float tt = a * sqrtf(u.u[1] / (1.0f - u.u[1]));
        float ct = rsqrtf(1.0f + tt * tt);
        float st = tt * ct;
        float sp, cp;
        sincosf(2.0f * NEB_PI * u.u[2], &sp, &cp);
        f3 t1, t2;
        basis(ns, t1, t2);
        f3 h = normalize3(t1 * (st * cp) + t2 * (st * sp) + ns * ct);
        float wh = dot3(wi, h);
        if (wh <= 0.f) return s;
        s.dir = h * (2.0f * wh) - wi;
        float co = dot3(s.dir, ns);
        if (co <= 0.f) return s;
        float cim = fabsf(ci);
        float G = ggx_g1(a, cim) * ggx_g1(a, co);
        s.pdf = ggx_d(a, ct) * ct / (4.0f * wh);
        s.w = alb * (G * wh / (cim * ct));
        s.ev = 1;
    }
    return s;
}

// ---------------------------------------------------------------------------
// eq. (area): area of the plane (p, n) inside the box [bmin, bmax].  The plane
// offset is taken relative to the box's min corner; the 3-D case sums in FP64.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float plane_box_area(f3 bmin, f3 bmax, f3 p, f3 n) {
    f3 s = bmax - bmin;
    f3 a = mk3(fabsf(n.x), fabsf(n.y), fabsf(n.z));
    if (fabsf(a.x - 1.0f) < 1e-3f) return s.y * s.z;
    if (fabsf(a.y - 1.0f) < 1e-3f) return s.x * s.z;
    if (fabsf(a.z - 1.0f) < 1e-3f) return s.x * s.y;
    f3 q = p - bmin;
    for (int d = 0; d < 3; ++d) {
        if (get3(a, d) < 1e-4f) {
            int ix = d == 0 ? 1 : (d == 1 ? 2 : 0);
            int iy = d == 0 ? 2 : (d == 1 ? 0 : 1);
            float nx = get3(n, ix), ny = get3(n, iy);
            float ex = nx * get3(s, ix), ey = ny * get3(s, iy);
            float t = nx * get3(q, ix) + ny * get3(q, iy);
            float sum = fmaxf(0.f, t) - fmaxf(0.f, t - ex) - fmaxf(0.f, t - ey) + fmaxf(0.f, t - ex - ey);
            return get3(s, d) * fabsf(sum / (nx * ny));
        }
    }
    double ex = (double)n.x * s.x, ey = (double)n.y * s.y, ez = (double)n.z * s.z;
    double t = (double)n.x * q.x + (double)n.y * q.y + (double)n.z * q.z;
    double sum = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        double h = t - ((c & 1) ? ex : 0.0) - ((c & 2) ? ey : 0.0) - ((c & 4) ? ez : 0.0);
        double v = h > 0.0 ? h * h : 0.0;
        sum += (__popc(c) & 1) ? -v : v;
    }
    return (float)fabs(sum / (2.0 * (double)n.x * (double)n.y * (double)n.z));
}

// ---------------------------------------------------------------------------
// Octree addressing (FP32, no contraction, as the class of Appendix B) and
// the density query of eq. (octdensity).
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool oct_norm(const OctParams& P, f3 p, float q[3]) {
    float pv[3] = {p.x, p.y, p.z};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        float v = __fmul_rn(__fsub_rn(pv[i], P.min_bound[i]), P.size_inv[i]);
        if (!(v >= 0.0f && v < 1.0f)) return false;
        q[i] = v;
    }
    return true;
}

// A point's cell at the octree's finest level: integer coordinates
// floor(q * 2^depth) of its normalised position q.  The leaf reached at level
// L holds the cell c >> (depth - L); the child taken below level L is bit
// depth - L - 1 of each coordinate (the same child as the deposits take from
// floor(q * 2^(L+1)) & 1, as scaling by a power of two is exact).
struct OctCell {
    int32_t c[3];
};

__device__ __forceinline__ bool oct_cell(const OctParams& P, int depth, f3 p, OctCell& k) {
    float q[3];
    if (!oct_norm(P, p, q)) return false;
    const float fine = (float)(1 << depth);
#pragma unroll
    for (int a = 0; a < 3; ++a) k.c[a] = (int32_t)(q[a] * fine);
    return true;
}

// the child of inner node word w (< 0) on the way to cell k, `shift` = depth -
// (level of the child)
__device__ __forceinline__ int32_t oct_child(int32_t w, const OctCell& k, int shift) {
    const int32_t child = ((k.c[0] >> shift) & 1) | (((k.c[1] >> shift) & 1) << 1) | (((k.c[2] >> shift) & 1) << 2);
    return child - w;
}

// Floor under the area of the surface inside a leaf of diagonal `diag`, so
// that a surface grazing a cell does not give an unbounded density: a tenth
// of diag^2 for the probe at the query point, a hundredth for the offset
// probes (Appendix B).
__device__ __forceinline__ float oct_area_floor(float diag, bool centre) {
    return diag * diag * (centre ? 0.1f : 0.01f);
}

// the fresh words, where queries have to add them to the node words
__device__ __forceinline__ const int32_t* oct_unfolded(const OctState& st, const int32_t* fresh) {
    return st.folded ? nullptr : fresh;
}
// a leaf's count, its word and node given
__device__ __forceinline__ int32_t oct_count(int32_t w, int32_t at, const int32_t* __restrict__ unfolded) {
    return (w & kOctCountMask) + (unfolded ? unfolded[at] : 0);
}

// eq. (octdensity) at the leaf (its count, level `level`) holding cell k of the
// point p with normal n: the leaf's count over the area of the plane through
// p inside the leaf's box (eq. area), times the density scale.  centre: the
// probe at the query point; then *diag_out receives the leaf's diagonal (if
// the leaf has a count).
__device__ __forceinline__ float oct_leaf_density(const OctParams& P, float density_scale, int depth,
                                                  const OctCell& k, int level, int32_t count, f3 p, f3 n, bool centre,
                                                  float* diag_out) {
    if (count <= 0) return 0.f;
    const int32_t cells = 1 << level;  // per axis at this level
    const int shift = depth - level;
    float edge[3], lo[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        edge[a] = 1.0f / ((float)cells * P.size_inv[a]);
        lo[a] = (float)(k.c[a] >> shift) * edge[a];
    }
    const f3 bmin = mk3(lo[0], lo[1], lo[2]);
    const f3 bmax = bmin + mk3(edge[0], edge[1], edge[2]);
    const f3 rel = mk3(p.x - P.min_bound[0], p.y - P.min_bound[1], p.z - P.min_bound[2]);
    const float area = plane_box_area(bmin, bmax, rel, n);
    const float diag = P.scene_scale / (float)cells;
    if (centre) *diag_out = diag;
    return density_scale * (float)count / fmaxf(oct_area_floor(diag, centre), area);
}

// upper median of n (1..5) values: the (n/2)-th smallest (sorts v)
__device__ __forceinline__ float upper_median(float* v, int n) {
    for (int i = 1; i < n; ++i) {
        const float x = v[i];
        int j = i;
        for (; j > 0 && v[j - 1] > x; --j) v[j] = v[j - 1];
        v[j] = x;
    }
    return v[n / 2];
}

// eq. (octdensity) at the leaf holding p (Appendix B get_density)
__device__ __forceinline__ float oct_query(const int32_t* __restrict__ nodes, const int32_t* __restrict__ unfolded,
                                           const OctParams& P, float density_scale,
                                           int depth, f3 p, f3 n, bool centre, float* diag_out) {
    OctCell k;
    if (!oct_cell(P, depth, p, k)) return 0.f;
    int32_t at = P.root, w = nodes[at];
    int level = 0;
    while (w < 0) {
        ++level;
        at = oct_child(w, k, depth - level);
        w = nodes[at];
    }
    return oct_leaf_density(P, density_scale, depth, k, level, oct_count(w, at, unfolded), p, n, centre, diag_out);
}

// Appendix B get_density_robust: the densities at p and at four points
// offset along the tangents by 1.1 leaf diagonals of p's leaf (1.1e-3
// scene units when that leaf is empty); the upper median of the non-zero
// ones (0 if none)
__device__ __forceinline__ float oct_query_robust(const int32_t* __restrict__ nodes,
                                                  const int32_t* __restrict__ unfolded, const OctParams& P,
                                                  float density_scale, int depth, f3 p, f3 n) {
    f3 tx, ty;
    basis(n, tx, ty);
    float diag = 1e-3f;
    float found[5];
    int nf = 0;
    const float centre = oct_query(nodes, unfolded, P, density_scale, depth, p, n, true, &diag);
    if (centre > 0.f) found[nf++] = centre;
    const float step = diag * 1.1f;
    const f3 probe[4] = {p + tx * step, p - tx * step, p + ty * step, p - ty * step};
    // the four offset probes descend together, one level per step, so that
    // their node loads are in flight at once (a probe outside the octree's
    // box stops at once with density 0)
    OctCell k[4];
    int32_t w[4], at[4];
    int level[4];
    const int32_t root = nodes[P.root];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool in = oct_cell(P, depth, probe[i], k[i]);
        if (!in) k[i].c[0] = k[i].c[1] = k[i].c[2] = 0;
        w[i] = in ? root : 0;
        at[i] = in ? P.root : -1;
        level[i] = 0;
    }
    while (w[0] < 0 || w[1] < 0 || w[2] < 0 || w[3] < 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (w[i] < 0) {
                ++level[i];
                at[i] = oct_child(w[i], k[i], depth - level[i]);
                w[i] = nodes[at[i]];
            }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = at[i] < 0 ? 0 : oct_count(w[i], at[i], unfolded);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float r = oct_leaf_density(P, density_scale, depth, k[i], level[i], w[i], probe[i], n, false, nullptr);
        if (r > 0.f) found[nf++] = r;
    }
    return nf ? upper_median(found, nf) : 0.f;
}

// ---------------------------------------------------------------------------
// BVH traversal: four child boxes per 128-byte node, per-lane stack in LDS,
// watertight ray-triangle test (Woop, Benthin, Wald, JCGT 2(1), 2013).
// ---------------------------------------------------------------------------
struct RayPre {
    f3 o, d, inv;
    int kx, ky, kz;
    float sx, sy, sz;
};

__device__ __forceinline__ RayPre ray_pre(f3 o, f3 d) {
    RayPre r;
    r.o = o;
    r.d = d;
    const float big = 1e30f;
    r.inv = mk3(fabsf(d.x) > 1e-30f ? 1.0f / d.x : copysignf(big, d.x),
                fabsf(d.y) > 1e-30f ? 1.0f / d.y : copysignf(big, d.y),
                fabsf(d.z) > 1e-30f ? 1.0f / d.z : copysignf(big, d.z));
    float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    int kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    int kx = kz == 2 ? 0 : kz + 1;
    int ky = kx == 2 ? 0 : kx + 1;
    if (get3(d, kz) < 0.f) {
        int t = kx;
        kx = ky;
        ky = t;
    }
    r.kx = kx;
    r.ky = ky;
    r.kz = kz;
    float dz = get3(d, kz);
    r.sx = get3(d, kx) / dz;
    r.sy = get3(d, ky) / dz;
    r.sz = fabsf(dz) > 1e-30f ? get3(r.inv, kz) : 1.0f / dz;
    return r;
}

// returns t in (0, tmax) or -1
__device__ __forceinline__ float tri_hit(const RayPre& r, f3 v0, f3 v1, f3 v2, float tmax) {
    f3 A = v0 - r.o, B = v1 - r.o, C = v2 - r.o;
    float az = get3(A, r.kz), bz = get3(B, r.kz), cz = get3(C, r.kz);
    float Ax = get3(A, r.kx) - r.sx * az, Ay = get3(A, r.ky) - r.sy * az;
    float Bx = get3(B, r.kx) - r.sx * bz, By = get3(B, r.ky) - r.sy * bz;
    float Cx = get3(C, r.kx) - r.sx * cz, Cy = get3(C, r.ky) - r.sy * cz;
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.f || V == 0.f || W == 0.f) {
        U = (float)((double)Cx * By - (double)Cy * Bx);
        V = (float)((double)Ax * Cy - (double)Ay * Cx);
        W = (float)((double)Bx * Ay - (double)By * Ax);
    }
    if ((U < 0.f || V < 0.f || W < 0.f) && (U > 0.f || V > 0.f || W > 0.f)) return -1.f;
    float det = U + V + W;
    if (det == 0.f) return -1.f;
    float T = U * (r.sz * az) + V * (r.sz * bz) + W * (r.sz * cz);
    float t = T / det;
    return (t > 0.f && t < tmax) ? t : -1.f;
}

// Closest-hit traversal, one ray per lane, in two kinds of step that the
// caller (k_extend) runs for the lanes that wait for them: trace_node picks
// the lane's next inner node and tests its four children's boxes, then
// trace_triangle tests the triangles of the leaves among them one at a time,
// slot by slot, before the next trace_node stacks the inner children still in
// reach, nearest on top.  The order is that of a walk of one ray by itself.
// Of the triangles tested, the lowest primitive id wins a tie on t; a child no
// nearer than the nearest hit is dropped, so of triangles at one distance in
// different leaves some may not be tested.  The stack is the lane's LDS slots
// (stride kTraceBlock, slot 0 never filled).
struct TraceState {
    RayPre r;
    // byte offsets in a node of the words with the ray's near and far planes
    // of each axis (low planes: words 0..2, high ones 3..5)
    uint32_t nx, ny, nz, fx, fy, fz;
    float best;
    int prim;
    // the last visited node's children: references (a node or ~ a leaf's
    // first triangle) and the distance of an inner child in reach, -1
    // for a leaf in reach whose triangles are still to test, else INFINITY
    int c0, c1, c2, c3;
    float d0, d1, d2, d3;
    float least;  // the smallest of the four: < 0 while triangles come first
    int tri;      // the next triangle of the leaf in hand (the first slot with distance -1), -1: its first
    int* top;     // topmost filled stack slot; bot: none is filled
    int* bot;     // the slot below its lowest filled one
};

// the lane's walk starts (or goes on, with another lane's ray) at node `from`
__device__ __forceinline__ void trace_at(TraceState& T, int from, int* stack) {
    T.nx = T.r.inv.x < 0.f ? 48u : 0u;
    T.ny = T.r.inv.y < 0.f ? 64u : 16u;
    T.nz = T.r.inv.z < 0.f ? 80u : 32u;
    T.fx = 48u - T.nx;
    T.fy = 80u - T.ny;
    T.fz = 112u - T.nz;
    T.d0 = T.least = 0.f;
    T.d1 = T.d2 = T.d3 = INFINITY;
    T.c0 = from;
    T.tri = -1;
    T.top = T.bot = stack;
}

// false: a ray that cannot hit anything (a NaN or an infinity among its
// numbers, or no length) and is spared the walk
__device__ __forceinline__ bool trace_begin(TraceState& T, int root, int* stack, f3 o, f3 d, float tmax = INFINITY) {
    T.r = ray_pre(o, d);
    T.best = tmax;
    T.prim = -1;
    trace_at(T, root, stack);
    return tmax > 0.f && fabsf(o.x) < INFINITY && fabsf(o.y) < INFINITY && fabsf(o.z) < INFINITY &&
           fabsf(d.x) < INFINITY && fabsf(d.y) < INFINITY && fabsf(d.z) < INFINITY;
}

// (distance, node) pair of a child still to visit; compare-exchange by distance
__device__ __forceinline__ void near_first(float& da, int& na, float& db, int& nb) {
    const bool sw = db < da;
    const float d = sw ? db : da;
    const int n = sw ? nb : na;
    db = sw ? da : db;
    nb = sw ? na : nb;
    da = d;
    na = n;
}

// 16 bytes at a byte offset of a pool (Off: 32 bits where the pool is below
// 4 GB, which spares the 64-bit address arithmetic)
template <typename Off>
__device__ __forceinline__ float4 pool16(const float4* base, Off byte) {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(base) + byte);
}

// One node step.  The near and far planes are loaded by the ray's direction
// signs, so a slab needs no minimum and maximum of its two distances.  An
// empty slot's planes lie the wrong way round (1e30 before -1e30), out of
// reach; a ray from so far off that both are one distance to it tests the
// slot's triangle, which is never hit.  Returns false when no node is left:
// the ray is done.
template <typename Off>
__device__ __forceinline__ bool trace_node(const SceneView& S, TraceState& T) {
    const RayPre& r = T.r;
    int next = *T.top;
    // inner children still in reach, sorted nearest first (five
    // compare-exchanges; those at or beyond the nearest hit come last and are
    // dropped); the nearest is next, the others are stacked farthest first
    float d0 = T.d0, d1 = T.d1, d2 = T.d2, d3 = T.d3;
    int c0 = T.c0, c1 = T.c1, c2 = T.c2, c3 = T.c3;
    near_first(d0, c0, d1, c1);
    near_first(d2, c2, d3, c3);
    near_first(d0, c0, d2, c2);
    near_first(d1, c1, d3, c3);
    near_first(d1, c1, d2, c2);
    if (d3 < T.best) *(T.top += kTraceBlock) = c3;
    if (d2 < T.best) *(T.top += kTraceBlock) = c2;
    if (d1 < T.best) *(T.top += kTraceBlock) = c1;
    if (d0 < T.best) {
        next = c0;
    } else {
        if (T.top == T.bot) return false;
        T.top -= kTraceBlock;
    }
    const Off nd = (Off)(uint32_t)next << 7;
    const float4 ax = pool16<Off>(S.bvh, nd + T.nx), ay = pool16<Off>(S.bvh, nd + T.ny),
                 az = pool16<Off>(S.bvh, nd + T.nz), bx = pool16<Off>(S.bvh, nd + T.fx),
                 by = pool16<Off>(S.bvh, nd + T.fy), bz = pool16<Off>(S.bvh, nd + T.fz),
                 rf = pool16<Off>(S.bvh, nd + 96u);
    auto reach = [&](float nx, float ny, float nz, float fx, float fy, float fz, int ref) {
        const float tn = fmaxf(fmaxf((nx - r.o.x) * r.inv.x, (ny - r.o.y) * r.inv.y),
                               fmaxf((nz - r.o.z) * r.inv.z, 0.0f));
        const float tf = fminf(fminf((fx - r.o.x) * r.inv.x, (fy - r.o.y) * r.inv.y),
                               fminf((fz - r.o.z) * r.inv.z, T.best));
        return tn <= tf * 1.00000024f ? (ref < 0 ? -1.0f : tn) : INFINITY;
    };
    T.c0 = __float_as_int(rf.x);
    T.c1 = __float_as_int(rf.y);
    T.c2 = __float_as_int(rf.z);
    T.c3 = __float_as_int(rf.w);
    T.d0 = reach(ax.x, ay.x, az.x, bx.x, by.x, bz.x, T.c0);
    T.d1 = reach(ax.y, ay.y, az.y, bx.y, by.y, bz.y, T.c1);
    T.d2 = reach(ax.z, ay.z, az.z, bx.z, by.z, bz.z, T.c2);
    T.d3 = reach(ax.w, ay.w, az.w, bx.w, by.w, bz.w, T.c3);
    T.least = fminf(fminf(T.d0, T.d1), fminf(T.d2, T.d3));
    return true;
}

// One triangle step; the leaf's next triangle follows unless this one is
// marked as its last (v1.w).  kAnyHit: any hit below the ray's end finishes
// it.  Returns false when the ray is done.
template <bool kAnyHit, typename Off>
__device__ __forceinline__ bool trace_triangle(const SceneView& S, TraceState& T) {
    const bool f0 = T.d0 < 0.f, f1 = !f0 && T.d1 < 0.f, f2 = !f0 && !f1 && T.d2 < 0.f, f3 = !f0 && !f1 && !f2;
    // (values, not a choice between the members' addresses, which would keep the state in memory)
    const int c0 = T.c0, c1 = T.c1, c2 = T.c2, c3 = T.c3;
    if (T.tri < 0) T.tri = ~(f0 ? c0 : f1 ? c1 : f2 ? c2 : c3);
    const Off at = (Off)(uint32_t)T.tri * 48u;
    const float4 p0 = pool16<Off>(S.tri, at), p1 = pool16<Off>(S.tri, at + 16u), p2 = pool16<Off>(S.tri, at + 32u);
    const float t = tri_hit(T.r, xyz(p0), xyz(p1), xyz(p2), kAnyHit ? T.best : T.best * 1.0000001f);
    const int id = __float_as_int(p0.w);
    if (t > 0.f && (t < T.best || (t == T.best && id < T.prim))) {
        T.best = t;
        T.prim = id;
        if (kAnyHit) return false;
    }
    const bool last = __float_as_int(p1.w) != 0;
    T.tri = last ? -1 : T.tri + 1;
    T.d0 = last && f0 ? INFINITY : T.d0;
    T.d1 = last && f1 ? INFINITY : T.d1;
    T.d2 = last && f2 ? INFINITY : T.d2;
    T.d3 = last && f3 ? INFINITY : T.d3;
    T.least = fminf(fminf(T.d0, T.d1), fminf(T.d2, T.d3));
    return true;
}

// LDS written by some lanes of the wave, to be read by others: the
// barrier alone orders no memory access for the compiler
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// device-wide counter add with one atomic per wave
__device__ __forceinline__ void wave_add_u64(unsigned long long* dst, unsigned v) {
    unsigned long long s = v;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0 && s) atomicAdd(dst, s);
}

// this block's stripe of the work statistics
__device__ __forceinline__ StatLine& stat_line(Counters* c) { return c->st[blockIdx.x & (kStatStripes - 1)]; }

// Block-wide slot reservation in one queue whose tail is *counter: one
// atomic per block (the waves' counts meet in wc[kWaves] and bb, LDS).  Every
// thread of the block must call it; lanes with take == false get -1.
template <int kWaves>
__device__ __forceinline__ int block_reserve(int32_t* counter, bool take, int* wc, int* bb) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const unsigned long long m = __ballot(take);
    if (lane == 0) wc[wid] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int w = 0; w < kWaves; ++w) tot += wc[w];
        *bb = tot ? atomicAdd(counter, tot) : 0;
    }
    __syncthreads();
    int base = *bb;
    for (int w = 0; w < wid; ++w) base += wc[w];
    __syncthreads();  // wc and bb are rewritten by the next call
    return take ? base + __popcll(m & ((1ull << lane) - 1ull)) : -1;
}

// wave-aggregated slot reservation: returns this lane's index in a queue
// whose tail is *counter; lanes with take == false get -1
__device__ __forceinline__ int wave_reserve(int* counter, bool take) {
    unsigned long long mask = __ballot(take);
    int lane = threadIdx.x & 63;
    int leader = __ffsll((long long)mask) - 1;
    int base = 0;
    if (mask == 0) return -1;
    if (lane == leader) base = atomicAdd(counter, __popcll(mask));
    base = __shfl(base, leader, 64);
    unsigned long long below = mask & ((1ull << lane) - 1ull);
    return take ? base + __popcll(below) : -1;
}

}  // namespace neb
