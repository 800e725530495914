// Host check of the tree as the device walks it (test infrastructure).
// Reads a mesh (int32 nv, nt; nv*3 float32 vertices; nt*3 int32 indices),
// lays its tree out at an offset in larger pools and walks it with the
// device's arithmetic (near and far planes picked by the direction's signs,
// leaves tested slot by slot).  Arguments: mesh, rays, log10 of the
// rays' distance from the mesh (-1: from inside it), 1 for directions with
// infinite components.  Prints one line of key=value figures:
//   rays, hits, differing (closest hit of the walk != brute force over every
//   triangle with the same test), outside (references that leave the scene's
//   part of the pools; the walk goes no further there), empty (empty slots
//   entered).
#include "neb_bvh.h"

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <utility>
#include <vector>

namespace {

constexpr int kNodeBase = 3, kTriBase = 5;

struct V3 {
    float x[3];
};
struct Ray {
    float o[3], d[3], inv[3];
    int kx, ky, kz;
    float sx, sy, sz;
};
Ray make_ray(const V3& o, const V3& d) {
    Ray r;
    for (int a = 0; a < 3; ++a) {
        r.o[a] = o.x[a];
        r.d[a] = d.x[a];
        r.inv[a] = fabsf(d.x[a]) > 1e-30f ? 1.f / d.x[a] : copysignf(1e30f, d.x[a]);
    }
    const float ax = fabsf(d.x[0]), ay = fabsf(d.x[1]), az = fabsf(d.x[2]);
    r.kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    r.kx = (r.kz + 1) % 3;
    r.ky = (r.kx + 1) % 3;
    if (d.x[r.kz] < 0.f) std::swap(r.kx, r.ky);
    r.sx = d.x[r.kx] / d.x[r.kz];
    r.sy = d.x[r.ky] / d.x[r.kz];
    r.sz = fabsf(d.x[r.kz]) > 1e-30f ? r.inv[r.kz] : 1.f / d.x[r.kz];
    return r;
}
// watertight ray-triangle test (Woop, Benthin, Wald, JCGT 2(1), 2013)
float hit_tri(const Ray& r, const float* t, float tmax) {
    float p[3][3];
    for (int v = 0; v < 3; ++v)
        for (int a = 0; a < 3; ++a) p[v][a] = t[4 * v + a] - r.o[a];
    float x[3], y[3], z[3];
    for (int v = 0; v < 3; ++v) {
        z[v] = p[v][r.kz];
        x[v] = p[v][r.kx] - r.sx * z[v];
        y[v] = p[v][r.ky] - r.sy * z[v];
    }
    float u = x[2] * y[1] - y[2] * x[1], v = x[0] * y[2] - y[0] * x[2], w = x[1] * y[0] - y[1] * x[0];
    if (u == 0.f || v == 0.f || w == 0.f) {
        u = (float)((double)x[2] * y[1] - (double)y[2] * x[1]);
        v = (float)((double)x[0] * y[2] - (double)y[0] * x[2]);
        w = (float)((double)x[1] * y[0] - (double)y[1] * x[0]);
    }
    if ((u < 0.f || v < 0.f || w < 0.f) && (u > 0.f || v > 0.f || w > 0.f)) return -1.f;
    const float det = u + v + w;
    if (det == 0.f) return -1.f;
    const float tt = (u * (r.sz * z[0]) + v * (r.sz * z[1]) + w * (r.sz * z[2])) / det;
    return (tt > 0.f && tt < tmax) ? tt : -1.f;
}
bool better(float t, int id, float bt, int bp) { return t > 0.f && (t < bt || (t == bt && id < bp)); }

int as_int(float f) {
    int i;
    std::memcpy(&i, &f, 4);
    return i;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc < 5) return 2;
    FILE* f = fopen(argv[1], "rb");
    if (!f) return 2;
    int32_t n[2];
    if (fread(n, 4, 2, f) != 2) return 2;
    std::vector<float> vert(3 * (size_t)n[0]);
    std::vector<int32_t> idx(3 * (size_t)n[1]);
    if (fread(vert.data(), 4, vert.size(), f) != vert.size() || fread(idx.data(), 4, idx.size(), f) != idx.size())
        return 2;
    fclose(f);
    const int rays = atoi(argv[2]);
    const float far = (float)atof(argv[3]);
    const bool infinite = atoi(argv[4]) != 0;
    neb::BvhHost H;
    if (!neb::build_bvh(vert.data(), n[0], idx.data(), n[1], H)) return 3;
    const int nt = n[1], none = kTriBase + nt;
    std::vector<float> nodes(32 * (size_t)(kNodeBase + H.n_nodes), 0.f), tris(12 * ((size_t)none + 1), 0.f);
    neb::bvh_device_layout(H, kNodeBase, kTriBase, none, &nodes[32 * kNodeBase], &tris[12 * kTriBase]);
    neb::bvh_no_triangle(&tris[12 * (size_t)none]);

    float lo[3] = {1e30f, 1e30f, 1e30f}, hi[3] = {-1e30f, -1e30f, -1e30f};
    for (int i = 0; i < n[0]; ++i)
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], vert[3 * (size_t)i + a]);
            hi[a] = std::max(hi[a], vert[3 * (size_t)i + a]);
        }
    std::mt19937 rng(7);
    std::uniform_real_distribution<float> U(0.f, 1.f);
    long hits = 0, differing = 0, outside = 0, empty = 0;
    for (int q = 0; q < rays; ++q) {
        const float z = 2.f * U(rng) - 1.f, ph = 6.2831853f * U(rng), s = sqrtf(std::max(0.f, 1.f - z * z));
        V3 d{{s * cosf(ph), s * sinf(ph), z}}, o;
        for (int a = 0; a < 3; ++a) o.x[a] = lo[a] + U(rng) * (hi[a] - lo[a]);
        if (far >= 0.f)
            for (int a = 0; a < 3; ++a) o.x[a] -= powf(10.f, far) * d.x[a];
        if (infinite)
            for (int a = 0; a < 3; ++a)
                if (a == q % 3 || U(rng) < 0.5f) d.x[a] = copysignf(INFINITY, d.x[a]);
        const Ray r = make_ray(o, d);
        float bt = INFINITY;
        int bp = -1;
        for (int p = 0; p < nt; ++p) {
            const float* t = &tris[12 * (size_t)(kTriBase + p)];
            const float tt = hit_tri(r, t, bt * 1.0000001f);
            if (better(tt, as_int(t[3]), bt, bp)) bt = tt, bp = as_int(t[3]);
        }
        float best = INFINITY;
        int prim = -1;
        std::vector<int> stack{kNodeBase};
        while (!stack.empty()) {
            const int nd = stack.back();
            stack.pop_back();
            if (nd < kNodeBase || nd >= kNodeBase + H.n_nodes) {
                ++outside;
                continue;
            }
            const float* D = &nodes[32 * (size_t)nd];
            int ref[4];
            float dist[4];
            for (int c = 0; c < 4; ++c) {
                ref[c] = as_int(D[24 + c]);
                float tn = 0.f, tf = best;
                for (int a = 0; a < 3; ++a) {
                    const bool neg = r.inv[a] < 0.f;
                    tn = fmaxf(tn, (D[4 * (neg ? 3 + a : a) + c] - r.o[a]) * r.inv[a]);
                    tf = fminf(tf, (D[4 * (neg ? a : 3 + a) + c] - r.o[a]) * r.inv[a]);
                }
                dist[c] = tn <= tf * 1.00000024f ? (ref[c] < 0 ? -1.f : tn) : INFINITY;
            }
            for (int c = 0; c < 4; ++c) {
                if (!(dist[c] < 0.f)) continue;
                for (int t = ~ref[c];; ++t) {
                    if (t < kTriBase || t > none) {
                        ++outside;
                        break;
                    }
                    empty += t == none;
                    const float* T = &tris[12 * (size_t)t];
                    const float tt = hit_tri(r, T, best * 1.0000001f);
                    if (better(tt, as_int(T[3]), best, prim)) best = tt, prim = as_int(T[3]);
                    if (as_int(T[7]) != 0) break;
                }
            }
            std::vector<std::pair<float, int>> inner;
            for (int c = 0; c < 4; ++c)
                if (dist[c] >= 0.f && dist[c] < best) inner.push_back({dist[c], ref[c]});
            std::sort(inner.begin(), inner.end());
            for (size_t j = inner.size(); j-- > 0;) stack.push_back(inner[j].second);
        }
        hits += bp >= 0;
        differing += bp != prim || (bp >= 0 && bt != best);
    }
    printf("rays=%d hits=%ld differing=%ld outside=%ld empty=%ld\n", rays, hits, differing, outside, empty);
    return 0;
}
