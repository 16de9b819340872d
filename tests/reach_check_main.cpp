// Driver for the CPU test of the key windows' bound (csrc/reach.h): posed bodies of every kind, their vertices taken through
// the renderer's arithmetic one by one, against the pixels that the bound says the body can touch.  The depths' reciprocals
// and the square root are given errors such as the hardware's: one unit in the last place either way, 0 for the reciprocal
// of a depth beyond 2^126.  Built and run by tests/test_host_reach.py; prints "ok <bodies> <in view> <out of view> <near>".
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../paper_2502_00021_amd/csrc/pxr_internal.h"
#include "../paper_2502_00021_amd/csrc/reach.h"

namespace {

std::mt19937_64 gen(20250200021ull);
double uniform(double lo, double hi) { return std::uniform_real_distribution<double>(lo, hi)(gen); }
bool chance(double p) { return uniform(0.0, 1.0) < p; }

float one_ulp_off(float x) {
    const int way = (int)(gen() % 3) - 1;
    return way == 0 ? x : std::nextafterf(x, way > 0 ? INFINITY : -INFINITY);
}
float rough_reciprocal(float x) {
    if (std::fabs(x) > 0x1p126f) return 0.0f;
    return one_ulp_off(1.0f / x);
}
float dot3(float a0, float a1, float a2, float b0, float b1, float b2) { return std::fmaf(a0, b0, std::fmaf(a1, b1, a2 * b2)); }

pxr_body_desc body(uint32_t type, uint32_t lon, uint32_t lat) {
    pxr_body_desc d{};
    d.type = type;
    for (float& s : d.shape) s = 1.0f;
    d.n_lon = lon;
    d.n_lat = lat;
    return d;
}

int fail(const char* what, int n, uint32_t b, const pxr::AxisReach& a, int lo, int hi) {
    std::fprintf(stderr, "scene %d body %u: %s: bound [%u, %u), vertices' pixels [%d, %d]\n", n, b, what, a.begin, a.end, lo, hi);
    return 1;
}

}  // namespace

int main(int argc, char** argv) {
    const int scenes = argc > 1 ? std::atoi(argv[1]) : 20000;
    // the templates: every primitive kind and a mesh away from its origin (one scene build: only its tables are used)
    std::vector<float> mv;
    for (int i = 0; i < 60; ++i) mv.push_back((float)uniform(-0.3, 1.7));
    std::vector<uint32_t> mt;
    for (uint32_t i = 0; i + 2 < 20; ++i) mt.insert(mt.end(), {i, i + 1, i + 2});
    pxr_body_desc mesh = body(PXR_MESH, 0, 0);
    mesh.mesh_verts = mv.data();
    mesh.mesh_tris = mt.data();
    mesh.n_mesh_verts = 20;
    mesh.n_mesh_tris = (uint32_t)mt.size() / 3;
    const std::vector<pxr_body_desc> bodies = {body(PXR_CAPSULE, 12, 6), body(PXR_SPHERE, 16, 8), body(PXR_BOX, 4, 0), mesh};
    pxr_scene_desc d{};
    d.width = d.height = 64;
    d.n_bodies = (uint32_t)bodies.size();
    d.bodies = bodies.data();
    d.fov_y_deg = 60.0f;
    d.cam_offset[0] = -2.5f;
    d.cam_up[2] = 1.0f;
    d.z_near = 0.1f;
    d.z_far = 50.0f;
    d.light_dir[2] = 1.0f;
    d.ground_cell = 1.0f;
    pxr::HostScene hs;
    std::string err;
    if (pxr::build_host_scene(d, hs, err) != PXR_OK || hs.body_bound.size() != bodies.size() * 4) {
        std::fprintf(stderr, "scene: %s\n", err.c_str());
        return 1;
    }

    long seen = 0, outside = 0, near_plane = 0, total = 0;
    for (int n = 0; n < scenes; ++n) {
        // a camera (any rotation, unit up to rounding), an image, and a unit of length over the float range
        const int exponent = chance(0.25) ? (int)(gen() % 250) - 125 : 0;
        const float unit = std::ldexp(1.0f, exponent), z_near = 0.1f * unit;
        const uint32_t size[2] = {8u + (uint32_t)(gen() % 505), 8u + (uint32_t)(gen() % 505)};
        const float half[2] = {0.5f * (float)size[0], 0.5f * (float)size[1]};
        const float focal = (float)(0.5 * size[1] / std::tan(uniform(0.1, 1.4)));
        for (uint32_t b = 0; b < bodies.size(); ++b) {
            // M = a rotation, scaled (a quaternion need not have unit length) or collapsed; t; shape of either sign
            float q[4], M[3][3], t[3], shape[4];
            for (float& c : q) c = (float)uniform(-1.0, 1.0);
            const double len = std::sqrt((double)q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
            const double stretch = chance(0.7) ? 1.0 : chance(0.1) ? 0.0 : uniform(0.3, 2.0);
            for (float& c : q) c = (float)(c / len * stretch);
            const float w = q[0], x = q[1], y = q[2], z = q[3];
            const float R[3][3] = {{1.0f - 2.0f * (y * y + z * z), 2.0f * (x * y - w * z), 2.0f * (x * z + w * y)},
                                   {2.0f * (x * y + w * z), 1.0f - 2.0f * (x * x + z * z), 2.0f * (y * z - w * x)},
                                   {2.0f * (x * z - w * y), 2.0f * (y * z + w * x), 1.0f - 2.0f * (x * x + y * y)}};
            std::memcpy(M, R, sizeof(M));
            const double far = chance(0.3) ? 1.0 : uniform(1.0, 6.0), spread = chance(0.3) ? 4.0 : 0.8;
            t[2] = (float)uniform(-0.3, 1.0) * 0.6f * unit + (chance(0.8) ? (float)far : 0.0f) * unit;
            for (int i = 0; i < 2; ++i) t[i] = (float)(uniform(-spread, spread) * far) * unit;
            const float scale = (float)std::exp(uniform(-4.0, 0.2));
            for (float& s : shape) s = (float)uniform(-1.0, 1.0) * scale * unit;
            if (chance(0.1)) shape[gen() % 4] = 0.0f;

            // the bound
            const float* bound = &hs.body_bound[b * 4];
            float lo[3], hi[3];
            for (int i = 0; i < 3; ++i) {
                const float e = pxr::half_extent(M[i][0], M[i][1], M[i][2], t[i], shape[0], shape[1], shape[2], shape[3], bound[0],
                                                 bound[1], bound[2], bound[3], [](float v) { return one_ulp_off(std::sqrt(v)); });
                lo[i] = t[i] - e;
                hi[i] = t[i] + e;
            }
            const float near_inv = rough_reciprocal(lo[2]), far_inv = rough_reciprocal(hi[2]);
            const pxr::AxisReach axis[2] = {
                pxr::axis_reach(lo[0], hi[0], lo[2], hi[2], near_inv, far_inv, focal, half[0], size[0], z_near),
                pxr::axis_reach(-hi[1], -lo[1], lo[2], hi[2], near_inv, far_inv, focal, half[1], size[1], z_near)};

            // the vertices
            int least[2] = {INT32_MAX, INT32_MAX}, most[2] = {INT32_MIN, INT32_MIN};
            int behind = 0, in_front = 0;
            for (uint32_t v = 0; v < hs.c.V; ++v) {
                uint32_t code;
                std::memcpy(&code, &hs.vtmpl[v * 4 + 3], 4);
                if (code >> 2 != b) continue;
                const float* u = &hs.vtmpl[v * 4];
                const float lx = shape[0] * u[0], ly = shape[1] * u[1], lz = std::fmaf(shape[2], u[2], (float)((int)(code & 3u) - 1) * shape[3]);
                float pv[3];
                for (int i = 0; i < 3; ++i) pv[i] = std::fmaf(M[i][0], lx, std::fmaf(M[i][1], ly, std::fmaf(M[i][2], lz, t[i])));
                if (pv[2] < z_near) {
                    ++behind;
                    continue;
                }
                ++in_front;
                const float inv = 1.0f / pv[2];
                const float s[2] = {std::fmaf(focal, pv[0] * inv, half[0]), std::fmaf(-focal, pv[1] * inv, half[1])};
                if (!(std::fabs(s[0]) <= 16384.0f) || !(std::fabs(s[1]) <= 16384.0f)) continue;
                for (int i = 0; i < 2; ++i) {
                    const int snapped = (int)std::floor(std::fmaf(s[i], 256.0f, 0.5f));
                    least[i] = std::min(least[i], snapped);
                    most[i] = std::max(most[i], snapped);
                }
            }
            ++total;
            if (behind && in_front) {  // triangles to be clipped: they may reach anywhere
                ++near_plane;
                for (int i = 0; i < 2; ++i)
                    if (axis[i].begin != 0u || axis[i].end != size[i]) return fail("crosses the near plane", n, b, axis[i], 0, 0);
                continue;
            }
            if (least[0] > most[0]) continue;  // no usable vertex: any bound will do
            bool none = false, far_out = false;
            for (int i = 0; i < 2; ++i) {
                const int first = std::max(0, (least[i] + 127) >> 8), last = std::min((int)size[i] - 1, (most[i] - 128) >> 8);
                if (first > last) none = true;
                if (most[i] < -256 * 1024 || least[i] > 256 * 1024) far_out = true;
            }
            for (int i = 0; !none && i < 2; ++i) {
                const int first = std::max(0, (least[i] + 127) >> 8), last = std::min((int)size[i] - 1, (most[i] - 128) >> 8);
                if ((int)axis[i].begin > first || (int)axis[i].end <= last) return fail("pixels cut off", n, b, axis[i], first, last);
            }
            if (none) ++outside;
            else ++seen;
            // a small body far out of the image along one axis: the bound says so on that axis
            if (far_out && lo[2] > 0.5f * hi[2] && lo[2] > z_near && !axis[0].none() && !axis[1].none() && hi[2] <= pxr::kReachDepthMax &&
                lo[2] >= pxr::kReachDepthMin)
                return fail("far out of view, yet touched", n, b, axis[0], least[0] >> 8, most[0] >> 8);
        }
    }
    std::printf("ok %ld %ld %ld %ld\n", total, seen, outside, near_plane);
    return 0;
}
