// C ABI of libpxr (declared in include/pxr.h): argument checking, scene
// lifetime, distractor binding and the launch of the render kernel.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <utility>

#include "pxr_internal.h"

struct pxr_scene {
    pxr::SceneConsts sc{};
    pxr::DistractConsts dc{};
    void* d_arena = nullptr;
    pxr::SkeletonConsts sk{};
    void* d_skeleton = nullptr;
    int device = 0;
    uint32_t block_threads = 0;    // of launches that fill the device, or those of every launch if the caller has chosen
    uint32_t default_threads = 0;
    bool threads_chosen = false;
    uint32_t n_cus = 0;
};

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string& msg) {
    g_last_error = msg;
    return code;
}

}  // namespace

int pxr::set_error(int code, const std::string& msg) { return fail(code, msg); }

void pxr::scene_shape(const pxr_scene* s, uint32_t* K, uint32_t* H, uint32_t* W) {
    *K = s->sc.K;
    *H = s->sc.H;
    *W = s->sc.W;
}

namespace {

// How many workgroups a compute unit's LDS holds: it is handed out in steps of 1280 bytes.  (Meshes of 40x40, 30 016 bytes a frame, are five: 1280
// frames in workgroups of 256 threads take 14.7 us, one round.  Chains of 32x32, 32 528 bytes, are four and not five: 15.5 us, 10.2 for 1024.)
uint32_t groups_in_lds(const pxr::SceneConsts& sc) {
    const uint32_t steps = 160u * 1024u / 1280u, per_group = (sc.lds_total + 1279u) / 1280u;
    return steps / std::max(per_group, 1u);
}

// How many of a compute unit's workgroups are resident: what its LDS holds, and its 32 wave slots.  (The kernels for whole frames take 61 or 62
// vector and at most 80 scalar registers, eight wavefronts per SIMD.  The windowed ones of up to 768 threads take 70, seven per SIMD, but
// the LDS holds two of their workgroups at most, 24 wavefronts.)
uint32_t resident_groups(const pxr::SceneConsts& sc, uint32_t threads) { return std::min(groups_in_lds(sc), 2048u / threads); }

uint32_t pick_block_threads(const pxr::SceneConsts& sc) {
    // Fill the 32 wave slots of a compute unit: LDS decides how many frame workgroups are resident, the workgroup size makes up the rest.
    // us for 25 million pixels, 256 / 512 threads, by the workgroups in LDS: 7 (meshes 32x32) 138 / 174, 6 (capsules 48x48) 58.0 / 71.5, 5
    // (meshes 40x40) 133 / 139; 4 (capsules 64x64) 54.6 / 51.7, (chains 48x48) 108 / 92, (meshes 56x56) 111 / 90.5, (meshes 38x48 over a clip)
    // 173 / 145; 3 (quadrupeds 48x48) 163 / 120.
    const uint32_t groups_per_cu = groups_in_lds(sc);
    if (groups_per_cu >= 5) return 256;
    if (groups_per_cu >= 3) return 512;
    if (groups_per_cu == 2 && sc.key_capacity && sc.npix < pxr::kWideWindowedFrom) return 768;
    return 1024;
}

// Workgroup size of a launch: few frames leave compute units with fewer workgroups than their LDS would hold, and these then share its wave slots.
uint32_t launch_threads(const pxr_scene* s, uint64_t n_frames) {
    const uint32_t in_lds = groups_in_lds(s->sc);
    if (s->threads_chosen || in_lds < 3u) return s->block_threads;
    const uint64_t per_cu = (n_frames + s->n_cus - 1u) / s->n_cus;
    // One workgroup on a compute unit takes all the wavefronts that it has use for.  us for 256 frames, 256 / 512 / 1024 threads: meshes 64x64 15.3 /
    // 10.7 / 8.7, quadrupeds 48x48 12.3 / 8.6 / 7.4, chains 32x32 8.5 / 7.0 / 6.7; capsules, of 264 vertices, 40x40 7.0 / 6.4 / 6.6, 56x56 8.6 / 7.4 / 7.2.
    if (per_cu <= 1u) return s->sc.V >= 512u ? 1024u : 512u;
    if (in_lds <= 4u) return 512u;
    // From five workgroups in LDS on, 512 threads as long as that takes no more rounds: a frame is done sooner.  us, 256 / 512 threads: meshes
    // 40x40 (five), 1024 frames 13.0 / 12.5, 1280 14.7 / 16.9, 1536 20.7 / 18.3, 2792 30.6 / 29.1, 4096 40.8 / 40.4; meshes 28x28 (six), 1024
    // frames 10.2 / 9.9, 1280 11.2 / 13.0, 2048 17.5 / 17.3.  Frames of few vertices have less to gain: capsules 48x48 (six), 768 frames 8.6 / 8.4, 1024
    // 9.4 / 9.6, 2048 16.3 / 17.1; 40x40 (eight), 512 frames 7.5 / 7.3, 768 7.9 / 8.2.
    if (s->sc.V < 512u) return per_cu <= (in_lds < 8u ? 3u : 2u) ? 512u : 256u;
    const uint64_t wide = resident_groups(s->sc, 512u), narrow = resident_groups(s->sc, 256u);
    return (per_cu + wide - 1u) / wide <= (per_cu + narrow - 1u) / narrow ? 512u : 256u;
}

// pxr::render_envs, which takes the poses as they are (fk null), or makes them in the same launch.
int render_posed(pxr_scene* s, const pxr::FkArgs* fk, const float* d_poses, const float* d_shapes, uint32_t e0, uint32_t n, uint32_t S,
                 uint32_t step0, uint32_t env0, uint8_t* d_frames, uint32_t* d_ids, void* stream, std::string& err) {
    if (n == 0 || S == 0 || (uint64_t)n * S > 0x7FFFFFFFull) {
        err = "B*S must lie in [1, 2^31-1]";
        return PXR_ERR_INVALID_ARG;
    }
    if ((uint64_t)step0 + S > 0x100000000ull || (uint64_t)env0 + e0 + n > 0x100000000ull) {
        err = "step0 + S or env0 + B overflows 32 bits";
        return PXR_ERR_INVALID_ARG;
    }
    const size_t K = s->sc.K, npix = s->sc.npix;
    const float* poses = d_poses + (size_t)e0 * S * K * 7;
    const float* shapes = d_shapes ? d_shapes + (size_t)e0 * K * 4 : nullptr;
    uint8_t* frames = d_frames + (size_t)e0 * S * npix * 3;
    uint32_t* ids = d_ids ? d_ids + (size_t)e0 * S * npix : nullptr;
    if ((reinterpret_cast<uintptr_t>(poses) & 3u) || (reinterpret_cast<uintptr_t>(shapes) & 15u) ||
        (reinterpret_cast<uintptr_t>(frames) & 3u) || (reinterpret_cast<uintptr_t>(ids) & 15u)) {
        err = "poses/frames must be 4-byte and shapes/ids 16-byte aligned";
        return PXR_ERR_INVALID_ARG;
    }
    pxr::DistractConsts dc = s->dc;  // the per-environment arrays follow the environments
    if (dc.env_offset) dc.env_offset += e0;
    if (dc.env_video) dc.env_video += e0;
    return pxr::launch_render(s->sc, dc, fk, poses, shapes, n * S, S, step0, env0 + e0, frames, ids, launch_threads(s, (uint64_t)n * S), s->n_cus, stream, err);
}

}  // namespace

int pxr::render_envs(pxr_scene* s, const float* d_poses, const float* d_shapes, uint32_t e0, uint32_t n, uint32_t S,
                     uint32_t step0, uint32_t env0, uint8_t* d_frames, uint32_t* d_ids, void* stream, std::string& err) {
    return render_posed(s, nullptr, d_poses, d_shapes, e0, n, S, step0, env0, d_frames, d_ids, stream, err);
}

namespace {

// The kernels' dynamic-LDS caps are raised once per device and process, by the first scene created there.
int prepare_device_once(int device, std::string& err) {
    static std::mutex mu;
    static bool done[64] = {};
    if (device < 0 || device >= 64) return pxr::prepare_kernels(err);
    std::lock_guard<std::mutex> lock(mu);
    if (done[device]) return PXR_OK;
    const int rc = pxr::prepare_kernels(err);
    if (rc == PXR_OK) done[device] = true;
    return rc;
}

}  // namespace

extern "C" {

const char* pxr_last_error(void) { return g_last_error.c_str(); }

int pxr_create_scene(const pxr_scene_desc* desc, pxr_scene** out) {
    if (!desc || !out) return fail(PXR_ERR_INVALID_ARG, "pxr_create_scene: null argument");
    pxr::HostScene hs;
    std::string err;
    int rc = pxr::build_host_scene(*desc, hs, err);
    if (rc != PXR_OK) return fail(rc, "pxr_create_scene: " + err);

    // one arena, 256-byte aligned sub-tables, one synchronous upload
    struct Part {
        const void* src;
        size_t bytes;
        size_t off;
    };
    // The device copy of the pair table holds, in place of the four vertex indices, the LDS byte addresses of
    // the vertices' cell codes (the kernel reads them without any address arithmetic, and two of them without unpacking): code v sits at
    // lds_keys + 4 v of the dynamic LDS segment, which starts at address 0 (prepare_kernels checks that the
    // kernels have no static LDS in front of it).
    // It is padded to a multiple of 64 entries (a wavefront reads 64 without a bounds test) with entries that
    // hold no triangle and point four times at the word after the last code, which the kernel sets to code 0.
    if ((uint64_t)hs.c.lds_keys + 4ull * (hs.c.V + 1ull) > 0x10000ull)
        return fail(PXR_ERR_UNSUPPORTED, "pxr_create_scene: too many vertices for 16-bit LDS addresses in the pair table");

    pxr_scene* s = new (std::nothrow) pxr_scene();
    if (!s) return fail(PXR_ERR_OOM, "pxr_create_scene: host allocation failed");
    s->sc = hs.c;
    int n_cus = 0;
    if (hipGetDevice(&s->device) != hipSuccess ||
        hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, s->device) != hipSuccess) {
        delete s;
        return fail(PXR_ERR_DEVICE, "pxr_create_scene: no HIP device");
    }
    s->n_cus = (uint32_t)n_cus;
    std::vector<uint32_t> pair_dev;
    const auto code_at = [&](uint32_t v) { return hs.c.lds_keys + 4u * v; };
    const auto add_entry = [&](uint32_t q0, uint32_t q1, uint32_t q2, uint32_t q3, uint32_t triangles) {
        for (uint32_t word : {code_at(q0) | (code_at(q1) << 16), code_at(q2), code_at(q3), triangles}) pair_dev.push_back(word);
    };
    for (size_t p = 0; p < hs.pair_tbl.size(); p += 4)
        add_entry(hs.pair_tbl[p] & 0xFFFFu, hs.pair_tbl[p] >> 16, hs.pair_tbl[p + 1] & 0xFFFFu, hs.pair_tbl[p + 1] >> 16, hs.pair_tbl[p + 2]);
    while ((pair_dev.size() / 4) % 64 != 0)
        add_entry(hs.c.V, hs.c.V, hs.c.V, hs.c.V, pxr::kNoTriangle | (pxr::kNoTriangle << 16));
    // Likewise the device copy of the vertex templates: its fourth word holds the LDS address of the body's
    // record, in units of 16 bytes, and the cap selector as a half float (-1, 0, +1) above it, in
    // place of body << 2 | (selector + 1).
    std::vector<float> vtmpl_dev(hs.vtmpl);
    for (size_t v = 0; v < vtmpl_dev.size() / 4; ++v) {
        uint32_t code;
        std::memcpy(&code, &hs.vtmpl[v * 4 + 3], 4);
        const uint32_t body_at = hs.c.lds_body + (code >> 2) * pxr::kBodyStride * 4u;
        constexpr uint32_t kHalfFloat[3] = {0xBC00u, 0x0000u, 0x3C00u};
        const uint32_t dev = (body_at / 16u) | (kHalfFloat[code & 3u] << 16);
        std::memcpy(&vtmpl_dev[v * 4 + 3], &dev, 4);
    }
    vtmpl_dev.resize((hs.c.V + 63u) / 64u * 64u * 4u, 0.0f);  // (a wavefront reads 64 without a bounds test)
    // Behind the bodies' constants: the rows (right, up, forward) of the view rotation and the light direction, for
    // the lanes of the kernel's set-up phase that take one row each.
    std::vector<float> body_dev(hs.body_const);
    for (const float* row : {hs.c.Rt, hs.c.Up, hs.c.Fw, hs.c.l}) body_dev.insert(body_dev.end(), row, row + 3);
    body_dev.insert(body_dev.end(), hs.body_bound.begin(), hs.body_bound.end());
    // The checker's parity is the sum of two cell indices, whichever of them is called x.  A camera along the y axis (its right vector's y is a
    // zero) is given to the kernel as one along the x axis, whose rows share the x index.
    if (s->sc.Rt[1] == 0.0f && s->sc.Rt[0] != 0.0f) {
        s->sc.eye_first = 1u;
        for (float* row : {s->sc.Rt, s->sc.Up, s->sc.Fw}) std::swap(row[0], row[1]);
    }
    // And the device copy of the index table has, in place of a triangle's body, where that body's record is.
    std::vector<uint32_t> tri_dev(hs.tri_idx);
    for (size_t t = 1; t < tri_dev.size(); t += 2)
        tri_dev[t] = (tri_dev[t] & 0xFFFFu) | ((hs.c.lds_body / 16u + (tri_dev[t] >> 16) * (pxr::kBodyStride / 4u)) << 16);
    Part parts[6] = {{vtmpl_dev.data(), vtmpl_dev.size() * 4, 0},
                     {tri_dev.data(), tri_dev.size() * 4, 0},
                     {hs.tri_shade.data(), hs.tri_shade.size() * 4, 0},
                     {body_dev.data(), body_dev.size() * 4, 0},
                     {hs.cxcy.data(), hs.cxcy.size() * 4, 0},
                     {pair_dev.data(), pair_dev.size() * 4, 0}};
    size_t total = 0;
    for (Part& p : parts) {
        p.off = total;
        total += (p.bytes + 255) / 256 * 256;
    }
    std::vector<unsigned char> staging(total, 0);
    for (const Part& p : parts) std::memcpy(staging.data() + p.off, p.src, p.bytes);
    hipError_t hrc = hipMalloc(&s->d_arena, total);
    if (hrc != hipSuccess) {
        delete s;
        return fail(hrc == hipErrorOutOfMemory ? PXR_ERR_OOM : PXR_ERR_DEVICE,
                    std::string("pxr_create_scene: hipMalloc failed: ") + hipGetErrorString(hrc));
    }
    hrc = hipMemcpy(s->d_arena, staging.data(), total, hipMemcpyHostToDevice);
    if (hrc != hipSuccess) {
        (void)hipFree(s->d_arena);
        delete s;
        return fail(PXR_ERR_DEVICE, std::string("pxr_create_scene: upload failed: ") + hipGetErrorString(hrc));
    }
    const unsigned char* base = static_cast<const unsigned char*>(s->d_arena);
    s->sc.vtmpl = reinterpret_cast<const float*>(base + parts[0].off);
    s->sc.tri_idx = reinterpret_cast<const uint32_t*>(base + parts[1].off);
    s->sc.tri_shade = reinterpret_cast<const float*>(base + parts[2].off);
    s->sc.body_const = reinterpret_cast<const float*>(base + parts[3].off);
    s->sc.cxcy = reinterpret_cast<const float*>(base + parts[4].off);
    s->sc.pair_tbl = reinterpret_cast<const uint32_t*>(base + parts[5].off);
    s->sc.P = (uint32_t)(pair_dev.size() / 4);  // (with the padding)

    rc = prepare_device_once(s->device, err);
    if (rc != PXR_OK) {
        (void)hipFree(s->d_arena);
        delete s;
        return fail(rc, "pxr_create_scene: " + err);
    }
    s->default_threads = s->block_threads = pick_block_threads(s->sc);
    s->dc.mode = PXR_DISTRACT_NONE;
    *out = s;
    return PXR_OK;
}

int pxr_destroy_scene(pxr_scene* s) {
    if (!s) return PXR_OK;
    hipError_t hrc = hipFree(s->d_arena);
    if (s->d_skeleton) {
        const hipError_t hrc2 = hipFree(s->d_skeleton);
        if (hrc == hipSuccess) hrc = hrc2;
    }
    delete s;
    if (hrc != hipSuccess) return fail(PXR_ERR_DEVICE, std::string("pxr_destroy_scene: hipFree failed: ") + hipGetErrorString(hrc));
    return PXR_OK;
}

int pxr_apply_distractor(pxr_scene* s, const pxr_distractor_desc* d) {
    if (!s) return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: null scene");
    pxr::DistractConsts dc{};
    dc.mode = PXR_DISTRACT_NONE;
    if (d && d->mode != PXR_DISTRACT_NONE) {
        dc.seed_lo = (uint32_t)d->seed;
        dc.seed_hi = (uint32_t)(d->seed >> 32);
        if (d->mode == PXR_DISTRACT_COLOR) {
            if (!std::isfinite(d->scale_lo) || !std::isfinite(d->scale_hi) || !std::isfinite(d->offset_lo) ||
                !std::isfinite(d->offset_hi))
                return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: non-finite colour range");
            dc.mode = PXR_DISTRACT_COLOR;
            dc.scale_lo = d->scale_lo;
            dc.scale_span = d->scale_hi - d->scale_lo;
            dc.offset_lo = d->offset_lo;
            dc.offset_span = d->offset_hi - d->offset_lo;
        } else if (d->mode == PXR_DISTRACT_VIDEO) {
            if (!d->d_video || d->n_frames == 0)
                return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: video mode needs d_video and n_frames > 0");
            if (!(d->alpha >= 0.0f && d->alpha <= 1.0f))
                return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: alpha must lie in [0,1]");
            if ((reinterpret_cast<uintptr_t>(d->d_video) & 3u) || (reinterpret_cast<uintptr_t>(d->d_env_offset) & 3u) ||
                (reinterpret_cast<uintptr_t>(d->d_env_video) & 3u))
                return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: d_video, d_env_offset and d_env_video must be 4-byte aligned");
            if ((uint64_t)(d->n_videos ? d->n_videos : 1u) * d->n_frames > 0xFFFFFFFFull)
                return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: n_videos * n_frames overflows 32 bits");
            dc.mode = PXR_DISTRACT_VIDEO;
            dc.video = d->d_video;
            dc.n_frames = d->n_frames;
            dc.alpha = d->alpha;
            dc.env_offset = d->d_env_offset;
            dc.n_videos = d->n_videos ? d->n_videos : 1u;
            dc.env_video = dc.n_videos > 1 ? d->d_env_video : nullptr;
        } else {
            return fail(PXR_ERR_INVALID_ARG, "pxr_apply_distractor: unknown mode");
        }
    }
    s->dc = dc;
    return PXR_OK;
}

int pxr_render_batch(pxr_scene* s, const float* d_poses, const float* d_shapes, uint32_t B, uint32_t S, uint32_t step0,
                     uint32_t env0, uint8_t* d_frames, uint32_t* d_ids, void* hip_stream) {
    if (!s || !d_poses || !d_frames) return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch: null scene, poses or frames");
    std::string err;
    const int rc = pxr::render_envs(s, d_poses, d_shapes, 0, B, S, step0, env0, d_frames, d_ids, hip_stream, err);
    if (rc != PXR_OK) return fail(rc, "pxr_render_batch: " + err);
    return PXR_OK;
}

int pxr_set_skeleton(pxr_scene* s, const pxr_skeleton_desc* k) {
    if (!s) return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: null scene");
    if (!k) {
        if (s->d_skeleton) (void)hipFree(s->d_skeleton);
        s->d_skeleton = nullptr;
        s->sk = pxr::SkeletonConsts{};
        return PXR_OK;
    }
    if (!k->parent || !k->slot || !k->anchor || !k->axis || !k->offset)
        return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: null array");
    const uint32_t K = s->sc.K;
    if (k->n_bodies != K) return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: n_bodies differs from the scene's");
    for (uint32_t b = 0; b < K; ++b) {
        const int32_t p = k->parent[b], sl = k->slot[b];
        if (p < 0) {
            if (sl < 0 || (uint32_t)sl >= k->n_free)
                return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: a free body needs a slot in [0, n_free)");
        } else {
            if ((uint32_t)p >= b) return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: a parent must precede its child");
            if (sl < -1 || (sl >= 0 && (uint32_t)sl >= k->n_angles))
                return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: hinge slot outside [-1, n_angles)");
        }
        for (int c = 0; c < 3; ++c)
            if (!std::isfinite(k->anchor[b * 3 + c]) || !std::isfinite(k->axis[b * 3 + c]) ||
                !std::isfinite(k->offset[b * 3 + c]))
                return fail(PXR_ERR_INVALID_ARG, "pxr_set_skeleton: non-finite anchor, axis or offset");
    }
    pxr::SkeletonConsts sk{};
    sk.K = K;
    sk.J = k->n_angles;
    sk.F = k->n_free;
    // (a limit of the interface: the kernel itself keeps only the poses in LDS, 64 * (7 K | 1) floats, for K <= 64 at most 115 KB)
    if ((uint64_t)sk.J + 7ull * sk.F + 7ull * K > 630ull)
        return fail(PXR_ERR_UNSUPPORTED, "pxr_set_skeleton: 7*n_bodies + 7*n_free + n_angles must not exceed 630");
    // one allocation: the records in order of depth (a parent precedes its child, so one pass finds the depths), then
    // where each depth begins, then the records' links
    std::vector<uint32_t> depth(K), begin(1, 0u), links;
    std::vector<pxr::SkeletonRecord> records;
    for (uint32_t b = 0; b < K; ++b) depth[b] = k->parent[b] < 0 ? 0u : depth[(uint32_t)k->parent[b]] + 1u;
    for (uint32_t d = 0; records.size() < K; ++d) {
        for (uint32_t b = 0; b < K; ++b) {
            if (depth[b] != d) continue;
            pxr::SkeletonRecord r{};
            r.body = b;
            r.parent = k->parent[b];
            uint32_t parent_record = 0;
            while (d > 0 && records[parent_record].body != (uint32_t)r.parent) ++parent_record;
            links.push_back(d | (parent_record << 16));
            r.slot = k->slot[b];
            for (int c = 0; c < 3; ++c) {
                r.anchor[c] = k->anchor[b * 3 + c];
                r.axis[c] = k->axis[b * 3 + c];
                r.offset[c] = k->offset[b * 3 + c];
            }
            records.push_back(r);
        }
        begin.push_back((uint32_t)records.size());
    }
    sk.depths = (uint32_t)begin.size() - 1u;
    std::vector<uint32_t> staging(K * (sizeof(pxr::SkeletonRecord) / 4) + begin.size() + K);
    std::memcpy(staging.data(), records.data(), K * sizeof(pxr::SkeletonRecord));
    std::memcpy(staging.data() + K * (sizeof(pxr::SkeletonRecord) / 4), begin.data(), begin.size() * 4);
    std::memcpy(staging.data() + K * (sizeof(pxr::SkeletonRecord) / 4) + begin.size(), links.data(), K * 4);
    std::string err;
    int rc = pxr::prepare_fk_kernel(err);
    if (rc != PXR_OK) return fail(rc, "pxr_set_skeleton: " + err);
    void* d = nullptr;
    hipError_t hrc = hipMalloc(&d, staging.size() * 4);
    if (hrc != hipSuccess)
        return fail(hrc == hipErrorOutOfMemory ? PXR_ERR_OOM : PXR_ERR_DEVICE,
                    std::string("pxr_set_skeleton: hipMalloc failed: ") + hipGetErrorString(hrc));
    hrc = hipMemcpy(d, staging.data(), staging.size() * 4, hipMemcpyHostToDevice);
    if (hrc != hipSuccess) {
        (void)hipFree(d);
        return fail(PXR_ERR_DEVICE, std::string("pxr_set_skeleton: upload failed: ") + hipGetErrorString(hrc));
    }
    {
        // set-up is the place to look up this device's copy of the static pose buffer (used by
        // pxr_render_batch_kinematic_static), so that the hot call finds it cached
        float* unused = nullptr;
        std::string e2;
        (void)pxr::static_pose_scratch(&unused, nullptr, e2);
    }
    if (s->d_skeleton) (void)hipFree(s->d_skeleton);
    s->d_skeleton = d;
    sk.records = static_cast<const pxr::SkeletonRecord*>(d);
    sk.depth_begin = reinterpret_cast<const uint32_t*>(sk.records + K);
    sk.links = sk.depth_begin + begin.size();
    s->sk = sk;
    return PXR_OK;
}

namespace {

int check_pose_batch(const pxr_scene* s, const float* d_free_poses, const float* d_angles, uint32_t n_frames, const float* d_poses) {
    if (!s) return fail(PXR_ERR_INVALID_ARG, "pxr_pose_batch: null scene");
    if (!s->d_skeleton) return fail(PXR_ERR_INVALID_ARG, "pxr_pose_batch: no skeleton bound (pxr_set_skeleton)");
    if (n_frames == 0 || n_frames > 0x7FFFFFFFu) return fail(PXR_ERR_INVALID_ARG, "pxr_pose_batch: n_frames must lie in [1, 2^31-1]");
    if (!d_poses || (s->sk.F && !d_free_poses) || (s->sk.J && !d_angles))
        return fail(PXR_ERR_INVALID_ARG, "pxr_pose_batch: null buffer");
    if ((reinterpret_cast<uintptr_t>(d_free_poses) & 3u) || (reinterpret_cast<uintptr_t>(d_angles) & 3u) ||
        (reinterpret_cast<uintptr_t>(d_poses) & 3u))
        return fail(PXR_ERR_INVALID_ARG, "pxr_pose_batch: buffers must be 4-byte aligned");
    return PXR_OK;
}

}  // namespace

int pxr_pose_batch(pxr_scene* s, const float* d_free_poses, const float* d_angles, uint32_t n_frames, float* d_poses,
                   void* hip_stream) {
    int rc = check_pose_batch(s, d_free_poses, d_angles, n_frames, d_poses);
    if (rc != PXR_OK) return rc;
    std::string err;
    rc = pxr::launch_fk(s->sk, d_free_poses, d_angles, n_frames, d_poses, hip_stream, err);
    if (rc != PXR_OK) return fail(rc, "pxr_pose_batch: " + err);
    return PXR_OK;
}

namespace {

constexpr uint64_t kPosedRoundsTimesDepths = 20;

bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return a && b && p < q + b_bytes && q < p + a_bytes;
}

// Whether the render kernel makes the poses itself, in the same launch.  That saves the kinematics kernel's launch (4 to 5 us) and
// costs every round of workgroups the chain of steps from the angles to the poses: about as long for a tree of d depths as
// d + 1 times 0.25 us.  (A round is what is resident with either kernel: the pose-making ones take no more registers than the others.)
// us per call, two launches / one, 64x64 unless said otherwise: humanoid (4 depths) 1 frame 11.9 / 9.0, 256 frames 13.9 / 9.9, 1024 (two
// rounds) 27.4 / 24.2, 2048 (four) 45.4 / 44.0, 4096 (eight) 81.0 / 83.0; quadruped (3 depths) 256 frames 11.7 / 8.9, 2048 38.9 / 38.6, at worst 2560
// 46.5 / 47.1, 4096 68.9 / 72.3; chain (7 depths) 256 frames 13.2 / 10.3, 1024 24.3 / 23.1, 1280 28.9 / 29.4; chains of 48x48 (four resident) 1024
// frames 17.2 / 14.3, 2048 26.8 / 25.7, 2560 31.3 / 31.4, 4096 43.7 / 46.2; quadrupeds of 256x256 (a workgroup per compute unit), 256 frames
// 34.5 / 30.6, 1280 130.7 / 129.3, 1800 188.8 / 189.9.
bool worth_one_launch(const pxr_scene* s, uint64_t n_frames) {
    const uint32_t threads = launch_threads(s, n_frames), per_cu = resident_groups(s->sc, threads);
    if (!pxr::makes_poses(threads, s->sc.key_capacity != 0u)) return false;
    const uint64_t resident = (uint64_t)per_cu * s->n_cus, rounds = (n_frames + resident - 1) / resident;
    return rounds * (s->sk.depths + 1u) <= kPosedRoundsTimesDepths;
}

bool poses_made_by_renderer(const pxr_scene* s, const float* d_free_poses, const float* d_angles, const float* d_shapes, uint32_t B,
                            uint64_t n_frames, const float* d_poses, const uint8_t* d_frames, const uint32_t* d_ids) {
    if (!worth_one_launch(s, n_frames)) return false;
    // (a caller may let the outputs take the place of the angles or the free poses: then all of these are read first)
    const size_t free_bytes = n_frames * s->sk.F * 28, angle_bytes = n_frames * s->sk.J * 4, pose_bytes = n_frames * s->sc.K * 28,
                 frame_bytes = n_frames * s->sc.npix * 3, id_bytes = n_frames * s->sc.npix * 4;
    for (int out = 0; out < 3; ++out) {
        const void* p = out == 0 ? (const void*)d_poses : (out == 1 ? (const void*)d_frames : (const void*)d_ids);
        const size_t bytes = out == 0 ? pose_bytes : (out == 1 ? frame_bytes : id_bytes);
        if (overlap(p, bytes, d_free_poses, free_bytes) || overlap(p, bytes, d_angles, angle_bytes)) return false;
    }
    // (and all poses are written before the rest of the inputs is read and before a frame is written)
    const pxr::DistractConsts& dc = s->dc;
    return !overlap(d_poses, pose_bytes, d_frames, frame_bytes) && !overlap(d_poses, pose_bytes, d_ids, id_bytes) &&
           !overlap(d_poses, pose_bytes, d_shapes, (size_t)B * s->sc.K * 16) && !overlap(d_poses, pose_bytes, dc.env_offset, (size_t)B * 4) &&
           !overlap(d_poses, pose_bytes, dc.env_video, (size_t)B * 4) &&
           !overlap(d_poses, pose_bytes, dc.video, (size_t)dc.n_videos * dc.n_frames * s->sc.npix * 3);
}

}  // namespace

int pxr_render_batch_kinematic(pxr_scene* s, const float* d_free_poses, const float* d_angles, const float* d_shapes,
                               uint32_t B, uint32_t S, uint32_t step0, uint32_t env0, float* d_poses, uint8_t* d_frames,
                               uint32_t* d_ids, void* hip_stream) {
    if (B == 0 || S == 0 || (uint64_t)B * S > 0x7FFFFFFFull)
        return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch_kinematic: B*S must lie in [1, 2^31-1]");
    if (!d_frames) return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch_kinematic: null frames");
    int rc = check_pose_batch(s, d_free_poses, d_angles, B * S, d_poses);
    if (rc != PXR_OK) return rc;
    if (poses_made_by_renderer(s, d_free_poses, d_angles, d_shapes, B, (uint64_t)B * S, d_poses, d_frames, d_ids)) {
        const pxr::FkArgs fk = {s->sk, d_free_poses, d_angles, d_poses};
        std::string err;
        rc = render_posed(s, &fk, d_poses, d_shapes, 0, B, S, step0, env0, d_frames, d_ids, hip_stream, err);
        if (rc != PXR_OK) return fail(rc, "pxr_render_batch: " + err);
        return PXR_OK;
    }
    rc = pxr_pose_batch(s, d_free_poses, d_angles, B * S, d_poses, hip_stream);
    if (rc != PXR_OK) return rc;
    return pxr_render_batch(s, d_poses, d_shapes, B, S, step0, env0, d_frames, d_ids, hip_stream);
}

int pxr_render_batch_kinematic_static(pxr_scene* s, const float* d_free_poses, const float* d_angles,
                                      const float* d_shapes, uint32_t B, uint32_t S, uint32_t step0, uint32_t env0,
                                      uint8_t* d_frames, uint32_t* d_ids, void* hip_stream) {
    if (!s) return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch_kinematic_static: null scene");
    if (B == 0 || S == 0 || (uint64_t)B * S > 0x7FFFFFFFull)
        return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch_kinematic_static: B*S must lie in [1, 2^31-1]");
    if (!d_frames) return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch_kinematic_static: null frames");
    float* d_poses = nullptr;
    size_t capacity = 0;
    std::string err;
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device != s->device)
        return fail(PXR_ERR_INVALID_ARG, "pxr_render_batch_kinematic_static: the scene's device must be the current one");
    const int rc = pxr::static_pose_scratch(&d_poses, &capacity, err);
    if (rc != PXR_OK) return fail(rc, "pxr_render_batch_kinematic_static: " + err);
    const uint64_t need = (uint64_t)B * S * s->sc.K * 7ull * sizeof(float);
    if (need > capacity)
        return fail(PXR_ERR_UNSUPPORTED, "pxr_render_batch_kinematic_static: B*S*n_bodies*28 = " + std::to_string(need) +
                                             " bytes of poses exceed the library's " + std::to_string(capacity) +
                                             "-byte static buffer; use pxr_render_batch_kinematic with a buffer of your own");
    // (every pose the render kernel reads is written by the kinematics kernel in front of it on the same stream, or made by
    // itself and only written: nothing of an earlier call's contents is used, so nothing needs clearing)
    return pxr_render_batch_kinematic(s, d_free_poses, d_angles, d_shapes, B, S, step0, env0, d_poses, d_frames, d_ids,
                                      hip_stream);
}

int pxr_kinematic_info(const pxr_scene* s, uint32_t n_frames, uint32_t* n_launches) {
    if (!s || !n_launches || n_frames == 0) return fail(PXR_ERR_INVALID_ARG, "pxr_kinematic_info: null argument or n_frames == 0");
    if (!s->d_skeleton) return fail(PXR_ERR_INVALID_ARG, "pxr_kinematic_info: no skeleton bound (pxr_set_skeleton)");
    *n_launches = worth_one_launch(s, n_frames) ? 1u : 2u;
    return PXR_OK;
}

int pxr_scene_info(const pxr_scene* s, uint32_t* n_verts, uint32_t* n_tris, uint32_t* lds_bytes, uint32_t* block_threads) {
    if (!s) return fail(PXR_ERR_INVALID_ARG, "pxr_scene_info: null scene");
    if (n_verts) *n_verts = s->sc.V;
    if (n_tris) *n_tris = s->sc.T;
    if (lds_bytes) *lds_bytes = s->sc.lds_total;
    if (block_threads) *block_threads = s->block_threads;
    return PXR_OK;
}

int pxr_host_tables(const pxr_scene_desc* desc, uint32_t* n_verts, uint32_t* n_tris, float* vtmpl, uint32_t* tri_idx,
                    float* tri_shade, float* cxcy, float* consts, uint32_t* n_pairs, uint32_t* pair_tbl) {
    if (!desc) return fail(PXR_ERR_INVALID_ARG, "pxr_host_tables: null desc");
    pxr::HostScene hs;
    std::string err;
    const int rc = pxr::build_host_scene(*desc, hs, err);
    if (rc != PXR_OK) return fail(rc, "pxr_host_tables: " + err);
    if (n_verts) *n_verts = hs.c.V;
    if (n_tris) *n_tris = hs.c.T;
    if (vtmpl) std::memcpy(vtmpl, hs.vtmpl.data(), hs.vtmpl.size() * 4);
    if (tri_idx) std::memcpy(tri_idx, hs.tri_idx.data(), hs.tri_idx.size() * 4);
    if (tri_shade) std::memcpy(tri_shade, hs.tri_shade.data(), hs.tri_shade.size() * 4);
    if (cxcy) std::memcpy(cxcy, hs.cxcy.data(), hs.cxcy.size() * 4);
    if (n_pairs) *n_pairs = hs.c.P;
    if (pair_tbl)
        for (uint32_t p = 0; p < hs.c.P; ++p)
            for (int w = 0; w < 3; ++w) pair_tbl[p * 3 + w] = hs.pair_tbl[p * 4 + w];
    if (consts) {
        for (int i = 0; i < 3; ++i) {
            consts[i] = hs.c.Rt[i];
            consts[3 + i] = hs.c.Up[i];
            consts[6 + i] = hs.c.Fw[i];
            consts[12 + i] = hs.c.l[i];
        }
        consts[9] = hs.c.f;
        consts[10] = hs.c.gs[0];
        consts[11] = hs.c.gs[1];
        consts[15] = (float)hs.c.lds_total;
    }
    return PXR_OK;
}

int pxr_selftest_arithmetic(uint64_t* counts) {
    if (!counts) return fail(PXR_ERR_INVALID_ARG, "pxr_selftest_arithmetic: null output");
    std::string err;
    unsigned long long c[4] = {0, 0, 0, 0};
    const int rc = pxr::selftest_arithmetic(c, err);
    if (rc != PXR_OK) return fail(rc, "pxr_selftest_arithmetic: " + err);
    for (int i = 0; i < 4; ++i) counts[i] = c[i];
    return PXR_OK;
}

int pxr_measure_peaks(double* fma_tlaneops, double* imad_tlaneops, double* copy_gbs, double* read_gbs, double* write_gbs) {
    std::string err;
    const int rc = pxr::measure_peaks(fma_tlaneops, imad_tlaneops, copy_gbs, read_gbs, write_gbs, err);
    if (rc != PXR_OK) return fail(rc, "pxr_measure_peaks: " + err);
    return PXR_OK;
}

int pxr_set_block_threads(pxr_scene* s, uint32_t threads) {
    if (!s) return fail(PXR_ERR_INVALID_ARG, "pxr_set_block_threads: null scene");
    const bool chosen = threads != 0;
    if (threads == 0) threads = s->default_threads;
    if (threads != 256 && threads != 512 && threads != 768 && threads != 1024)
        return fail(PXR_ERR_INVALID_ARG, "pxr_set_block_threads: must be 256, 512, 768 or 1024");
    s->block_threads = threads;
    s->threads_chosen = chosen;
    return PXR_OK;
}

}  // extern "C"
