// Internal layout shared by the host-side scene builder and the HIP kernels of
// libpxr.  Nothing here is visible through the C ABI (include/pxr.h).
#ifndef PXR_INTERNAL_H
#define PXR_INTERNAL_H

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "pxr.h"

namespace pxr {

// Sentinel stored in the snapped-X array for a vertex that is unusable (outside the
// guard band, or a non-finite depth); any triangle touching it is dropped.
constexpr int32_t kRejectedX = INT32_MIN;
// Sentinel for a vertex behind the near plane: its triangles are clipped against the plane in the
// raster phase.  (Snapped coordinates stay within +-2^22, so both sentinels sort below every real one.)
constexpr int32_t kBehindX = INT32_MIN + 1;

// Raster bins by the number of pixel centres in a surviving triangle's clamped bounding box:
//   tiny  <= kTinyMaxPixels   one lane
//   small <= kSmallMaxPixels  a team of 2^kSmallLanesLog2 lanes, rows dealt round-robin
//   large otherwise           a whole wavefront, rows by columns (also: triangles to be clipped)
// The first two hold narrow triangles only (extents below 2^15 sub-pixels: their loops multiply 24 bits); wide ones of up to kSmallMaxPixels are
// kept apart and take a team each, in 64 bits.
// What is balanced here is the longest chain in the raster phase, not the instruction count: one lane
// walking a 12-pixel triangle holds up its whole workgroup at the next barrier.
constexpr uint32_t kTinyMaxPixels = 3;
constexpr uint32_t kSmallMaxPixels = 128;
constexpr uint32_t kSmallLanesLog2 = 2;
constexpr uint32_t kNoTriangle = 0xFFFFu;
// Windowed frames: a band may pick the triangles that touch its rows out of the frame's bins, in rounds of one per lane,
// which pays if walking the bins for one band costs this many turns of a wavefront (a triangle of the large bin is a
// turn, 16 small ones are one).  Humanoid and box, us per launch with 80 / 160 / 400: 256x256 140 / 137 / 137, 384x384 141 /
// 141 / 143, 512x512 126 / 126 / 149.
constexpr uint32_t kBandListsFrom = 160;
// ... or this many, if one round (one triangle per lane) looks at all of the frame's.  A mesh scene, lists from 160 / 60 / 30
// turns: 160x160 130 / 130 / 124, 192x192 127 / 127 / 119, 256x256 135 / 126 / 120, 320x320 163 / 147 / 148; everything else
// within 1 %.  From 30 / 26 / 20, with a body at the near plane, which puts capsule scenes beside the line: 368x368 506 / 439 / 441, 384x384 525 / 440 / 441,
// 400x400 666 / 577 / 580; in view all within 0.3 %.
constexpr uint32_t kBandListsFromOneRound = 26;
// Windowed frames take half a compute unit's LDS (two workgroups cover each other's barriers) if that leaves room for this
// share of the frame's keys, in thousandths, and all of it otherwise (fewer bands).  us per launch of 25 million pixels, half /
// all, and the share that half leaves:
//   humanoid and box  144x144 66/75 (177)   160x160 64/67 (141)   176x176 67/60 (115)   192x192 74/65 (95)    224x224 78/61 (68)
//   humanoid          144x144 57/71 (185)   160x160 59/65 (148)   176x176 61/57 (120)   192x192 64/61 (105)   224x224 67/55 (75)
//   64 bodies         176x176 104/106 (180) 192x192 100/104 (150) 224x224 107/105 (108) 256x256 121/105 (81)
//   quadrupeds        192x192 42/53 (155)   224x224 43/45 (112)   256x256 50/50 (84)    288x288 49/34 (66)
//   meshes            192x192 61/65 (207)   224x224 55/60 (150)   256x256 67/69 (114)   288x288 66/53 (89)
//   capsules          224x224 31/34 (170)   256x256 35/38 (129)   288x288 35/29 (101)   320x320 41/34 (80)
// and humanoids over a clip 192x192 139/163.  No share is right for every scene: the line costs the humanoids of 176x176 8 to
// 12 %, one at 130 would cost the humanoids over the clip 17 % and quadrupeds and capsules up to 8 %.  What a body at the near plane
// costs (the window is the frame then): humanoid and box 160x160 240/151, 176x176 268/165, but quadrupeds 224x224 400/431, capsules
// 160x160 305/484.
constexpr uint32_t kHalfKeysFrom = 103;
// ... and run 768 threads below this many pixels (two workgroups then have registers to spare), 1024 from there on (more
// lanes for the pixels).  us per launch, 768 / 1024: 84x84 over a clip 415 / 442, humanoid and box 84x84 217 / 222, 96x96 190 /
// 185, 128x128 144 / 142, 160x160 138 / 134, humanoids 192x192 126 / 122, quadrupeds 192x192 84 / 80.
constexpr uint32_t kWideWindowedFrom = 20000;

// Per-body record kept in LDS for the duration of one frame (floats).
//   [0..8]  M  = view rotation * body rotation, row-major
//   [9..11] t  = body origin in view space
//   [12..14] lb = light direction in the body frame
//   [15]    pad
//   [16..19] shape (a,b,c,h)
//   [20..22] rgb, [23] pad
constexpr uint32_t kBodyStride = 24;

// Everything the kernel needs that is constant for a scene.  Passed by value
// as the kernel argument (lands in SGPRs / scalar loads).
struct SceneConsts {
    // camera rows (right, up, forward), eye offset, focal length in pixels.  The kernel takes only the ground from these rows (the bodies'
    // transforms have a table of their own): where eye_first is 1 its copy has x and y exchanged in all three, like the eye that goes with them.
    float Rt[3], Up[3], Fw[3], off[3];
    uint32_t eye_first;
    float f, halfW, halfH, z_near, z_far;
    // light, ground, background
    float l[3], ambient, diffuse;
    float cell, gs[2], bg[3];
    uint32_t ground_on;
    uint32_t checker_short_form;  // cell == 1 and z_far <= 2^64: no division, and ground points of a frame whose eye is no NaN are no NaNs
    // sizes
    uint32_t W, H, npix, K, root, V, T, P;  // P = entries of the pair table (on the device: padded to a multiple of 64)
    uint32_t key_capacity;                  // windowed frames: pixel keys that the LDS buffer holds; 0 = it holds the whole frame
    uint32_t key_capacity_video;            // (the same beside the video distractor's tables)
    uint32_t pitch;                         // keys per row where the buffer holds the whole frame: W rounded up to a multiple of 4
    uint32_t magic_groups;                  // ceil(2^32 / (pitch / 4)): g / (pitch / 4) == mulhi(g, magic_groups) for every group of four pixels
    uint32_t magic24_groups;                // ceil(2^24 / (pitch / 4)): the same as (g << 8) * magic24_groups >> 32, for frames whose width is a multiple of 4
    // device tables
    const float* vtmpl;       // [V][4]  ux,uy,uz, bits = LDS address of the body's record in units of 16 bytes | s as a half float << 16
                              //         (the host-side table holds body<<2 | (s+1)); the device copy is padded to a multiple of 64 entries
    const uint32_t* tri_idx;  // [T][2]  v0 | v1<<16 ,  v2 | (LDS address of the body's record in units of 16 bytes)<<16 (the host-side table: body)
    const float* tri_shade;   // [T][4]  unit normal (body frame), colour multiplier
    const uint32_t* pair_tbl; // [P][4]  a0 | a1<<16 , a2 , a3 , triA | triB<<16 (a_i = LDS byte address of the cell
                              //         code of vertex q_i; the host-side table holds q0 | q1<<16 , q2 | q3<<16 , triA | triB<<16 , 0): two triangles sharing the
                              //         edge q0-q2, or one triangle (q3 = q2, triB = kNoTriangle); the device copy ends with padding entries
    //         (no triangles; the four addresses are that of the word after the last vertex's code, which holds code 0)
    const float* body_const;  // [K][8]  shape a,b,c,h ; rgb r,g,b,0   then, on the device, [4][3]: Rt, Up, Fw, l, and
                              // [K][4]  largest |u_x|, |u_y|, |u_z| and |u| of the body's template vertices
    const float* cxcy;        // [W+H]   pixel-centre ray slopes
    // LDS carve-up (byte offsets into the dynamic segment)
    // the lds_keys region first holds the per-vertex cell codes (u32[V]) and the candidate list (u16[T])
    uint32_t lds_keys, lds_vxy, lds_vd, lds_body, lds_list, lds_large, lds_cxcy, lds_rows, lds_misc, lds_total;
    uint32_t lds_vlut;  // video-blend tables (kVideoTableBytes), or 0 if the frame's LDS has no room for them
};

// Video distractor: for each of the five colours that can lie under the clip (background r, g, b; the two ground
// greys) the blended, quantised byte for every clip byte: [5][256] bytes, rebuilt per frame in LDS.
constexpr uint32_t kVideoTableBytes = 9 * 256;  // background r, g, b; first grey x 3; second grey x 3

// Distractor state bound by pxr_apply_distractor.
struct DistractConsts {
    uint32_t mode;
    uint32_t seed_lo, seed_hi;
    float scale_lo, scale_span, offset_lo, offset_span;
    const uint8_t* video;
    uint32_t n_frames;
    float alpha;
    const uint32_t* env_offset;
    uint32_t n_videos;          // >= 1
    const uint32_t* env_video;  // [B] or null
};

// Skeleton bound by pxr_set_skeleton (device tables live in their own allocation).
struct SkeletonRecord {
    uint32_t body;    // index of the body in a frame's poses
    int32_t parent;   // body it hangs from, -1 = free body
    int32_t slot;     // free: index of its pose; hinged: index of its angle, -1 = rigid
    float anchor[3];  // hinge position in the parent's frame
    float axis[3];    // unit hinge axis
    float offset[3];  // body centre relative to the hinge, body frame
};
struct SkeletonConsts {
    uint32_t K, J, F;                // bodies, hinge angles per frame, free poses per frame
    uint32_t depths;                 // number of depths; depth 0 = the free bodies
    const SkeletonRecord* records;   // [K], in order of depth
    const uint32_t* depth_begin;     // [depths + 1] first record of each depth
    const uint32_t* links;           // [K] each record's depth | its parent's record << 16 (0 for a free body)
};

// The render kernel's own kinematics stage: inputs and where the poses go.
struct FkArgs {
    SkeletonConsts sk;
    const float* free_poses;  // [frames, F, 7]
    const float* angles;      // [frames, J]
    float* poses;             // [frames, K, 7], written
};
static_assert(sizeof(SkeletonRecord) == 48, "a lane reads a record as three 16-byte words");

// Host-side result of tessellation + camera derivation.
struct HostScene {
    SceneConsts c{};
    std::vector<float> vtmpl;
    std::vector<uint32_t> tri_idx;
    std::vector<float> tri_shade;
    std::vector<uint32_t> pair_tbl;
    std::vector<float> body_const;
    std::vector<float> body_bound;
    std::vector<float> cxcy;
};

// scene.cpp: validates `desc`, fills `hs` (device pointers and LDS offsets are
// left for the caller).  Returns a PXR_* code and a message on failure.
int build_host_scene(const pxr_scene_desc& desc, HostScene& hs, std::string& err);

// Which render kernels are built to make poses as well: not those of few threads with windows, which only a caller's choice reaches.
constexpr bool makes_poses(uint32_t block_threads, bool windowed) { return !windowed || block_threads >= 768u; }

// render.hip: enqueue one batch.  `block_threads` in {256,512,768,1024}; `n_cus` compute units of the device.
// `fk`: the poses are not read but made in the same launch, from joint angles (null: read from d_poses).
int launch_render(const SceneConsts& sc, const DistractConsts& dc, const FkArgs* fk, const float* d_poses, const float* d_shapes,
                  uint32_t n_frames, uint32_t S, uint32_t step0, uint32_t env0, uint8_t* d_frames, uint32_t* d_ids,
                  uint32_t block_threads, uint32_t n_cus, void* stream, std::string& err);

// render.hip: raise the dynamic-LDS limit of every kernel instantiation on the current device (the caller sees
// to it that this runs once per device).
int prepare_kernels(std::string& err);

// Frame consumer (first convolutional layer of the policy), bound by pxr_conv_create.
// 3x3 kernel, stride 2, 32 output channels; the frame stack is the channel axis.
struct ConvConsts {
    uint32_t H, W, S;        // input frames [S,H,W,3] per environment
    uint32_t Ho, Wo;         // output size
    uint32_t wo_magic;       // ceil(2^20 / Wo): p / Wo == (p * wo_magic) >> 20 for every pixel p of a band (p * Wo < 2^20: a band's
                             // input has at most 4096 pixels, its output a quarter of that, and Wo is at most 127)
    uint32_t band_rows;      // output rows of a work item, at most
    uint32_t bands;          // work items per environment
    uint32_t extra_rows;     // this many bands have band_rows rows, the others one less; 0 = all have band_rows
    uint32_t rows_in;        // input rows held in LDS per frame = 2 * band_rows + 1
    uint32_t relu;
    const uint32_t* wtab;    // [3S][64 lanes][4] the A operands of the matrix instruction, bf16 pairs
    const float* bias;       // [32]
};

// api.cpp: record the calling thread's last error and return `code`.
int set_error(int code, const std::string& msg);

// conv.hip
uint32_t conv_lds_bytes(const ConvConsts& cc);
uint32_t conv_max_quads();  // 12-byte input quads (4 pixels) one work item may hold: S * rows_in * W / 4
int prepare_conv_kernels(std::string& err);
int launch_conv(const ConvConsts& cc, const uint8_t* d_frames, uint32_t B, uint16_t* d_out, uint32_t n_groups,
                void* stream, std::string& err);

// peaks.hip: sustained fp32-FMA and 24-bit integer multiply-add rates (T lane-operations/s) and the
// read+write bandwidth of a plain 1 GiB copy and of 2 GiB read-only / write-only streams (GB/s) on the current device.
int measure_peaks(double* fma_tlaneops, double* imad_tlaneops, double* copy_gbs, double* read_gbs, double* write_gbs,
                  std::string& err);

// selftest.hip: the render kernel's arithmetic shortcuts against the plain forms over every float
// (counts: reciprocal mismatches, floor-convert mismatches, patterns looked at by each check).
int selftest_arithmetic(unsigned long long counts[4], std::string& err);

// kinematics.hip: joint angles -> poses, 64 frames per workgroup.
uint32_t fk_lds_bytes(const SkeletonConsts& sk);
int prepare_fk_kernel(std::string& err);
int launch_fk(const SkeletonConsts& sk, const float* d_free_poses, const float* d_angles, uint32_t n_frames,
              float* d_poses, void* stream, std::string& err);

// pipeline.cpp works through these (api.cpp / conv_api.cpp own the handles' layouts).
constexpr uint32_t kMaxPipelineChunks = 16;
void scene_shape(const pxr_scene* s, uint32_t* K, uint32_t* H, uint32_t* W);
void conv_shape(const pxr_conv* c, uint32_t* H, uint32_t* W, uint32_t* S, uint32_t* Ho, uint32_t* Wo);
// Environments [e0, e0 + n) of a batch whose buffers start at the given pointers (arguments as pxr_render_batch /
// pxr_conv_forward, whose checks they repeat; per-environment distractor arrays are indexed by position in the batch).
int render_envs(pxr_scene* s, const float* d_poses, const float* d_shapes, uint32_t e0, uint32_t n, uint32_t S,
                uint32_t step0, uint32_t env0, uint8_t* d_frames, uint32_t* d_ids, void* stream, std::string& err);
int conv_envs(pxr_conv* c, const uint8_t* d_frames, uint32_t e0, uint32_t n, uint16_t* d_out, void* stream, std::string& err);

// static_scratch.hip: this device's copy of the library's file-scope pose buffer (looked up on the first call
// per device, cached afterwards) and its size.  Allocates nothing.
int static_pose_scratch(float** out, size_t* capacity_bytes, std::string& err);

}  // namespace pxr

#endif
