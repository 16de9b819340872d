// The hot path of libpxr: one HIP kernel, one workgroup per frame
// (= environment x step), the whole frame resident in LDS from the posed
// vertices to the packed uint8 store.  gfx950 only.
//
// What it renders is what PixelBrax (arXiv 2502.00021, sections 1-2) asks of
// its renderer: a small RGB observation per parallel environment per step,
// built on the device from the simulator's body poses, with the colour / video
// distractors applied inside the renderer and all randomness coming from a
// seeded counter-based generator.
//
// Phases of one workgroup (barriers between them):
//   0  per-body transforms, per-frame draws and the three non-triangle colours
//   1  instancing: template vertex -> view space -> snapped fixed point, plus
//      a per-vertex "cell code" saying between which pixel centres it lies
//   2a binning, coarse: one lane per PAIR of edge-sharing triangles; from the
//      cell codes alone (xor / or, no coordinates) decide per triangle whether
//      its bounding box can hold a pixel centre; candidates are compacted
//      wave-wide (ballot + mbcnt) into a list in LDS
//   2b binning, exact: one lane per candidate: exact area sign, pixel range,
//      then compaction into three bins by candidate-pixel count
//   3  raster: bins are walked by 1, 4 or 64 lanes per triangle (rows are
//      dealt round-robin to a triangle's lanes); integer edge functions,
//      top-left rule, float reversed depth, 64-bit LDS atomic max on
//      (depth bits << 32 | ~triangle id)
//   4  resolve: ground ray, id -> flat Lambert colour, distractor, uint8 pack,
//      coalesced 12-byte stores
//
// Floating point is written with explicit fmaf and compiled with
// -ffp-contract=off: the order of operations is part of the output contract
// (coverage is decided by integers derived from these floats).

#include <hip/hip_runtime.h>

#include <type_traits>

#include "arith.h"
#include "hinge.h"
#include "pxr_internal.h"
#include "reach.h"

namespace pxr {
namespace {

typedef unsigned long long u64;

__device__ __forceinline__ float dot3(float a0, float a1, float a2, float b0, float b1, float b2) {
    return __builtin_fmaf(a0, b0, __builtin_fmaf(a1, b1, a2 * b2));
}

__device__ __forceinline__ int imin3(int a, int b, int c) { return min(a, min(b, c)); }
__device__ __forceinline__ int imax3(int a, int b, int c) { return max(a, max(b, c)); }

// Workgroups are dealt round-robin to the 8 XCDs.  Renumber them so that each
// XCD works on one contiguous run of frames: neighbouring frames share pose
// cache lines and (video mode) neighbouring clip frames in that XCD's L2.
__device__ __forceinline__ uint32_t frame_of_block(uint32_t bid, uint32_t nb) {
    const uint32_t q = nb >> 3, r = nb & 7u, xcd = bid & 7u, idx = bid >> 3;
    return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// ---------------------------------------------------------------- generator
// 10 rounds of the 4x32 multiply / xor counter network, key = 64-bit seed,
// counter = (env, step, stream, 0).
__device__ __forceinline__ void counter_rng(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                            uint32_t out[4]) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}
__device__ __forceinline__ float unit_float(uint32_t x) { return (float)(x >> 8) * 5.9604644775390625e-08f; }

// ---------------------------------------------------------------- raster helpers

// Snapped coordinates are kept with their origin moved by 127, so that pixel centre i lies at 256 i + 255: a
// coordinate's upper bits are then the number of the cell between two centres that it lies in, and the first and the last
// centre of a range follow from them without an addition (31 trips of gathers per frame of 64x64, four additions each).
__device__ __forceinline__ int snap(float s) { return floor_to_int(__builtin_fmaf(s, 256.0f, 0.5f)) + 127; }
__device__ __forceinline__ int centre_of(int i) {
    int r;
    asm("v_lshl_or_b32 %0, %1, 8, %2" : "=v"(r) : "v"(i), "s"(255));  // (i << 8) + 255
    return r;
}
__device__ __forceinline__ int first_centre(int lowest) { return lowest >> 8; }
// One past the last centre that a triangle reaching up to `highest` can cover: one that lies on its right or lower end exactly is
// not covered, whatever its shape.  (Both edges at a right end would have to be top-left ones, which then turn the wrong way
// round; an edge that goes down, or along the bottom, is none.)
__device__ __forceinline__ int centres_end(int highest) { return highest >> 8; }

// Products and sums of the narrow triangles' setup, as the instructions they are.  (Written with operators the compiler takes them apart: sign
// extensions around the products, and a fourth induction variable in place of a three-way sum.)
__device__ __forceinline__ int mul24(int a, int b) {
    int r;
    asm("v_mul_i32_i24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ int mad24(int a, int b, int c) {
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ int add3(int a, int b, int c) {
    int r;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// A triangle's snapped corners in screen order: a = v0, b = v2, c = v1.
struct Corners {
    int ax, ay, bx, by, cx, cy;
    // Both fixed-point extents below 2^15 ("narrow"): every product of coordinate differences is below 2^30 then, and 24-bit
    // multiplies are exact.  (Coordinates reach 2^22, products 2^46.)
    __device__ __forceinline__ bool narrow() const {
        return ((imax3(ax, bx, cx) - imin3(ax, bx, cx)) | (imax3(ay, by, cy) - imin3(ay, by, cy))) < 32768;
    }
};

// Candidate pixels [i0, i_end) x [j0, j_end) of a triangle.
struct PixelBox {
    int i0, i_end, j0, j_end;
    __device__ __forceinline__ bool empty() const { return i0 >= i_end || j0 >= j_end; }
};

// The pixels the key buffer stands for: columns [x_lo, x_end) and rows [y_lo, y_end) of the frame, `pitch` keys per row.
struct RasterWindow {
    int x_lo, x_end, y_lo, y_end;
    uint32_t pitch;
};

__device__ __forceinline__ PixelBox candidate_pixels(const RasterWindow& win, const Corners& t) {
    return {max(win.x_lo, first_centre(imin3(t.ax, t.bx, t.cx))), min(win.x_end, centres_end(imax3(t.ax, t.bx, t.cx))),
            max(win.y_lo, first_centre(imin3(t.ay, t.by, t.cy))), min(win.y_end, centres_end(imax3(t.ay, t.by, t.cy)))};
}

// Depth of the plane through a triangle's corners: at corner a, and the differences of b and c to it.
struct DepthPlane {
    float Da, dDb, dDc;
};

// Edge pq is "top-left" when it points up, or is horizontal pointing right
// (y grows downwards): pixels exactly on it belong to the triangle.
__device__ __forceinline__ int edge_bias(int dx, int dy) { return (dy < 0 || (dy == 0 && dx > 0)) ? 0 : -1; }

// The pixel loops below walk rows j0 + r, j0 + r + 2^shift, ... of a triangle's candidate pixels, and in each of them the columns
// i0 + c, i0 + c + 2^cshift, ... (a team of 2^shift x 2^cshift lanes shares the triangle; c = cshift = 0: whole rows).
//
// Narrow triangles.  What most of the raster phase's instructions are for is not the pixels but getting started, once per team and
// lane (of the triangles that reach this phase two thirds have one candidate pixel).  So: edges ab and ca are taken relative to corner a, with signs
// that make each edge function a multiply and a multiply-add; edge bc is what is left of twice the area; "top-left" is the sign of one
// number per edge, 2^16 dy - dx, and of the sum of the other two's for bc.  (With three edge functions of their own and comparisons for the
// fill rule, 95 instructions instead of 55, 65 536 x 3 frames of 64x64 3401 us, now 3192, 16 384 of 84x84 over a clip 408 / 388, 4096 quadrupeds 64.4 /
// 60.7, meshes of 110x75 31.0 / 29.5, 256 chains from angles 10.3 / 10.1.  Kept with their fill rule's k taken off, an edge is inside by its sign, and the k
// is added again where a pixel is covered: for triangles of many pixels two instructions a pixel less; 8503 capsule frames of 84x84 137.8 us with three
// comparisons per pixel, 131.)
__device__ __forceinline__ void raster_rows_narrow(const Corners& t, const PixelBox& box, const DepthPlane& d, uint32_t tri,
                                                   const RasterWindow& win, u64* keys, int r, int shift, int c = 0, int cshift = 0) {
    const int i = box.i0 + c;
    int j = box.j0 + r;
    if (j >= box.j_end) return;
    if (cshift != 0 && i >= box.i_end) return;
    const int P = t.ax - t.bx, Q = t.by - t.ay, S = t.cx - t.ax, R = t.ay - t.cy;  // ab = (-P, Q), ca = (-S, R)
    const int A2 = mul24(P, R) - mul24(Q, S);                                 // > 0: binned triangles face the camera
    const float invA = recip_in_range((float)A2);
    // e = - the edge function; a point of ab or ca is inside at e < k, with k = 1 on a top-left edge, else 0.  Kept is e - k.
    const int u = centre_of(i) - t.ax, v = centre_of(j) - t.ay;
    const int w_ab = (int)((uint32_t)Q << 16) + P, w_ca = (int)((uint32_t)R << 16) + S;
    const int k_ab = (int)((uint32_t)w_ab >> 31), k_ca = (int)((uint32_t)w_ca >> 31);
    int e_ab_row = mad24(P, v, mul24(Q, u)) - k_ab, e_ca_row = mad24(S, v, mul24(R, u)) - k_ca;
    // the third edge function is A2 + e_ab + e_ca, and inside at > -1 on a top-left edge, > 0 else
    const int rest = A2 + k_ab + k_ca - (w_ab + w_ca > 0 ? 0 : 1);
    const int x_ab = (int)((uint32_t)Q << (8 + cshift)), x_ca = (int)((uint32_t)R << (8 + cshift));
    const int y_ab = (int)((uint32_t)P << (8 + shift)), y_ca = (int)((uint32_t)S << (8 + shift));
    u64* row = keys + (__umul24((uint32_t)(j - win.y_lo), win.pitch) + (uint32_t)(i - win.x_lo));
    const int n = box.i_end - i;
    for (;;) {
        int e_ab = e_ab_row, e_ca = e_ca_row;
        u64* p = row;
        u64* const end = row + n;
        do {
            if ((e_ab & e_ca & ~add3(e_ab, e_ca, rest)) < 0) {
                // (the additions of zero make a weight of zero a positive one)
                const float beta = __builtin_fmaf((float)(e_ca + k_ca), -invA, 0.0f), gamma = __builtin_fmaf((float)(e_ab + k_ab), -invA, 0.0f);
                const float depth = __builtin_fmaf(beta, d.dDb, __builtin_fmaf(gamma, d.dDc, d.Da));
                atomicMax(p, ((u64)__float_as_uint(depth) << 32) | (u64)(0xFFFFFFFFu - tri));
            }
            e_ab += x_ab;
            e_ca += x_ca;
            p += 1 << cshift;
        } while (p < end);
        j += 1 << shift;
        if (j >= box.j_end) break;
        e_ab_row += y_ab;
        e_ca_row += y_ca;
        row += win.pitch << shift;
    }
}

// Any triangle, in 64-bit arithmetic.  Edge functions carry their fill-rule bias and are stepped incrementally; a
// pixel centre is covered when all three are >= 0.
__device__ __forceinline__ void raster_rows_wide(const Corners& t, const PixelBox& box, const DepthPlane& d, uint32_t tri,
                                                 const RasterWindow& win, u64* keys, int r, int shift, int c, int cshift) {
    typedef long long I;
    int j = box.j0 + r;
    if (j >= box.j_end) return;
    const int dx_ab = t.bx - t.ax, dy_ab = t.by - t.ay;
    const int dx_bc = t.cx - t.bx, dy_bc = t.cy - t.by;
    const int dx_ca = t.ax - t.cx, dy_ca = t.ay - t.cy;
    const I A2 = (I)dx_ab * (I)(t.cy - t.ay) - (I)dy_ab * (I)(t.cx - t.ax);
    const float invA = recip_in_range((float)A2);  // a front face: 1 <= A2 < 2^47
    const I b_ab = edge_bias(dx_ab, dy_ab), b_bc = edge_bias(dx_bc, dy_bc), b_ca = edge_bias(dx_ca, dy_ca);
    const int px0 = centre_of(box.i0 + c), py = centre_of(j);
    I f_ab = (I)dx_ab * (I)(py - t.ay) - (I)dy_ab * (I)(px0 - t.ax) + b_ab;
    I f_bc = (I)dx_bc * (I)(py - t.by) - (I)dy_bc * (I)(px0 - t.bx) + b_bc;
    I f_ca = (I)dx_ca * (I)(py - t.cy) - (I)dy_ca * (I)(px0 - t.cx) + b_ca;
    const I sx_ab = (I)dy_ab << (8 + cshift), sx_bc = (I)dy_bc << (8 + cshift), sx_ca = (I)dy_ca << (8 + cshift);
    const I sy_ab = (I)dx_ab << (8 + shift), sy_bc = (I)dx_bc << (8 + shift), sy_ca = (I)dx_ca << (8 + shift);
    for (;;) {
        I e_ab = f_ab, e_bc = f_bc, e_ca = f_ca;
        uint32_t pix = (uint32_t)(j - win.y_lo) * win.pitch + (uint32_t)(box.i0 + c - win.x_lo);
        for (int i = box.i0 + c; i < box.i_end; i += 1 << cshift, pix += 1u << cshift) {
            if ((e_ab | e_bc | e_ca) >= 0) {
                const float beta = (float)(e_ca - b_ca) * invA, gamma = (float)(e_ab - b_ab) * invA;
                const float depth = __builtin_fmaf(beta, d.dDb, __builtin_fmaf(gamma, d.dDc, d.Da));
                atomicMax(&keys[pix], ((u64)__float_as_uint(depth) << 32) | (u64)(0xFFFFFFFFu - tri));
            }
            e_ab -= sx_ab;
            e_bc -= sx_bc;
            e_ca -= sx_ca;
        }
        j += 1 << shift;
        if (j >= box.j_end) break;  // (stepping past the last row could leave the exactly representable range)
        f_ab += sy_ab;
        f_bc += sy_bc;
        f_ca += sy_ca;
    }
}

// How a whole wavefront shares a triangle of n rows: 2^shift lanes down the rows (as many as there are rows, up to
// 64), the other 2^(6 - shift) across each row, so that a wide triangle of a few rows (every large triangle of a
// frame that is rendered in bands of a few rows) keeps all lanes busy.
__device__ __forceinline__ void wave_team(int n_rows, int lane, int& r, int& shift, int& c, int& cshift) {
    shift = n_rows >= 33 ? 6 : (32 - __builtin_clz((uint32_t)max(n_rows, 1) * 2u - 1u)) - 1;  // ceil(log2(n_rows))
    cshift = 6 - shift;
    r = lane & ((1 << shift) - 1);
    c = lane >> shift;
}

// base + scale * one of a word's halves, in one instruction.
template <int SCALE>
__device__ __forceinline__ uint32_t at_low_half(uint32_t word, uint32_t base) {
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(word), "n"(SCALE), "s"(base));
    return r;
}
template <int SCALE>
__device__ __forceinline__ uint32_t at_high_half(uint32_t word, uint32_t base) {
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(word), "n"(SCALE), "s"(base));
    return r;
}

// A word of LDS by its byte address.  (The dynamic LDS segment starts at address 0: the kernels here have
// no static LDS, which prepare_kernels verifies; tables built on the host can therefore hold LDS addresses.)
template <typename T>
__device__ __forceinline__ T lds_at(uint32_t byte_address) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T*>(static_cast<uintptr_t>(byte_address));
}

// A triangle's corners (ti = its entry of the device's index table: v0 | v1 << 16, v2 | where its body's record is << 16).
__device__ __forceinline__ Corners gather_corners(const uint2 ti, uint32_t lds_vxy) {
    // (x, y) pairs: one 8-byte LDS read per vertex (as one integer each: read as pairs, the compiler would fetch
    // the y's separately, after the test of the x's, in a second round trip)
    const u64 a = lds_at<u64>(at_low_half<8>(ti.x, lds_vxy)), b = lds_at<u64>(at_low_half<8>(ti.y, lds_vxy)),
              c = lds_at<u64>(at_high_half<8>(ti.x, lds_vxy));
    return {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)(uint32_t)b, (int)(uint32_t)(b >> 32), (int)(uint32_t)c, (int)(uint32_t)(c >> 32)};
}

__device__ __forceinline__ DepthPlane gather_depths(const uint2 ti, uint32_t lds_vd) {
    const float Da = lds_at<float>(at_low_half<4>(ti.x, lds_vd));
    return {Da, lds_at<float>(at_low_half<4>(ti.y, lds_vd)) - Da, lds_at<float>(at_high_half<4>(ti.x, lds_vd)) - Da};
}

// kTriNone if a corner is unusable or all of them lie behind the near plane; kTriClip if the triangle straddles it (the snapped
// corners say nothing then); kTriPlain otherwise.
enum { kTriNone = 0, kTriPlain = 1, kTriClip = 2 };
__device__ __forceinline__ int tri_kind(const Corners& t) {
    const int minx = imin3(t.ax, t.bx, t.cx);
    if (minx > kBehindX) return kTriPlain;  // (a sentinel among the three is rare)
    return minx == kRejectedX || imax3(t.ax, t.bx, t.cx) == kBehindX ? kTriNone : kTriClip;
}

// Which image rows a binned triangle can touch: kTriPlain with [j0, j_end) (not clamped), or kTriClip for a
// triangle that straddles the near plane (its snapped corners say nothing: it counts for every row).
__device__ __forceinline__ int tri_rows(const uint2 ti, uint32_t lds_vxy, int& j0, int& j_end) {
    const Corners t = gather_corners(ti, lds_vxy);
    if (imin3(t.ax, t.bx, t.cx) <= kBehindX) return kTriClip;
    j0 = first_centre(imin3(t.ay, t.by, t.cy));
    j_end = centres_end(imax3(t.ay, t.by, t.cy));
    return kTriPlain;
}

// View-space position of template vertex v (the instancing arithmetic of phase 1; also used when a
// triangle has to be clipped).  The template's fourth word says where in LDS its body's record is, in units of 16 bytes, and holds the cap
// selector s (-1, 0 or +1) as a half float above that.
__device__ __forceinline__ void view_position(const float4 tv, float& pvx, float& pvy, float& pvz) {
    uint32_t record;
    asm("v_mad_u32_u16 %0, %1, 16, 0" : "=v"(record) : "v"(__float_as_uint(tv.w)));
    // (body records are 96 bytes at a 16-byte aligned base: four 16-byte LDS reads)
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const __attribute__((address_space(3))) f32x4* o4 = reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(static_cast<uintptr_t>(record));
    const f32x4 m0 = o4[0], m1 = o4[1], m2 = o4[2], sh = o4[4];  // M and t as floats 0..11, the shape as 16..19
    float cap;  // s * h
    asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(cap) : "v"(__float_as_uint(tv.w)), "v"(sh.w));
    const float lx = sh.x * tv.x;
    const float ly = sh.y * tv.y;
    const float lz = __builtin_fmaf(sh.z, tv.z, cap);
    pvx = __builtin_fmaf(m0.x, lx, __builtin_fmaf(m0.y, ly, __builtin_fmaf(m0.z, lz, m2.y)));
    pvy = __builtin_fmaf(m0.w, lx, __builtin_fmaf(m1.x, ly, __builtin_fmaf(m1.y, lz, m2.z)));
    pvz = __builtin_fmaf(m1.z, lx, __builtin_fmaf(m1.w, ly, __builtin_fmaf(m2.x, lz, m2.w)));
}

// A triangle or a clipped triangle's piece, by a whole wavefront.
__device__ __forceinline__ void raster_by_wave(const Corners& t, const DepthPlane& d, uint32_t tri, const RasterWindow& win, u64* keys, int lane) {
    const PixelBox box = candidate_pixels(win, t);
    if (box.empty()) return;
    int r, shift, c, cshift;
    wave_team(box.j_end - box.j0, lane, r, shift, c, cshift);
    if (t.narrow())
        raster_rows_narrow(t, box, d, tri, win, keys, r, shift, c, cshift);
    else
        raster_rows_wide(t, box, d, tri, win, keys, r, shift, c, cshift);
}

// A triangle with corners on both sides of the near plane (every lane of the wavefront computes the
// same clip).  Walk the edges v0->v1, v1->v2, v2->v0: a corner in front is kept, an edge that crosses
// the plane adds its intersection, computed from the corner in front (P) towards the one behind (Q) so
// that both triangles sharing the edge get the same point:
//   t = (z_near - P.z) / (Q.z - P.z),  I = (fma(t, Q.x - P.x, P.x), fma(t, Q.y - P.y, P.y), z_near).
// The 3 or 4 corners w0.. keep the winding; new ones are projected and snapped like template vertices
// (outside the guard band = unusable) and the pieces (w0,w1,w2), (w0,w2,w3) are rastered under id t.
//
// Which corner the walk emits k-th depends only on which of the three vertices are in front: a 4-bit
// code per corner (P << 2 | Q, P == Q for a kept vertex), four corners per pattern, patterns indexed by
// the in-front mask (bit e = vertex e in front).  Corners are recomputed per piece rather than kept, so
// that this rarely taken path does not raise the kernel's register count.
__device__ __forceinline__ void raster_clipped(const SceneConsts& sc, const RasterWindow& win, uint32_t t, const int2* vxy,
                                               const float* vd, u64* keys, int lane) {
#pragma unroll 1
    for (uint32_t piece = 0; piece < 2u; ++piece) {
        // everything is re-derived per piece so that nothing but `t` stays live across the raster loops
        const uint2 ti = reinterpret_cast<const uint2*>(sc.tri_idx)[t];
        const uint32_t v0 = ti.x & 0xFFFFu, v1 = ti.x >> 16, v2 = ti.y & 0xFFFFu;
        const uint32_t mask = (vxy[v0].x != kBehindX ? 1u : 0u) | (vxy[v1].x != kBehindX ? 2u : 0u) | (vxy[v2].x != kBehindX ? 4u : 0u);
        // corners k = 0..3 in bits 4k..4k+3; V_e = e<<2|e, I_pq = p<<2|q
        //   001: V0 I01 I02      010: I10 V1 I12      100: I21 V2 I20
        //   011: V0 V1 I12 I02   110: I10 V1 V2 I20   101: V0 I01 I21 V2
        const uint32_t pattern = mask == 1u ? 0x0210u : mask == 2u ? 0x0654u : mask == 4u ? 0x08A9u
                               : mask == 3u ? 0x2650u : mask == 6u ? 0x8A54u : 0xA910u;
        if (piece == 1u && (mask == 1u || mask == 2u || mask == 4u)) break;  // one corner in front: one piece
        const float inv = 1.0f / sc.z_near;
        // screen order (a, b, c) = (w0, w2, w1), then (w0, w3, w2)
        const uint32_t order = piece == 0 ? 0x120u : 0x230u;
        int cX[3], cY[3];
        float cD[3];
        bool usable = true;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint32_t code = (pattern >> (4u * ((order >> (4 * c)) & 15u))) & 15u;
            const uint32_t p = code >> 2, q = code & 3u;
            const uint32_t vp = p == 0 ? v0 : (p == 1 ? v1 : v2), vq = q == 0 ? v0 : (q == 1 ? v1 : v2);
            if (p == q) {
                cX[c] = vxy[vp].x;
                cY[c] = vxy[vp].y;
                cD[c] = vd[vp];
            } else {
                float px, py, pz, qx, qy, qz;
                view_position(reinterpret_cast<const float4*>(sc.vtmpl)[vp], px, py, pz);
                __builtin_amdgcn_sched_barrier(0);  // one vertex at a time: keeps this path within the register budget
                view_position(reinterpret_cast<const float4*>(sc.vtmpl)[vq], qx, qy, qz);
                __builtin_amdgcn_sched_barrier(0);
                const float tt = (sc.z_near - pz) / (qz - pz);
                const float ix = __builtin_fmaf(tt, qx - px, px);
                const float iy = __builtin_fmaf(tt, qy - py, py);
                const float sx = __builtin_fmaf(sc.f, ix * inv, sc.halfW);
                const float sy = __builtin_fmaf(-sc.f, iy * inv, sc.halfH);
                const bool ok = (__builtin_fabsf(sx) <= 16384.0f) && (__builtin_fabsf(sy) <= 16384.0f);
                usable = usable && ok;
                cX[c] = ok ? snap(sx) : 0;
                cY[c] = ok ? snap(sy) : 0;
                cD[c] = sc.z_near * inv;
            }
        }
        const Corners piece_corners = {cX[0], cY[0], cX[1], cY[1], cX[2], cY[2]};
        const bool front = (long long)(cX[1] - cX[0]) * (long long)(cY[2] - cY[0]) > (long long)(cY[1] - cY[0]) * (long long)(cX[2] - cX[0]);
        if (usable && front) raster_by_wave(piece_corners, {cD[0], cD[1] - cD[0], cD[2] - cD[0]}, t, win, keys, lane);
    }
}

// A triangle of the tiny or small bin (narrow, not clipped), with lane `r` of the 2^shift lanes that share it, restricted to the window that
// the key buffer currently holds.  WINDOWED: which may hold none of its pixels.
template <bool WINDOWED>
__device__ __forceinline__ void raster_binned(const RasterWindow& win, uint32_t t, const uint2 ti, uint32_t lds_vxy, uint32_t lds_vd, u64* keys,
                                              int r, int shift) {
    const Corners corners = gather_corners(ti, lds_vxy);
    const DepthPlane depths = gather_depths(ti, lds_vd);
    const PixelBox box = candidate_pixels(win, corners);
    if (WINDOWED && box.empty()) return;
    raster_rows_narrow(corners, box, depths, t, win, keys, r, shift);
}

// A triangle of the large bin, by a whole wavefront: one of many candidate pixels, or one to be clipped.
__device__ __forceinline__ void raster_large(const SceneConsts& sc, const RasterWindow& win, uint32_t t, const uint2 ti, const int2* vxy,
                                             const float* vd, u64* keys, int lane) {
    const Corners corners = gather_corners(ti, sc.lds_vxy);
    if (tri_kind(corners) == kTriClip)
        raster_clipped(sc, win, t, vxy, vd, keys, lane);
    else
        raster_by_wave(corners, gather_depths(ti, sc.lds_vd), t, win, keys, lane);
}

// A wide triangle that shows few pixels, with lane `r` of the 2^shift lanes that share it.
__device__ __forceinline__ void raster_few(const SceneConsts& sc, const RasterWindow& win, uint32_t t, const uint2 ti, u64* keys, int r, int shift) {
    const Corners corners = gather_corners(ti, sc.lds_vxy);
    const PixelBox box = candidate_pixels(win, corners);
    if (box.empty()) return;
    raster_rows_wide(corners, box, gather_depths(ti, sc.lds_vd), t, win, keys, r, shift, 0, 0);
}

// Per-axis cell code of a snapped coordinate for an image of n pixels: c = after pixel centre c - 1 and up to centre c,
// clamped to [0, n] (0 = up to centre 0, n = beyond centre n - 1).  No triangle whose corners have the same code on an
// axis covers a pixel centre (centres_end).  (With a code of its own for "exactly on a centre", as if it were covered from
// both sides, the code took six instructions more per vertex and axis pair and the test of a pair of triangles four: 65 536 x 3
// frames of 64x64 3478 us, now 3401, 16 384 of 84x84 over a clip 412.7 / 408.0, 4096 quadrupeds 65.1 / 64.4.)
__device__ __forceinline__ uint32_t cell_code(int x, int n) {
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x >> 8), "s"(n));  // clamp(x >> 8, 0, n) in one instruction (n > 0)
    return (uint32_t)r;
}

// The bits in which three words are not all the same, in one instruction.
__device__ __forceinline__ uint32_t any_differ(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x7E); }

// Low half times high half of a word (non-zero iff both are), in one instruction.
__device__ __forceinline__ uint32_t halves_product(uint32_t x) {
    uint32_t r;
    asm("v_mul_u32_u24_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_0" : "=v"(r) : "v"(x));
    return r;
}

__device__ __forceinline__ uint32_t lanes_below(u64 m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t quantise(float c) {
    return (uint32_t)floor_to_int(__builtin_fmaf(c, 255.0f, 0.5f)) & 0xFFu;
}

// ---------------------------------------------------------------- the kernel

// The render kernel's arguments as they lie in the kernel-argument segment: in order, each at its type's alignment.
struct RenderArguments {
    SceneConsts sc;
    DistractConsts dc;
    const float* poses;
    const float* shapes;
    uint32_t S, step0, env0;
    uint8_t* frames;
    uint32_t* ids;
    uint32_t slabs_log2;
    FkArgs fk;  // (of the kernels that make their poses)
};

// An argument where it lies in that segment.  The compiler takes a by-value argument apart as soon as it can, loads
// its members at the kernel's head and keeps each in scalar registers until its last use.  Read through this, a member is
// loaded where it is used.  What that decides is how many scalar registers a kernel takes, and with them how many of its wavefronts
// are resident: a SIMD has 800 and hands them out in steps of 16, and each wavefront has 16 more than its kernel names (for the trap
// handler), so eight wavefronts have 80 each.  With more, four workgroups of 512 threads do not fit a compute unit (with 82 three do).
// us by value (92 to 106 scalar registers) / in place (65 to 80): 12 000 capsule frames of 64x64 109.9 / 92.5, 16 384 of chains of 48x48
// 155.4 / 134.5, over a clip 180.6 / 153.5, 47 wide 198.7 / 167; 2048 from joint angles 30.7 / 25.7.  The kernels of 1024 threads are
// held to 80 and parked what they had no room for in lanes of vector registers: 8192 humanoid frames of 63x63 over a clip 221.9 (48
// parked) / 162 (none), 64x64 163.2 (18) / 153.7.
template <typename T>
__device__ __forceinline__ const T& argument_in_place(uint32_t byte_offset) {
    typedef const __attribute__((address_space(4))) unsigned char* KernargBytes;
    return *(const T*)(const __attribute__((address_space(4))) T*)((KernargBytes)__builtin_amdgcn_kernarg_segment_ptr() + byte_offset);
}

// The same, read afresh: whatever the compiler loaded from it before is not reused after this point.  The band loop of tall frames takes
// its constants through this at the top of every trip, so that they are fetched again (scalar loads that hit the
// constant cache) instead of being kept in scalar registers across the whole loop, which the 1024-thread
// variants do not have.
template <typename T>
__device__ __forceinline__ const T& argument_reloaded(uint32_t byte_offset) {
    typedef const __attribute__((address_space(4))) unsigned char* KernargBytes;
    KernargBytes p = (KernargBytes)__builtin_amdgcn_kernarg_segment_ptr() + byte_offset;
    asm volatile("" : "+s"(p));
    return *(const T*)(const __attribute__((address_space(4))) T*)p;
}
#define PXR_ARGUMENT(READ, MEMBER) argument_##READ<decltype(RenderArguments::MEMBER)>((uint32_t)offsetof(RenderArguments, MEMBER))

// Ask for every cache line of the kernel's arguments at once, of which it has BYTES.  They lie in memory that a launch's first wavefronts
// find in no cache; as the compiler places the loads, each next group of arguments would wait for a miss of its own.
// A word of each line that they fill, and the first word behind them (the implicit arguments, of which the grid's size is the first), which
// lies in the line of the last ones.  (A word more than one of a line is not free: 12 000 capsule frames of 64x64 92.5 us, 94.0 with two more.)
template <size_t BYTES>
__device__ __forceinline__ void request_arguments() {
    typedef const __attribute__((address_space(4))) uint32_t* KernargWords;
    static_assert(BYTES % 8u == 0u, "the implicit arguments follow at a multiple of 8 bytes");
    const KernargWords p = (KernargWords)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t any = 0;
#pragma unroll
    for (uint32_t at = 0; at + 64u <= BYTES; at += 64u) any |= p[at / 4u];
    any |= *(KernargWords)__builtin_amdgcn_implicitarg_ptr();
    asm volatile("" : : "s"(any));
}

// Phase probes: empty in the library.  A profiling build (-DPXR_PROFILING_BUILD, made into a file of its own
// by build.py --define) takes them from a header that the library's build never includes.
#ifdef PXR_PROFILING_BUILD
#include "profiling/phase_probes.h"
#else
#define PXR_PHASE_BEGIN()
#define PXR_PHASE_MARK(i)
#define PXR_TIMED_BARRIER(i) __syncthreads()
#define PXR_PHASE_END()
#endif

struct FrameUniforms {  // written in phase 0 (one lane) or by LDS atomics, read by all after a barrier
    u64 bins;           // 16-bit counters: tiny | small << 16 | large << 32, for whole frames | wide ones with few pixels << 48
    uint32_t n_cand;
    uint32_t n_few;     // windowed frames: wide ones with few pixels (a fourth part of the counters' word parks six scalars more there)
    uint32_t video_frame;
    float scale[3], offs[3];
    float base_col[3][3];     // background, ground grey 0, ground grey 1 after the colour distractor
    uint32_t base_packed[3];  // the same three, quantised: R | G<<8 | B<<16
    float eye[3];             // camera position (in the kernels that make their poses)
    float ground_eye[3];      // the same for phase 4, its first two in the order of the ground's axes (written by the first lane in phase 0)
    uint32_t ticket;          // windowed frames: next chunk of the pixels outside the window
    u64 band_bins[2];         // windowed frames: the three counters of one band round's lists, double-buffered by round
    uint32_t reach[4];        // windowed frames: columns [0], [1) and rows [2], [3) that the bodies can touch
    // ... and the window made of them, in groups of four columns (written by one lane in phase 1):
    uint32_t win_x0;          // first column (a multiple of 4)
    uint32_t win_groups;      // groups per row of the window (2 or more)
    uint32_t win_y0, win_rows;
    uint32_t band_rows;       // rows of it that the key buffer holds at a time
    uint32_t win_magic;       // ceil(2^32 / win_groups)
    uint32_t side_magic;      // ceil(2^32 / groups of a row beside the window), 0 = none
};
static_assert(sizeof(FrameUniforms) <= 64 * 4, "the frame's uniforms have 256 bytes of LDS");

// Everything phase 4 needs that is uniform over the frame.
struct ResolveCtx {
    float eye_x, eye_y, eye_z, inv_ez;
    bool ground_ok;
    float alpha;
    float scale[3], offs[3];
    uint32_t col_addr;     // LDS byte address of the three colours as floats [3][3]
    uint32_t packed[3];    // and as packed bytes: background, first grey, second grey
    uint32_t vlut;         // LDS byte address of the video-blend tables, 0 = none
    const uint8_t* vframe;
    const float* tri_shade;  // (what the shading of triangles needs of the scene)
    float ambient, diffuse;
};

// Ground plane z = 0 along the pixel's ray: returns its z-test key (0 = miss)
// and the ray parameter (= view depth) of the hit.
__device__ __forceinline__ u64 ground_key(const SceneConsts& sc, const ResolveCtx& rc, float ndz, float& tg) {
    tg = 0.0f;
    if (rc.ground_ok && ndz > 0.0f) {
        tg = rc.eye_z / ndz;
        if (tg >= sc.z_near && tg <= sc.z_far) {
            const float dg = (sc.z_near * ndz) * rc.inv_ez;
            return ((u64)__float_as_uint(dg) << 32) | 1ull;
        }
    }
    return 0ull;
}

// Triangle g as a 24-bit colour: flat Lambert + ambient in the body frame, then the colour distractor.
template <bool VIDEO>
__device__ __forceinline__ uint32_t shade_triangle(const SceneConsts& sc, const ResolveCtx& rc, uint32_t g) {
    // (byte offsets of 32 bits from scalar addresses: as indices they would be 64-bit address arithmetic for each)
    const float4 ns = *reinterpret_cast<const float4*>(reinterpret_cast<const unsigned char*>(rc.tri_shade) + g * 16u);
    const uint32_t record = (uint32_t)*reinterpret_cast<const uint16_t*>(reinterpret_cast<const unsigned char*>(sc.tri_idx) + (g * 8u + 6u)) * 16u;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 lb = lds_at<f32x4>(record + 48u), col = lds_at<f32x4>(record + 80u);  // floats 12..14: light in the body frame, 20..22: colour
    const float o_rgb[3] = {col.x, col.y, col.z};
    float I = __builtin_fmaf(ns.x, lb.x, __builtin_fmaf(ns.y, lb.y, ns.z * lb.z));
    I = I > 0.0f ? I : 0.0f;
    const float sh = __builtin_fmaf(rc.diffuse, I, rc.ambient);
    uint32_t rgb = 0;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        float v = (o_rgb[ch] * ns.w) * sh;
        v = v < 1.0f ? v : 1.0f;
        if (!VIDEO) {  // (without the colour distractor the factor is 1 and the offset 0, which leaves a value in [0, 1] as it is)
            v = __builtin_fmaf(v, rc.scale[ch], rc.offs[ch]);
            v = v > 0.0f ? v : 0.0f;
            v = v < 1.0f ? v : 1.0f;
        }
        rgb |= quantise(v) << (8 * ch);
    }
    return rgb;
}

// Sum of the two checker cell indices where the pixel's ray (parameter tg, direction dwx, dwy) meets the ground:
// its lowest bit says which of the two greys shows.
// UNIT_CELL: the checkerboard cell is 1 m, so the division by the cell size is the identity, and the ground point
// cannot be a NaN (a finite or infinite eye, a far plane within 2^64), so the one-instruction floor-and-convert serves.
template <bool UNIT_CELL>
__device__ __forceinline__ uint32_t checker_cells(const SceneConsts& sc, const ResolveCtx& rc, float tg, float dwx, float dwy) {
    const float wx = __builtin_fmaf(tg, dwx, rc.eye_x);
    const float wy = __builtin_fmaf(tg, dwy, rc.eye_y);
    if (UNIT_CELL)  // (wx and wy are no NaNs here: the caller has looked at the eye and at z_far)
        return (uint32_t)floor_to_int(wx) + (uint32_t)floor_to_int(wy);
    return (uint32_t)(int)__builtin_floorf(wx / sc.cell) + (uint32_t)(int)__builtin_floorf(wy / sc.cell);
}

// One pixel: winner of (triangles, ground, background) -> colour -> distractor
// -> 24-bit RGB.  `low` returns ~id.  `vbytes` = the pixel's three video bytes
// (R | G<<8 | B<<16), only read in video mode.
// (A triangle pixel returns 0: the caller shades it, compacted over the wavefront.)
template <bool UNIT_CELL, bool VIDEO>
__device__ __forceinline__ uint32_t resolve_pixel(const SceneConsts& sc, const ResolveCtx& rc, u64 key, u64 gkey, float tg,
                                                  float dwx, float dwy, uint32_t vbytes, uint32_t& low, u64& tri_lanes) {
    key = key > gkey ? key : gkey;
    low = (uint32_t)key;
    tri_lanes = __ballot(low > 1u);  // (taken here, beside the branch on the same comparison, it costs nothing)
    if (low > 1u) return 0u;
    // background or ground: one of three colours per frame (consecutive in LDS: background, grey 0, grey 1)
    if (!VIDEO) {
        uint32_t rgb = rc.packed[0];
        if (low == 1u) rgb = (checker_cells<UNIT_CELL>(sc, rc, tg, dwx, dwy) & 1u) != 0u ? rc.packed[2] : rc.packed[1];
        return rgb;
    }
    uint32_t col = rc.col_addr;
    if (low == 1u) {
        uint32_t grey = checker_cells<UNIT_CELL>(sc, rc, tg, dwx, dwy) & 1u;
        asm("" : "+v"(grey));  // (kept from the compiler, which would turn the multiply-add into compare, select, add)
        col = __umul24(grey, 12u) + (rc.col_addr + 12u);
    }
    const __attribute__((address_space(3))) float* c3 =
        reinterpret_cast<const __attribute__((address_space(3))) float*>(static_cast<uintptr_t>(col));
    uint32_t rgb = 0;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float c = c3[ch];
        const float vf = (float)((vbytes >> (8 * ch)) & 0xFFu) * (1.0f / 255.0f);
        rgb |= quantise(__builtin_fmaf(rc.alpha, vf - c, c)) << (8 * ch);
    }
    return rgb;
}

// The groups of four pixels that a call of resolve_groups takes.
//   kWholeFrame     every group of the frame; the key buffer holds the frame
//   kInsideWindow   the groups of the window's current band; the key buffer holds exactly these, in this order
//   kBesideWindow   the groups that no triangle can touch (sky, ground, clip: no key is looked at), handed out in
//                   chunks of 64 to whichever wavefront comes next
enum ResolvePart { kWholeFrame = 0, kInsideWindow = 1, kBesideWindow = 2 };
struct ResolveRange {
    uint32_t x0, groups, magic;         // window: first column, groups per row, ceil(2^32 / groups)
    uint32_t y0, rows;                  // its rows (inside: of the band)
    uint32_t first_row, end_row;        // beside: rows of the frame this workgroup renders
    uint32_t side_groups, side_magic;   // beside: groups of a row left and right of the window, ceil(2^32 / that) or 0
    uint32_t* ticket;
};

// Phase 4: four consecutive pixels of one row (a group) per lane.  The row part of the ray is shared, and without camera
// roll (NO_ROLL: the right vector is horizontal) so is the whole ground test, which then costs one division per image
// row, not one per pixel.
// RAGGED: the width is no multiple of 4.  A row's last group is then partial, and a group's twelve bytes start at any
// byte: they leave as one unaligned 12-byte store, the last group's pixels as two shorter ones.  (One pixel per lane with byte
// stores and a ground test with its division per pixel, which such widths took before: 11 840 quadruped frames of 71x71
// with the colour distractor 254 us, now 196.)
// ALONG_AXIS: the camera's right vector has no x component either (it looks along the x axis, seen from above; or along the y axis, which the host
// hands over as x), so a row's ground points share their x, and with it one of the checker's two cell indices.  (With a unit cell and without roll; per
// four pixels ten instructions less: 65 536 x 3 frames of 64x64 3128 us without, 3110 with, 4096 quadrupeds 61.0 / 60.5, 16 384 of 84x84 over a clip 376.3 / 374.1, 8503 capsule frames of
// 84x84 129.6 / 128.5, quadrupeds of 128x128 96.4 / 95.5; along y 4096 quadrupeds of 64x64 63.8 / 63.4, of 84x84 84.9 / 83.9, 2048 x 3 humanoids and
// boxes of 84x84 151.6 / 150.1.)
template <int NT, bool UNIT_CELL, bool NO_ROLL, bool VIDEO, bool RAGGED, ResolvePart PART, bool ALONG_AXIS = false>
__device__ __forceinline__ void resolve_groups(const SceneConsts& sc, const ResolveCtx& rc, const float* cxcy,
                                               const float4* rows, u64* keys, uint8_t* out, uint32_t* out_ids,
                                               uint32_t tid, const ResolveRange& range) {
    constexpr bool HAS_KEYS = PART != kBesideWindow;
    const uint32_t lane = tid & 63u;
    const uint32_t row_groups = (sc.W + 3u) >> 2;
    // how many groups there are, and (beside the window) how many of them lie above it and left or right of it
    uint32_t n_groups, n_above = 0, n_side = 0;
    if (PART == kWholeFrame) {
        n_groups = row_groups * sc.H;
    } else if (PART == kInsideWindow) {
        n_groups = range.groups * range.rows;
    } else {
        n_above = (range.y0 - range.first_row) * row_groups;
        n_side = range.rows * range.side_groups;
        n_groups = (range.end_row - range.first_row - range.rows) * row_groups + n_side;
    }
    uint32_t g = tid;
    // (The next chunk's ticket is drawn while the present one is resolved, but not under roll, where a division per pixel covers the wait and the
    // register costs more.  us without / with: 1024 frames of 256x256 144.4 / 143.2, quadrupeds of 128x128 96.4 / 95.7; meshes of 110x75 under roll 29.2 /
    // 29.5.)
    constexpr bool kTicketAhead = PART == kBesideWindow && NO_ROLL;
    uint32_t chunk = 0;
    const auto draw_ticket = [&]() {
        if (lane == 0) chunk = atomicAdd(range.ticket, 1u);
    };
    if (kTicketAhead) draw_ticket();
    for (;;) {
        if (PART == kBesideWindow) {
            if (!kTicketAhead) draw_ticket();
            g = ((uint32_t)__builtin_amdgcn_readfirstlane((int)chunk) << 6) + lane;
            if (g - lane >= n_groups) return;
            if (kTicketAhead) draw_ticket();
            g = min(g, n_groups - 1u);  // (the last chunk's spare lanes repeat its last group: the same bytes)
        } else if (g >= n_groups) {
            return;
        }
        // ---- where the group lies: row j, first column i0, first pixel p0
        uint32_t j, i0, p0;
        if (PART == kWholeFrame && !RAGGED) {
            // (24-bit products only: a frame has at most 2^16 groups, a row at most 2^7, and 2^8 g times ceil(2^24 / groups) >> 32 is exact for them)
            asm("v_mul_hi_u32_u24 %0, %1, %2" : "=v"(j) : "v"(g << 8), "s"(sc.magic24_groups));
            i0 = (g - __umul24(j, row_groups)) * 4u;
            p0 = g * 4u;
        } else if (PART == kInsideWindow) {
            const uint32_t r = __umulhi(g, range.magic);
            j = range.y0 + r;
            i0 = range.x0 + (g - r * range.groups) * 4u;
            p0 = j * sc.W + i0;
        } else {
            uint32_t c;
            const uint32_t m = g - n_above;
            if (PART == kBesideWindow && m < n_side) {  // (above the window m wraps round and is not below)
                uint32_t r = range.side_magic ? __umulhi(m, range.side_magic) : 0u;
                c = m - r * range.side_groups;
                c += c * 4u >= range.x0 ? range.groups : 0u;
                j = range.y0 + r;
            } else {
                uint32_t q = g;
                if (PART == kBesideWindow) {
                    q += range.first_row * row_groups;
                    if (g >= n_above) q += range.rows * range.groups;  // below: the window's groups lie in between
                }
                j = __umulhi(q, sc.magic_groups);
                c = q - j * row_groups;
            }
            i0 = c * 4u;
            p0 = j * sc.W + i0;
        }
        const bool whole = !RAGGED || i0 + 4u <= sc.W;  // all four pixels exist
        const uint32_t byte0 = PART == kWholeFrame && !RAGGED ? __umul24(g, 12u) : __umul24(p0, 3u);
        // what is shared by a row's pixels was worked out once per row in phase 0
        const float4 row = rows[j];
        const float rx = row.x, ry = row.y;
        const float rz = NO_ROLL ? 0.0f : row.z;
        const float4 cx4 = *reinterpret_cast<const float4*>(cxcy + i0);
        const float cxs[4] = {cx4.x, cx4.y, cx4.z, cx4.w};
        uint32_t vid[3] = {0u, 0u, 0u};
        if (VIDEO) {
            if (!RAGGED) {
                __builtin_memcpy(vid, __builtin_assume_aligned(rc.vframe + byte0, 4), 12);
            } else {
                const uint8_t* vsrc = rc.vframe + byte0;
                if (whole) {
                    __builtin_memcpy(vid, vsrc, 12);
                } else {
                    // (the twelve bytes that end with the row - it has eight pixels or more -, moved down to their place)
                    uint32_t end[3];
                    __builtin_memcpy(end, vsrc - (4u - (sc.W & 3u)) * 3u, 12);
                    if ((sc.W & 3u) == 3u) {
                        vid[0] = __builtin_amdgcn_alignbit(end[1], end[0], 24u);
                        vid[1] = __builtin_amdgcn_alignbit(end[2], end[1], 24u);
                        vid[2] = end[2] >> 24;
                    } else if ((sc.W & 3u) == 2u) {
                        vid[0] = __builtin_amdgcn_alignbit(end[2], end[1], 16u);
                        vid[1] = end[2] >> 16;
                    } else {
                        vid[0] = end[2] >> 8;
                    }
                }
            }
        }
        const uint32_t vb[4] = {vid[0] & 0xFFFFFFu, (vid[0] >> 24) | ((vid[1] & 0xFFFFu) << 8),
                                (vid[1] >> 16) | ((vid[2] & 0xFFu) << 16), vid[2] >> 8};
        // without roll the ground test is the row's: ray parameter (0 = miss) and depth bits from the row table
        const float tg_row = NO_ROLL ? row.z : 0.0f;
        // (a miss has depth bits 0 in the table: the key is 0 then)
        const u64 gkey_row = NO_ROLL ? (((u64)__float_as_uint(row.w) << 32) | (tg_row != 0.0f ? 1ull : 0ull)) : 0ull;
        // the lane's four keys are 32 contiguous, aligned bytes: two 16-byte LDS reads
        u64 key4[4] = {0ull, 0ull, 0ull, 0ull};
        u64* own_keys = keys + g * 4u;
        if (HAS_KEYS) {
            const uint4 k01 = reinterpret_cast<const uint4*>(own_keys)[0], k23 = reinterpret_cast<const uint4*>(own_keys)[1];
            key4[0] = ((u64)k01.y << 32) | k01.x;
            key4[1] = ((u64)k01.w << 32) | k01.z;
            key4[2] = ((u64)k23.y << 32) | k23.x;
            key4[3] = ((u64)k23.w << 32) | k23.z;
        }
        uint32_t rgb[4] = {0u, 0u, 0u, 0u}, low[4];
        uint32_t ow[3] = {0u, 0u, 0u};  // the 12 bytes that leave
        bool direct = false;            // they were put together as they were looked up (rgb[] is not used)
        u64 tri_lanes[4] = {0ull, 0ull, 0ull, 0ull};
        // (the right vector's x being a zero, the ray's is the row's; a zero's sign makes no difference to the sum)
        const uint32_t row_cell = ALONG_AXIS ? (uint32_t)floor_to_int(__builtin_fmaf(tg_row, rx, rc.eye_x)) : 0u;
        const auto cells = [&](float tg, float cx) -> uint32_t {
            const float dwy = __builtin_fmaf(sc.Rt[1], cx, ry);
            if (ALONG_AXIS) return row_cell + (uint32_t)floor_to_int(__builtin_fmaf(tg, dwy, rc.eye_y));
            return checker_cells<UNIT_CELL>(sc, rc, tg, __builtin_fmaf(sc.Rt[0], cx, rx), dwy);
        };
        if (!VIDEO) {
            // One of the frame's three colours (background, two greys), without a branch per pixel.  A triangle pixel
            // picks up one of them as well, to be overwritten below.  Without roll a row is ground or sky as a whole,
            // so the choice between "background" and "a grey by the checker" is the lane's, not the pixel's: a lane
            // above the horizon has the background in place of both greys, and a pixel is a bitwise choice by the
            // checker's parity.  (As a read of the colour's word in LDS, a round trip for every group of pixels: 1024 frames of
            // 256x256 158.5 us, now 157.5, 999 mesh frames of 110x75 31.3, now 31.0, capsules of 84x84 136.3, now 133.1.)
            const bool ground_row = tg_row != 0.0f;
            const uint32_t even = NO_ROLL && !ground_row ? rc.packed[0] : rc.packed[1], odd = NO_ROLL && !ground_row ? rc.packed[0] : rc.packed[2];
            const bool ground_in_sight = !NO_ROLL || __ballot(ground_row) != 0ull;  // (a wavefront above the horizon)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float tg = tg_row;
                u64 gkey = gkey_row;
                if (!NO_ROLL) gkey = ground_key(sc, rc, -__builtin_fmaf(sc.Rt[2], cxs[k], rz), tg);
                const u64 key = HAS_KEYS && key4[k] > gkey ? key4[k] : gkey;
                low[k] = (uint32_t)key;
                if (HAS_KEYS) tri_lanes[k] = __ballot(low[k] > 1u);
                rgb[k] = even;
                if (ground_in_sight) {
                    uint32_t is_odd = (uint32_t)__builtin_amdgcn_sbfe((int)cells(tg, cxs[k]), 0, 1);  // all ones or none
                    asm("" : "+v"(is_odd));  // (kept from the compiler, which would turn the two instructions into and, compare, select)
                    rgb[k] = (is_odd & odd) | (~is_odd & even);
                    if (!NO_ROLL && low[k] != 1u) rgb[k] = rc.packed[0];
                }
            }
        } else if (NO_ROLL && rc.vlut) {
            // Video distractor, no roll, tables in LDS: a row is sky or ground as a whole, so under the clip lies
            // the background or one of the two greys by the checker's parity, and the blended byte of a channel
            // is one byte read from the table of that colour, indexed by the clip's byte where it lies in the three
            // words that brought it (byte n = channel n % 3 of pixel n / 3), and put at the same place of the three
            // words that leave.  A triangle pixel gets a blended colour as well, replaced below.
            direct = true;
            const bool ground_row = tg_row != 0.0f;
            const uint32_t lane_base = rc.vlut + (ground_row ? 768u : 0u);  // background's tables, or the first grey's
            const uint32_t odd_step = ground_row ? 768u : 0u;               // the second grey's follow the first's
            uint32_t base[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u64 key = HAS_KEYS && key4[k] > gkey_row ? key4[k] : gkey_row;
                low[k] = (uint32_t)key;
                if (HAS_KEYS) tri_lanes[k] = __ballot(low[k] > 1u);
                uint32_t odd = cells(tg_row, cxs[k]) & 1u;
                asm("" : "+v"(odd));  // (kept from the compiler, which would turn the multiply-add into compare, select, add)
                base[k] = __umul24(odd, odd_step) + lane_base;
            }
#pragma unroll
            for (int w = 0; w < 3; ++w) {
                uint32_t word = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int n = 4 * w + b;
                    const uint32_t at = base[n / 3] + ((vid[w] >> (8 * b)) & 0xFFu) + 256u * (n % 3);
                    word |= (uint32_t)*reinterpret_cast<const __attribute__((address_space(3))) uint8_t*>(static_cast<uintptr_t>(at)) << (8 * b);
                }
                ow[w] = word;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float tg = tg_row;
                u64 gkey = gkey_row;
                if (!NO_ROLL) gkey = ground_key(sc, rc, -__builtin_fmaf(sc.Rt[2], cxs[k], rz), tg);
                const float dwx = __builtin_fmaf(sc.Rt[0], cxs[k], rx);
                const float dwy = __builtin_fmaf(sc.Rt[1], cxs[k], ry);
                rgb[k] = resolve_pixel<UNIT_CELL, VIDEO>(sc, rc, key4[k], gkey, tg, dwx, dwy, vb[k], low[k], tri_lanes[k]);
            }
        }
        // Triangle pixels are few and clustered: instead of every lane walking the shading code four
        // times, the wavefront compacts its triangle pixels into a list (in the LDS of its own, already
        // consumed, pixel keys), shades the list densely, and the owners pick their colours up.
        const u64 m0 = tri_lanes[0], m1 = tri_lanes[1], m2 = tri_lanes[2], m3 = tri_lanes[3];
        if (HAS_KEYS && (m0 | m1 | m2 | m3)) {
            uint32_t* list = reinterpret_cast<uint32_t*>(keys + (g - lane) * 4u);  // 256 keys = 512 words
            const uint32_t n0 = (uint32_t)__popcll(m0), n1 = n0 + (uint32_t)__popcll(m1), n2 = n1 + (uint32_t)__popcll(m2);
            const uint32_t total = n2 + (uint32_t)__popcll(m3);
            const uint32_t slot[4] = {lanes_below(m0), n0 + lanes_below(m1), n1 + lanes_below(m2), n2 + lanes_below(m3)};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (low[k] > 1u) list[slot[k]] = low[k];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const u64 active = __ballot(true);  // the last trip of a ragged band may run with fewer lanes
            for (uint32_t i = lanes_below(active); i < total; i += (uint32_t)__popcll(active))
                list[i] = shade_triangle<VIDEO>(sc, rc, 0xFFFFFFFFu - list[i]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (low[k] > 1u) rgb[k] = list[slot[k]];
            if (VIDEO && direct) {
                // (pixel k's three bytes start at byte 3 k of the twelve)
                if (low[0] > 1u) ow[0] = (ow[0] & 0xFF000000u) | rgb[0];
                if (low[1] > 1u) {
                    ow[0] = (ow[0] & 0x00FFFFFFu) | (rgb[1] << 24);
                    ow[1] = (ow[1] & 0xFFFF0000u) | (rgb[1] >> 8);
                }
                if (low[2] > 1u) {
                    ow[1] = (ow[1] & 0x0000FFFFu) | (rgb[2] << 16);
                    ow[2] = (ow[2] & 0xFFFFFF00u) | (rgb[2] >> 16);
                }
                if (low[3] > 1u) ow[2] = (ow[2] & 0x000000FFu) | (rgb[3] << 8);
            }
        }
        if (PART == kInsideWindow) {
            // the lane leaves its four keys cleared for the next band (nobody else touches them)
            reinterpret_cast<uint4*>(own_keys)[0] = make_uint4(0u, 0u, 0u, 0u);
            reinterpret_cast<uint4*>(own_keys)[1] = make_uint4(0u, 0u, 0u, 0u);
        }
        if (!(VIDEO && direct)) {
            ow[0] = rgb[0] | (rgb[1] << 24);
            ow[1] = (rgb[1] >> 8) | (rgb[2] << 16);
            ow[2] = (rgb[2] >> 16) | (rgb[3] << 8);
        }
        if (!RAGGED) {
            struct alignas(4) U3 {
                uint32_t a, b, c;
            };
            *reinterpret_cast<U3*>(out + byte0) = U3{ow[0], ow[1], ow[2]};
            if (out_ids)
                *reinterpret_cast<uint4*>(reinterpret_cast<unsigned char*>(out_ids) + p0 * 4u) =
                    make_uint4(0xFFFFFFFFu - low[0], 0xFFFFFFFFu - low[1], 0xFFFFFFFFu - low[2], 0xFFFFFFFFu - low[3]);
        } else {
            uint8_t* dst = out + byte0;
            const uint32_t id4[4] = {0xFFFFFFFFu - low[0], 0xFFFFFFFFu - low[1], 0xFFFFFFFFu - low[2], 0xFFFFFFFFu - low[3]};
            if (whole) {
                __builtin_memcpy(dst, ow, 12);
                if (out_ids) __builtin_memcpy(out_ids + p0, id4, 16);
            } else {  // 1, 2 or 3 pixels, the same number for every row's last group
                const uint16_t high = (uint16_t)(ow[0] >> 16), low1 = (uint16_t)ow[1];
                if ((sc.W & 3u) == 1u) {
                    __builtin_memcpy(dst, ow, 2);
                    dst[2] = (uint8_t)high;
                } else if ((sc.W & 3u) == 2u) {
                    __builtin_memcpy(dst, ow, 4);
                    __builtin_memcpy(dst + 4, &low1, 2);
                } else {
                    __builtin_memcpy(dst, ow, 8);
                    dst[8] = (uint8_t)ow[2];
                }
                if (out_ids) {
                    out_ids[p0] = id4[0];
                    if ((sc.W & 3u) > 1u) out_ids[p0 + 1u] = id4[1];
                    if ((sc.W & 3u) > 2u) out_ids[p0 + 2u] = id4[2];
                }
            }
        }
        if (PART != kBesideWindow) g += NT;
    }
}

// The value of another lane of the same four (quad permutation: lane i of the four gets lane (SEL >> 2 i) & 3's).
template <int SEL>
__device__ __forceinline__ float from_quad(float x) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), SEL, 0xF, 0xF, true));
}

// Which pixels of the frame the bodies can touch (reach.h; one wavefront; four lanes per body, lanes 0 to 2 of the four take
// an axis each).  A body that is out of view along one axis of the image touches nothing along the other either: counted
// all the same, one beside the frame stretches the window up to the frame's edge (the box out of view to the right / left /
// above, 1472 humanoid-and-box frames of 128x128 75 / 77 / 84 us, now 63.5; 320 of 256x256 85 / 84 / 96 us, now 69.5).
__device__ __forceinline__ void add_reach(const SceneConsts& sc, const float* body, uint32_t* reach, uint32_t lane) {
    const uint32_t axis = lane & 3u;
    for (uint32_t k0 = 0; k0 < sc.K; k0 += 16u) {
        const uint32_t k = k0 + (lane >> 2);
        const uint32_t i = min(axis, 2u);
        const float* record = body + min(k, sc.K - 1u) * kBodyStride;
        const float4 bound = reinterpret_cast<const float4*>(sc.body_const + sc.K * 8u + 12u)[min(k, sc.K - 1u)];
        const float t = record[9u + i];
        const float e = half_extent(record[3u * i], record[3u * i + 1u], record[3u * i + 2u], t, record[16], record[17], record[18],
                                    record[19], bound.x, bound.y, bound.z, bound.w, [](float x) { return __builtin_amdgcn_sqrtf(x); });
        const float lo = t - e, hi = t + e;
        const float z_lo = from_quad<0xAA>(lo), z_hi = from_quad<0xAA>(hi);
        // lane 0: columns, lane 1: rows (the y axis points up)
        const AxisReach a = axis_reach(axis == 0u ? lo : -hi, axis == 0u ? hi : -lo, z_lo, z_hi, __builtin_amdgcn_rcpf(z_lo),
                                       __builtin_amdgcn_rcpf(z_hi), sc.f, axis == 0u ? sc.halfW : sc.halfH, axis == 0u ? sc.W : sc.H,
                                       sc.z_near);
        const bool other_none = from_quad<0xB1>(a.none() ? 1.0f : 0.0f) != 0.0f;  // (lanes 0 and 1 of the four change places)
        if (k < sc.K && axis < 2u && !a.none() && !other_none) {
            atomicMin(&reach[2u * axis], a.begin);
            atomicMax(&reach[2u * axis + 1u], a.end);
        }
    }
}

// The frame's window from the bodies' reach, and how many of its rows the key buffer holds at a time (one wavefront; the
// reach's begin may lie past its end: nothing to be seen).
__device__ __forceinline__ void make_window(const SceneConsts& sc, uint32_t key_capacity, FrameUniforms* fu, uint32_t first_row,
                                            uint32_t end_row, uint32_t lane) {
    const uint32_t row_groups = (sc.W + 3u) >> 2;
    const uint32_t x0 = fu->reach[0], x1 = fu->reach[1];
    uint32_t g0 = x0 >> 2, g1 = min((x1 + 3u) >> 2, row_groups);
    uint32_t y0 = max(fu->reach[2], first_row), y1 = min(fu->reach[3], end_row);
    if (x0 >= x1 || y0 >= y1) {
        g0 = 0u;
        g1 = 2u;
        y0 = y1 = first_row;
    }
    if (g1 - g0 < 2u) {  // (two groups or more, so that the magic number below exists; frames have two or more)
        g0 = min(g0, row_groups - 2u);
        g1 = g0 + 2u;
    }
    if (g1 - g0 + 1u == row_groups) {  // (likewise beside the window: none or two and more)
        g0 = 0u;
        g1 = row_groups;
    }
    const uint32_t groups = g1 - g0, side = row_groups - groups, rows = y1 - y0;
    // one division, three lanes: ceil(2^32 / groups), ceil(2^32 / side), rows that the buffer holds (at least one)
    const uint32_t of = lane == 2u ? key_capacity : 0xFFFFFFFFu, by = lane == 0u ? groups : (lane == 1u ? max(side, 1u) : groups * 4u);
    const uint32_t quotient = of / by;
    const uint32_t held = (uint32_t)__builtin_amdgcn_readlane((int)quotient, 2);
    uint32_t band_rows = rows;
    if (rows > held) {  // even bands
        const uint32_t bands = (rows + held - 1u) / held;
        band_rows = (rows + bands - 1u) / bands;
    }
    if (lane == 0u) {
        fu->win_x0 = g0 * 4u;
        fu->win_groups = groups;
        fu->win_y0 = y0;
        fu->win_rows = rows;
        fu->band_rows = band_rows;
        fu->win_magic = quotient + 1u;
    }
    if (lane == 1u) fu->side_magic = side ? quotient + 1u : 0u;
}

// The frame's poses from its joint angles, by one wavefront, a lane per body: left in LDS (seven floats behind each body's
// view rows, where phase 0 reads them before it writes its own results there), in memory if `store`, and the camera position
// in the frame's uniforms.  Same arithmetic as the kinematics kernel's (hinge.h).
// A chain of dependent steps: everything that memory has to deliver is requested at once (the frame's angles and free poses as
// they lie, one word per lane, dealt out by lane exchange when the bodies' records have come in), then a step per depth of
// the tree.
__device__ __forceinline__ void pose_frame(const FkArgs& fk, uint32_t frame, float* body, FrameUniforms* fu, uint32_t root,
                                           float off_x, float off_y, float off_z, uint32_t lane, bool store) {
    const SkeletonConsts& sk = fk.sk;
    const uint4* from = reinterpret_cast<const uint4*>(sk.records + min(lane, sk.K - 1u));
    const uint4 r0 = from[0], r1 = from[1], r2 = from[2];
    const uint32_t link = sk.links[min(lane, sk.K - 1u)];
    const float* angles = fk.angles + (size_t)frame * sk.J;
    const float* free_poses = fk.free_poses + (size_t)frame * (sk.F * 7u);
    const bool by_exchange = sk.J <= 64u && sk.F * 7u <= 64u;
    // (without a branch around them: behind one, the compiler would request them only when the records have come in)
    const float* none = reinterpret_cast<const float*>(sk.records);
    const float my_angle = (sk.J ? angles : none)[min(lane, max(sk.J, 1u) - 1u)];
    const float my_free = (sk.F ? free_poses : none)[min(lane, max(sk.F * 7u, 1u) - 1u)];
    SkeletonRecord t;
    const uint4 words[3] = {r0, r1, r2};
    __builtin_memcpy(&t, words, sizeof(t));
    float theta = 0.0f, p[7];
    if (by_exchange) {
        const int slot = max(t.slot, 0);
        theta = __shfl(my_angle, slot);
        if (t.slot < 0) theta = 0.0f;
#pragma unroll
        for (int c = 0; c < 7; ++c) p[c] = __shfl(my_free, (t.parent < 0 ? slot * 7 : 0) + c);
    } else {
        if (t.parent >= 0 && t.slot >= 0) theta = angles[t.slot];
#pragma unroll
        for (int c = 0; c < 7; ++c) p[c] = t.parent < 0 ? free_poses[t.slot * 7 + c] : 0.0f;
    }
    float sn, cs;
    sincos_half(theta, sn, cs);
    for (uint32_t d = 1; d < sk.depths; ++d) {
        float pp[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) pp[c] = __shfl(p[c], (int)(link >> 16));
        if ((link & 0xFFFFu) == d) hinge_pose(t, pp, cs, sn, p);
    }
    if (lane < sk.K) {
        float* o = body + t.body * kBodyStride + 12u;
#pragma unroll
        for (int c = 0; c < 7; ++c) o[c] = p[c];
        if (t.body == root) {
            fu->eye[0] = p[0] + off_x;
            fu->eye[1] = p[1] + off_y;
            fu->eye[2] = p[2] + off_z;
        }
        if (store) {
            float* dst = fk.poses + ((size_t)frame * sk.K + t.body) * 7u;
#pragma unroll
            for (int c = 0; c < 7; ++c) dst[c] = p[c];
        }
    }
}

// What of the scene phase 1's vertices need.
struct Projection {
    float f, z_near;
    float half_w, half_h;  // in vector registers: a fused multiply-add takes one scalar operand, and the focal length is that
    uint32_t W, H;
    bool recip_long_form;
};

// One template vertex: instancing, projection, snap, cell code.
__device__ __forceinline__ void instance_vertex(const Projection& pr, uint32_t v, const float4 tv, int2* vxy, float* vd, uint32_t* vm) {
    float pvx, pvy, pvz;
    view_position(tv, pvx, pvy, pvz);
    // 1 / pvz is only used when pvz >= z_near (otherwise the vertex is behind the plane or unusable
    // whatever it is), so the short form serves unless some lane's depth is beyond its range
    float inv;
    if (__builtin_expect(pr.recip_long_form || __ballot(pvz > kRecipMax) != 0ull, 0))
        inv = 1.0f / pvz;
    else
        inv = recip_in_range(pvz);
    const float sx = __builtin_fmaf(pr.f, pvx * inv, pr.half_w);
    const float sy = __builtin_fmaf(-pr.f, pvy * inv, pr.half_h);
    const bool ok = (pvz >= pr.z_near) && (__builtin_fabsf(sx) <= 16384.0f) && (__builtin_fabsf(sy) <= 16384.0f);
    // (worked out for every lane, whatever sx and sy are, and replaced where the vertex is not usable: such
    // vertices are rare, and a wavefront without one skips the replacement altogether)
    int X = snap(sx), Y = snap(sy);
    uint32_t m = cell_code(X, (int)pr.W) | (cell_code(Y, (int)pr.H) << 16);
    if (__builtin_expect(__ballot(!ok) != 0ull, 0)) {
        if (!ok) {
            X = pvz < pr.z_near ? kBehindX : kRejectedX;
            Y = 0;
            // The code of no usable vertex, so that a triangle with one or two such corners is never dropped by its codes.  One with three is (they
            // are the same): it has an unusable corner or lies behind the near plane as a whole, and is kTriNone either way.
            m = 0xFFFFFFFFu;
        }
    }
    vxy[v] = make_int2(X, Y);
    vd[v] = pr.z_near * inv;
    vm[v] = m;
}

// The part of phase 0 that needs no pose: the frame's draws and what is made of them, counters set to zero, the video
// distractor's tables (by the second or fourth wavefront on).
template <int NT, bool WINDOWED, bool VIDEO>
__device__ __forceinline__ void draw_frame(const SceneConsts& sc, const DistractConsts& dc, FrameUniforms* fu, unsigned char* lds,
                                           uint32_t e, uint32_t env, uint32_t step, uint32_t tid) {
    // (The wavefronts of a workgroup start a few hundred clocks apart, four at a time; the last ones start more than
    // a thousand clocks after the first.  The draws are this phase's longest chain beside the bodies': they belong on
    // an early wavefront that has nothing else to do - the third - and the late ones get no work here at all.)
    constexpr uint32_t kDrawLane = NT >= 1024 ? 191u : NT - 1u;  // last lane of the third wavefront (of the last: smaller groups)
    if (!VIDEO && tid <= kDrawLane && tid >= kDrawLane - 1u && dc.mode == PXR_DISTRACT_COLOR) {
        // The colour draws are two generator streams, the longest serial chain of this phase: the two
        // lanes walk one stream each, side by side; the offsets go through LDS to the last lane.
        const uint32_t stream = kDrawLane - tid;
        uint32_t r[4];
        counter_rng(dc.seed_lo, dc.seed_hi, env, step, stream, 0u, r);
        const float span = stream == 0u ? dc.scale_span : dc.offset_span, lo = stream == 0u ? dc.scale_lo : dc.offset_lo;
        float* dst = stream == 0u ? fu->scale : fu->offs;
#pragma unroll
        for (int c = 0; c < 3; ++c) dst[c] = __builtin_fmaf(unit_float(r[c]), span, lo);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (tid == kDrawLane) {
        fu->bins = 0ull;
        fu->n_cand = 0;
        if (WINDOWED) {
            fu->n_few = 0;
            fu->band_bins[0] = fu->band_bins[1] = 0ull;
            fu->ticket = 0u;
            fu->reach[0] = fu->reach[2] = 0xFFFFFFFFu;
            fu->reach[1] = fu->reach[3] = 0u;
        }
        if (VIDEO) {
            uint32_t first;
            if (dc.env_offset) {
                first = dc.env_offset[e];
            } else {
                uint32_t r[4];
                counter_rng(dc.seed_lo, dc.seed_hi, env, 0xFFFFFFFFu, 2u, 0u, r);
                first = r[0] % dc.n_frames;
            }
            uint32_t clip = 0;  // each environment plays one clip of the set
            if (dc.n_videos > 1) {
                if (dc.env_video) {
                    clip = dc.env_video[e] % dc.n_videos;
                } else {
                    uint32_t r[4];
                    counter_rng(dc.seed_lo, dc.seed_hi, env, 0xFFFFFFFFu, 3u, 0u, r);
                    clip = r[0] % dc.n_videos;
                }
            }
            fu->video_frame = clip * dc.n_frames + (uint32_t)(((u64)first + (u64)step) % dc.n_frames);
        }
    }
    // (from the fourth wavefront of the largest workgroups on: the second has the rows of the image, the third the draws.  8192 frames of chains of
    // 56x84 over a clip from the second on 151.2 us, now 146.9; 768 threads, 84x84, the other way round 415 and 418.)
    constexpr uint32_t kTablesFrom = NT >= 1024 ? 192u : 64u;
    if (VIDEO && sc.lds_vlut && tid >= kTablesFrom) {
        // Video-blend tables: under the clip lies the background or a ground grey (no colour distractor in this
        // mode), so a blended channel is a function of (one of five colours, clip byte).  Four entries per lane.
        // Nine tables of 256 bytes: background r, g, b, then each grey's three times over - the channel of a byte is
        // then the same address offset (256 x channel) whatever lies under the clip, a constant in the read.
        uint32_t* vlut = reinterpret_cast<uint32_t*>(lds + sc.lds_vlut);
        for (uint32_t i = tid - kTablesFrom; i < 5u * 64u; i += NT - kTablesFrom) {
            const uint32_t t = i >> 6, at = i & 63u;
            const float c = t == 0 ? sc.bg[0] : t == 1 ? sc.bg[1] : t == 2 ? sc.bg[2] : t == 3 ? sc.gs[0] : sc.gs[1];
            uint32_t word = 0;
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const float vf = (float)(at * 4u + e) * (1.0f / 255.0f);
                word |= quantise(__builtin_fmaf(dc.alpha, vf - c, c)) << (8 * e);
            }
            if (t < 3u) {
                vlut[i] = word;
            } else {
                uint32_t* g = vlut + (t == 3u ? 3u * 64u : 6u * 64u) + at;
                g[0] = g[64] = g[128] = word;
            }
        }
    }
    if (tid <= kDrawLane && tid >= kDrawLane - 2u) {
        // Background and the two ground greys are the same for every pixel that shows them: they go through
        // the colour distractor and the quantiser once per frame, one lane per colour.
        const uint32_t k = kDrawLane - tid;
        float scale[3] = {1.0f, 1.0f, 1.0f}, offs[3] = {0.0f, 0.0f, 0.0f};
        if (!VIDEO && dc.mode == PXR_DISTRACT_COLOR) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                scale[c] = fu->scale[c];
                offs[c] = fu->offs[c];
            }
        }
        uint32_t packed = 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // (the three are loaded first: as "k == 0 ? sc.bg[c] : ..." the compiler chooses an address for each lane and loads through
            // the vector unit, three round trips in a row: 12 000 capsule frames of 64x64 95.7 us, now 92.5)
            const float sky = sc.bg[c], grey0 = sc.gs[0], grey1 = sc.gs[1];
            float v = k == 0u ? sky : (k == 1u ? grey0 : grey1);
            if (!VIDEO && dc.mode == PXR_DISTRACT_COLOR) {
                v = __builtin_fmaf(v, scale[c], offs[c]);
                v = v > 0.0f ? v : 0.0f;
                v = v < 1.0f ? v : 1.0f;
            }
            fu->base_col[k][c] = v;
            packed |= quantise(v) << (8 * c);
        }
        fu->base_packed[k] = packed;
        // (without the colour distractor too: the shading of triangles applies scale and offset whatever the mode)
        if (k == 0u && (VIDEO || dc.mode != PXR_DISTRACT_COLOR)) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                fu->scale[c] = 1.0f;
                fu->offs[c] = 0.0f;
            }
        }
    }
}

// (the kernels that read their poses do not carry the arguments of those that make them)
template <bool POSED>
struct KinematicArgs {
    FkArgs args;
};
template <>
struct KinematicArgs<false> {};

// Register budget: two 80 KB workgroups share a compute unit, so 1024-thread groups need all
// 8 wave slots per SIMD (<= 64 VGPRs, <= 80 scalar registers); the smaller groups with windows use more (70).
// RAGGED: the width is no multiple of 4 (resolve_groups).
// WINDOWED: the key buffer does not hold the frame but the part of it that the bodies can touch (its window, found per
// frame in phase 1), a band of rows at a time if need be; the other pixels need no keys at all and are resolved by
// whichever wavefronts are done with the raster phase first.  The bodies of the articulated scenes touch 7 to 17 % of a
// frame, so most windows fit in one piece where the whole frame took two to five bands, each a walk over all binned
// triangles and three barriers.  Against bands of whole rows: 16 384 humanoid frames of 84x84 over a clip 493 -> 415 us,
// 1024 humanoid-and-box frames of 256x256 242 -> 156 us, 3648 of 128x128 237 -> 144 us, quadrupeds of 256x256 184 -> 98 us.
// Frames whose keys fit as a whole beside a second workgroup (64x64) do not take it: the same number of instructions, and
// the few wavefronts that get the window's pixels shade them all (65 536 x 3 frames 3.53 -> 3.81 ms).
// 1 << slabs_log2 workgroups share a windowed frame, each takes a run of its rows (and repeats the geometry).
// POSED: the poses are not read from memory but made here, from joint angles (pose_frame).
template <int NT, bool RAGGED, bool WINDOWED, bool VIDEO, bool POSED>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT >= 1024 ? 8 : (NT >= 768 ? 6 : 4)))) void render_kernel(
    const SceneConsts sc_value, const DistractConsts dc_value, const float* __restrict__ poses, const float* __restrict__ shapes,
    uint32_t S, uint32_t step0, uint32_t env0, uint8_t* __restrict__ frames, uint32_t* __restrict__ ids, uint32_t slabs_log2,
    const KinematicArgs<POSED>) {
    // (the workgroups that 256 compute units hold at most.  On a part of the chip more ask, which costs what is said below of every workgroup; the
    // number of its compute units as an argument would be a miss itself.)
    constexpr uint32_t kFirstRound = 256u * (2048u / NT);
    // Who asks: all wavefronts of the kernels that make poses and of those of up to 512 threads, of the larger ones the first wavefront of the
    // first workgroups on the chip, which find the arguments in no cache.
    // (In the kernels that make poses, which serve a few rounds at most, and in those of up to 512 threads, whose launches may be one round or
    // hundreds.  us without / with: 16 capsule frames of 32x32 6.3 / 5.7, 256 of 48x48 7.2 / 6.6, 512 meshes of 40x40 9.5 / 9.1, 256 chains from angles
    // 10.8 / 10.3; of many rounds 10 850 capsule frames of 48x48 58.0 / 57.7, 31 887 of 28x28 101.2 / 102.2.  Larger workgroups: 256 quadrupeds of 48x48
    // 7.18 / 6.96, of 64x64 7.77 / 7.60, 200 meshes of 64x64 8.31 / 8.15, 8 frames of 256x256 12.8 / 12.5; of many rounds, where it is only a branch at the
    // kernel's head, 65 536 x 3 frames of 64x64 3133 / 3145, 8503 capsule frames of 84x84 128.7 / 130.2, the others the same.  In every workgroup's first
    // wavefront 200 meshes 7.98, but 4096 quadrupeds 61.0 / 61.2 and 16 384 humanoids of 84x84 over a clip 378.5 / 381.)
    if constexpr (POSED || NT <= 512)
        request_arguments<POSED ? sizeof(RenderArguments) : offsetof(RenderArguments, fk)>();
    else if (blockIdx.x < kFirstRound && __builtin_amdgcn_readfirstlane((int)threadIdx.x) == 0)
        request_arguments<offsetof(RenderArguments, fk)>();
    // The largest whole-frame kernels without a clip, which are bound by instruction issue, have their arguments by value all the same: fewer
    // loads and waits, six registers parked.  By value / in place: 65 536 x 3 frames of 64x64 3470 / 3531 us, 4096 quadrupeds 64.2 / 65.5, 8503
    // capsule frames of 84x84 133 / 136.  (Windowed: 1024 quadruped frames of 161x160 45.2 / 44.4.)  So have the windowed ones of 768, of which
    // the LDS holds two workgroups: 16 384 humanoid frames of 84x84 over a clip 411.9 / 417.2 us, 4096 of 110x75 113.2 / 113.9.
    constexpr bool kByValue = !POSED && ((NT >= 1024 && !VIDEO && !WINDOWED) || (NT == 768 && WINDOWED));
    const SceneConsts& sc = kByValue ? sc_value : PXR_ARGUMENT(in_place, sc);
    const DistractConsts& dc = kByValue ? dc_value : PXR_ARGUMENT(in_place, dc);
    extern __shared__ __align__(16) unsigned char lds[];
    // the key buffer's LDS holds the cell codes and the candidate list until the keys are cleared
    uint32_t* vm = reinterpret_cast<uint32_t*>(lds + sc.lds_keys);
    uint16_t* cand = reinterpret_cast<uint16_t*>(lds + sc.lds_keys + sc.V * 4 + 4);  // (after the word of code 0)
    int2* vxy = reinterpret_cast<int2*>(lds + sc.lds_vxy);
    float* vd = reinterpret_cast<float*>(lds + sc.lds_vd);
    float* body = reinterpret_cast<float*>(lds + sc.lds_body);
    float* cxcy = reinterpret_cast<float*>(lds + sc.lds_cxcy);
    float4* rows = reinterpret_cast<float4*>(lds + sc.lds_rows);
    FrameUniforms* fu = reinterpret_cast<FrameUniforms*>(lds + sc.lds_misc);
    uint16_t* list = reinterpret_cast<uint16_t*>(lds + sc.lds_list);    // tiny bin grows up, small bin grows down
    uint16_t* list2 = reinterpret_cast<uint16_t*>(lds + sc.lds_large);  // large bin

    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t block = frame_of_block(blockIdx.x, gridDim.x);
    const uint32_t frame = WINDOWED ? block >> slabs_log2 : block;
    const uint32_t e = frame / S;
    const uint32_t step = step0 + (frame - e * S);
    const uint32_t env = env0 + e;
    const float* pose = poses + (size_t)frame * sc.K * 7;

    // camera position: fixed world-space offset from the root body.
    // The root's position is fetched with vector loads (through an offset of 0 that the compiler cannot see
    // through), although it is the same for every lane: as scalar loads they share their counter with the loads
    // of the kernel's arguments, every wait for one of those would wait for memory as well, and the first
    // wavefront would request its bodies' poses only after the root's position had arrived.
    uint32_t opaque_zero = 0u;
    asm volatile("" : "+v"(opaque_zero));
    const float* root_pos = pose + sc.root * 7 + opaque_zero;
    // (Only requested here.  The additions, and with them the wait, are made where phase 0 uses the eye: after the
    // bodies' lanes have requested their poses, in particular.  Phase 4 gets the eye through LDS, so that these
    // registers are free in between.)
    const float root_x = POSED ? 0.0f : root_pos[0], root_y = POSED ? 0.0f : root_pos[1], root_z = POSED ? 0.0f : root_pos[2];

    // (Phase 1's first template depends on nothing: it comes in while the bodies' transforms are made.  4096 quadrupeds 65.0 us
    // without, 64.5 with, 65 536 x 3 humanoids and boxes 3485 / 3467, 8503 capsule frames of 84x84 139.7 / 136.1.  The later
    // ones: kTemplatesAhead.)
    const uint32_t wave_first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid & ~63u));
    float4 tv_first = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (wave_first < sc.V) tv_first = (reinterpret_cast<const float4*>(sc.vtmpl) + wave_first)[lane];

    PXR_PHASE_BEGIN();
    // ---- phase 0: per-body transforms, per-frame draws, the three non-triangle colours
    // (16-wavefront groups: copied by the fourth wavefront on, the first three have chains of their own in this
    // phase; measured the other way round for the smaller groups)
    constexpr uint32_t kCopyFrom = NT >= 1024 ? 192u : 0u;
    if (tid >= kCopyFrom)
        for (uint32_t i = tid - kCopyFrom; i < sc.W + sc.H; i += NT - kCopyFrom) cxcy[i] = sc.cxcy[i];
    // The draws come before the bodies in the large workgroups, whose third wavefront (or last) they are: 65 536 x 3 frames of 64x64 3665 us the
    // other way round, now 3484, 4096 quadrupeds 69.6 / 65.1, 8503 capsule frames of 84x84 140.4 / 133.4, 1024 quadrupeds of 83x256 over a clip 92.7 /
    // 91.7.  In the small ones after them: 256 capsule frames of 48x48 7.2 us the other way round, now 6.8.
    constexpr bool kDrawFirst = NT >= 768;
    if constexpr (!POSED && kDrawFirst) draw_frame<NT, WINDOWED, VIDEO>(sc, dc, fu, lds, e, env, step, tid);
    if constexpr (POSED) {
        if (tid < 64u)
            pose_frame(PXR_ARGUMENT(in_place, fk), frame, body, fu, sc.root, sc.off[0], sc.off[1], sc.off[2], lane, !WINDOWED || (block & ((1u << slabs_log2) - 1u)) == 0u);
        else
            draw_frame<NT, WINDOWED, VIDEO>(sc, dc, fu, lds, e, env, step, tid);
        __syncthreads();
    }
    if (tid < 4u * sc.K) {
        // Four lanes per body: each rebuilds the body's rotation and takes one row of the work (the view matrix
        // has three rows, the light direction is the fourth): a quarter of the dot products on the chain.
        const uint32_t b = tid >> 2, part = tid & 3u;
        const float* p = POSED ? body + b * kBodyStride + 12 : pose + b * 7;
        // Everything the lane will need from memory is requested here, in one go: the pose, the lane's row of
        // (right, up, forward, light) from the table behind the bodies' constants, the body's shape and colour
        // (all four lanes of a body ask for the same: one request).
        const float* vr = sc.body_const + sc.K * 8u + 3u * part;
        const float r0 = vr[0], r1 = vr[1], r2 = vr[2];
        const float4 shp = *reinterpret_cast<const float4*>(shapes ? shapes + ((size_t)e * sc.K + b) * 4 : sc.body_const + b * 8);
        const float4 col = *reinterpret_cast<const float4*>(sc.body_const + b * 8 + 4);
        const float w = p[3], x = p[4], y = p[5], z = p[6];
        float at_x = 0.0f, at_y = 0.0f, at_z = 0.0f;
        if (POSED) {  // (a body's four lanes have read its pose before one of them writes over it)
            at_x = p[0];
            at_y = p[1];
            at_z = p[2];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        float R[3][3];
        R[0][0] = 1.0f - 2.0f * (y * y + z * z);
        R[0][1] = 2.0f * (x * y - w * z);
        R[0][2] = 2.0f * (x * z + w * y);
        R[1][0] = 2.0f * (x * y + w * z);
        R[1][1] = 1.0f - 2.0f * (x * x + z * z);
        R[1][2] = 2.0f * (y * z - w * x);
        R[2][0] = 2.0f * (x * z - w * y);
        R[2][1] = 2.0f * (y * z + w * x);
        R[2][2] = 1.0f - 2.0f * (x * x + y * y);
        const float eye_x = POSED ? fu->eye[0] : root_x + sc.off[0], eye_y = POSED ? fu->eye[1] : root_y + sc.off[1],
                    eye_z = POSED ? fu->eye[2] : root_z + sc.off[2];
        const float dx = (POSED ? at_x : p[0]) - eye_x, dy = (POSED ? at_y : p[1]) - eye_y, dz = (POSED ? at_z : p[2]) - eye_z;
        if (tid == 0u) {
            fu->ground_eye[0] = sc.eye_first ? eye_y : eye_x;
            fu->ground_eye[1] = sc.eye_first ? eye_x : eye_y;
            fu->ground_eye[2] = eye_z;
        }
        float* o = body + b * kBodyStride;
#pragma unroll
        for (int c = 0; c < 3; ++c) o[3u * part + (part == 3u ? 3u : 0u) + c] = dot3(r0, r1, r2, R[0][c], R[1][c], R[2][c]);
        if (part < 3u) o[9u + part] = dot3(r0, r1, r2, dx, dy, dz);
        // (written by all four lanes, the same values: in a branch of its own the compiler would request them
        // only there, after the arithmetic, and the first wavefront would wait for memory twice)
        *reinterpret_cast<float4*>(o + 16) = shp;
        *reinterpret_cast<float4*>(o + 20) = col;  // (the fourth float is padding)
    }
    if (tid >= 64u) {
        // The second wavefront on: one lane per image row prepares what all pixels of the row share: the row
        // part of the ray, and - when the camera does not roll, so that the ray's z does not depend on the
        // column (fma(+-0, cx, rz) == rz) - the whole ground test with its division.
        //   rows[j] = (rx, ry, tg or 0 for a miss, depth bits)   without roll
        //   rows[j] = (rx, ry, rz, -)                            with roll
        const bool no_roll = sc.Rt[2] == 0.0f;
        ResolveCtx g;
        const float eye_z = POSED ? fu->eye[2] : root_z + sc.off[2];
        g.eye_z = eye_z;
        g.inv_ez = 1.0f / eye_z;
        g.ground_ok = sc.ground_on && eye_z > 0.0f;
        for (uint32_t j = tid - 64u; j < sc.H; j += NT - 64u) {
            const float cyj = sc.cxcy[sc.W + j];
            const float rz = __builtin_fmaf(sc.Up[2], cyj, sc.Fw[2]);
            float4 r;
            r.x = __builtin_fmaf(sc.Up[0], cyj, sc.Fw[0]);
            r.y = __builtin_fmaf(sc.Up[1], cyj, sc.Fw[1]);
            r.z = rz;
            r.w = 0.0f;
            if (no_roll) {
                float tg;
                const u64 key = ground_key(sc, g, -rz, tg);
                r.z = key ? tg : 0.0f;  // (a hit has tg >= z_near > 0)
                r.w = __uint_as_float((uint32_t)(key >> 32));
            }
            rows[j] = r;
        }
    }
    if constexpr (!POSED && !kDrawFirst) draw_frame<NT, WINDOWED, VIDEO>(sc, dc, fu, lds, e, env, step, tid);
    // (Phase 1's arguments where they are read in place, asked for before the wait at the barrier: the compiler would load each where it is first
    // used, and the vertices would wait for them.  256 chains from angles 10.41 us without, 10.15 with; windowed frames of 256x256 147.2 / 149.4.)
    Projection pr = {sc.f, sc.z_near, sc.halfW, sc.halfH, sc.W, sc.H, false};
    asm("" : "+v"(pr.half_w), "+v"(pr.half_h));
    if constexpr (!kByValue && !WINDOWED) {
        asm volatile("" : : "s"(pr.f), "s"(pr.z_near), "s"(pr.W), "s"(pr.H));
    }
    pr.recip_long_form = !(pr.z_near >= kRecipMin);
    PXR_TIMED_BARRIER(0);
    PXR_PHASE_MARK(0);

    // ---- phase 1: instancing + projection + snap + cell code (one lane per template vertex)
    if (WINDOWED && tid >= NT - 64u) {
        // what the bodies can touch, by the last wavefront (the vertices of most scenes give it a trip less)
        add_reach(sc, body, fu->reach, lane);
    }
    if (tid == NT - 1) vm[sc.V] = 0u;  // the code that the padding of the pair table points at: no pixel centre on either axis
    // The largest whole-frame kernels are bound by what they issue here, the others by waiting.  us without / with: 65 536 x 3 frames of 64x64 3140 /
    // 3155, 4096 quadrupeds 60.2 / 60.7, 8503 capsule frames of 84x84 130.2 / 134.2; 10 humanoids with their layer 13.04 / 12.79, 16 384 of 84x84 over a
    // clip 380.8 / 377.7.
    constexpr bool kTemplatesAhead = NT < 1024 || WINDOWED || POSED;
    // (counted by wavefront: where its templates lie is a scalar then, and a lane's offset from there a constant)
    const float4* templates = reinterpret_cast<const float4*>(sc.vtmpl);
    const auto instance = [&](uint32_t v0, const float4 tv) {
        if (v0 + lane < sc.V) instance_vertex(pr, v0 + lane, tv, vxy, vd, vm);
    };
    if constexpr (kTemplatesAhead) {
        // The next templates are requested before the present ones are used, and without a condition: with one, the compiler cannot know how many
        // requests are under way and waits for the one just made.  Past the end the last ones are asked for again.
        const uint32_t last_templates = (sc.V - 1u) & ~63u;
        for (uint32_t v0 = wave_first; v0 < sc.V; v0 += 2 * NT) {
            const float4 tv_second = (templates + min(v0 + NT, last_templates))[lane];
            instance(v0, tv_first);
            if (v0 + NT >= sc.V) break;
            tv_first = (templates + min(v0 + 2 * NT, last_templates))[lane];
            instance(v0 + NT, tv_second);
        }
    } else {
        for (uint32_t v0 = wave_first; v0 < sc.V; v0 += NT) {
            instance(v0, tv_first);
            if (v0 + NT < sc.V) tv_first = (templates + (v0 + NT))[lane];
        }
    }
    // (phase 2a's first table entry depends on nothing in LDS: requested before the barrier, it arrives while the
    // wavefront waits there; later ones are requested a trip ahead)
    uint4 rec_next = make_uint4(0u, 0u, 0u, 0u);
    if (wave_first < sc.P) rec_next = (reinterpret_cast<const uint4*>(sc.pair_tbl) + wave_first)[lane];
    PXR_TIMED_BARRIER(1);
    PXR_PHASE_MARK(1);

    // ---- phase 2a: coarse binning, one lane per pair of edge-sharing triangles (q0,q1,q2), (q0,q2,q3).
    // A triangle can cover a pixel centre only if, on both axes, its vertices' cell codes are not all
    // the same (low half = x, high half = y).
    // The device table is padded to whole wavefronts with entries whose four addresses are those of a word that holds
    // code 0 (never a candidate), so no lane needs a bounds test, and a wavefront past the end leaves.  "Both halves
    // non-zero" is one 16 x 16-bit product; the ballots are taken from single comparisons (their masks as they
    // are) and combined as scalars.
    // (Two trips per turn of the loop, the two entries in flight changing roles: a single "next" variable costs six
    // register moves per trip.  Entries are requested ahead without a condition, past the end the table's last ones again: with one, the compiler cannot
    // know how many requests are under way and waits for the one just made.  65 536 x 3 frames of 64x64 3189 us, now 3140, 16 384 of 84x84 over a clip
    // 385 / 381.)
    const auto coarse_trip = [&](const uint4 rec) {
        const uint32_t m0 = lds_at<uint32_t>(rec.x & 0xFFFFu), m1 = lds_at<uint32_t>(rec.x >> 16), m2 = lds_at<uint32_t>(rec.y), m3 = lds_at<uint32_t>(rec.z);
        const uint32_t da = any_differ(m0, m1, m2), db = any_differ(m0, m2, m3);
        const uint32_t ta = rec.w & 0xFFFFu, tb = rec.w >> 16;
        const bool keep_a = halves_product(da) != 0u;
        const bool both_b = halves_product(db) != 0u, has_b = tb != kNoTriangle;
        const bool keep_b = both_b && has_b;
        const u64 ma = __ballot(keep_a), mb = __ballot(both_b) & __ballot(has_b);
        if (ma | mb) {
            uint32_t base;
            asm("" : "=v"(base));  // (only the first lane's is looked at)
            if (lane == 0) base = atomicAdd(&fu->n_cand, (uint32_t)(__popcll(ma) + __popcll(mb)));
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            // (the first triangles of the wavefront's entries, then the second ones: the order is free)
            if (keep_a) cand[base + lanes_below(ma)] = (uint16_t)ta;
            if (keep_b) cand[base + (uint32_t)__popcll(ma) + lanes_below(mb)] = (uint16_t)tb;
        }
    };
    {
        const uint4* table = reinterpret_cast<const uint4*>(sc.pair_tbl);
        uint4 rec_a = rec_next;
        for (uint32_t p0 = wave_first; p0 < sc.P; p0 += 2 * NT) {
            const uint4 rec_b = (table + min(p0 + NT, sc.P - 64u))[lane];
            coarse_trip(rec_a);
            if (p0 + NT >= sc.P) break;
            rec_a = (table + min(p0 + 2 * NT, sc.P - 64u))[lane];
            coarse_trip(rec_b);
        }
    }
    PXR_TIMED_BARRIER(2);
    PXR_PHASE_MARK(2);

    // ---- phase 2b: exact binning, one lane per candidate triangle: reject, area sign, pixel range,
    // then one of three bins by the number of candidate pixel centres (one packed LDS atomic per wave).
    const uint32_t n_cand = fu->n_cand;
    // (the whole frame, or its columns and this workgroup's rows)
    RasterWindow image = {0, (int)sc.W, 0, (int)sc.H, sc.pitch};
    if (WINDOWED) {
        const uint32_t slab = block & ((1u << slabs_log2) - 1u);
        image.y_lo = (int)((slab * sc.H) >> slabs_log2);
        image.y_end = (int)(((slab + 1u) * sc.H) >> slabs_log2);
    }
    // (Where the candidates take several trips - smaller workgroups, taller frames - a lane's candidate and its entry
    // of the index table are requested a trip ahead, without a branch: a lane past the end reads a list entry that
    // nobody wrote and clamps it into the table.  The 1024-thread whole-frame kernel sees its ~900 candidates in one trip
    // and keeps the plain form: 256 chains from angles 10.1 us, 10.4 with requests ahead.)
    constexpr bool kAhead = NT < 1024 || WINDOWED;
    uint32_t t_ahead = 0;
    uint2 ti_ahead = make_uint2(0u, 0u);
    if (kAhead) {
        t_ahead = cand[min(tid, sc.T - 1u)];
        ti_ahead = reinterpret_cast<const uint2*>(sc.tri_idx)[min(t_ahead, sc.T - 1u)];
    }
    for (uint32_t k0 = 0; k0 < n_cand; k0 += NT) {
        const uint32_t k = k0 + tid;
        uint32_t t = t_ahead;
        uint2 ti = ti_ahead;
        if (kAhead) {
            if (k0 + NT < n_cand) {
                t_ahead = cand[min(k + NT, sc.T - 1u)];
                ti_ahead = reinterpret_cast<const uint2*>(sc.tri_idx)[min(t_ahead, sc.T - 1u)];
            }
        } else if (k < n_cand) {
            t = cand[k];
            ti = reinterpret_cast<const uint2*>(sc.tri_idx)[t];
        }
        // candidate pixels: none = dropped or binned already, kByWave = whatever their number, the triangle is a whole wavefront's
        constexpr uint32_t kByWave = 0xFFFFu;
        uint32_t n_px = 0;
        if (k < n_cand) {
            const Corners q = gather_corners(ti, sc.lds_vxy);
            if (__builtin_expect(imin3(q.ax, q.bx, q.cx) > kBehindX, 1)) {
                const PixelBox box = candidate_pixels(image, q);
                bool front = __mul24(q.bx - q.ax, q.cy - q.ay) > __mul24(q.by - q.ay, q.cx - q.ax);
                uint32_t n = __umul24((uint32_t)(box.i_end - box.i0), (uint32_t)(box.j_end - box.j0));  // (each at most 512)
                const bool wide = !q.narrow();
                if (__builtin_expect(__ballot(wide) != 0ull, 0)) {
                    // (The loops of the tiny and small bins take 24-bit products for granted.  Wide triangles that show few pixels have a bin of their
                    // own, from the other end of the large bin's array.  With a turn of a whole wavefront for each, as if they were large, 2048 frames at whose
                    // edges 400 of them end: 64x64 216 us, now 44, 96x96 246 / 77, 256x256 424 / 233.  Nothing but the room for it costs the others anything:
                    // 65 536 x 3 frames of 64x64 3072 / 3076, 256 chains from angles 10.11 / 10.22, 16 384 of 84x84 over a clip 374.0 / 376.5.)
                    bool few = false;
                    if (wide) {
                        front = (long long)(q.bx - q.ax) * (long long)(q.cy - q.ay) > (long long)(q.by - q.ay) * (long long)(q.cx - q.ax);
                        few = front && !box.empty() && n <= kSmallMaxPixels;
                        n = few ? 0u : kByWave;
                    }
                    const u64 mw = __ballot(few);
                    if (mw) {
                        const uint32_t first = (uint32_t)__builtin_ctzll(mw);
                        uint32_t at;
                        asm("" : "=v"(at));  // (only that lane's is looked at)
                        if (lane == first)
                            at = WINDOWED ? atomicAdd(&fu->n_few, (uint32_t)__popcll(mw)) : (uint32_t)(atomicAdd(&fu->bins, (u64)__popcll(mw) << 48) >> 48);
                        at = (uint32_t)__builtin_amdgcn_readlane((int)at, (int)first);
                        if (few) (list2 + (sc.T - 1 - at))[-(int)lanes_below(mw)] = (uint16_t)t;
                    }
                }
                n_px = (front & !box.empty()) ? n : 0u;
            } else if (tri_kind(q) == kTriClip) {
                n_px = kByWave;
            }
        }
        const u64 some = __ballot(n_px != 0u), up_to_tiny = __ballot(n_px <= kTinyMaxPixels), m3 = __ballot(n_px > kSmallMaxPixels);
        if (some) {
            const u64 m1 = some & up_to_tiny, m2 = ~(up_to_tiny | m3);
            u64 old;
            asm("" : "=v"(old));  // (only the first lane's is looked at)
            if (lane == 0)
                old = atomicAdd(&fu->bins, (u64)__popcll(m1) | ((u64)__popcll(m2) << 16) | ((u64)__popcll(m3) << 32));
            const uint32_t old_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)old);
            const uint32_t old_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(old >> 32));
            const bool tiny = n_px - 1u < kTinyMaxPixels, large = n_px > kSmallMaxPixels;
            if (tiny) list[(old_lo & 0xFFFFu) + lanes_below(m1)] = (uint16_t)t;
            if (!large && n_px > kTinyMaxPixels) (list + (sc.T - 1 - (old_lo >> 16)))[-(int)lanes_below(m2)] = (uint16_t)t;
            if (large) list2[(WINDOWED ? old_hi : old_hi & 0xFFFFu) + lanes_below(m3)] = (uint16_t)t;
        }
    }
    // (the frame's window, made of what was found in phase 1: the last wavefront has the fewest candidates)
    if (WINDOWED && tid >= NT - 64u) make_window(sc, VIDEO ? sc.key_capacity_video : sc.key_capacity, fu, (uint32_t)image.y_lo, (uint32_t)image.y_end, lane);
    PXR_TIMED_BARRIER(3);
    PXR_PHASE_MARK(3);

    // Windowed frames whose window does not fit the key buffer are rendered a band of its rows at a time: geometry
    // work (phases 0-2) is done once, raster and resolve per band.
    uint32_t bands_done = 0;
    uint32_t band_round = 0;  // rounds of the band-list builder so far (picks the counter slot)
    const uint32_t tid_kept = tid;
    bool more_bands;
    do {
        const SceneConsts& scb = WINDOWED ? PXR_ARGUMENT(reloaded, sc) : sc;
        const DistractConsts& dcb = WINDOWED ? PXR_ARGUMENT(reloaded, dc) : dc;
        // (In the band loop everything is derived again from the reloaded arguments and from a thread index the
        // compiler cannot see through: nothing but the band counter and the index stays live from band to band.)
        uint32_t tid = tid_kept;
        if (WINDOWED) asm volatile("" : "+v"(tid));
        const uint32_t lane = tid & 63u;
        u64* keys = reinterpret_cast<u64*>(lds + scb.lds_keys);
        int2* vxy = reinterpret_cast<int2*>(lds + scb.lds_vxy);
        float* vd = reinterpret_cast<float*>(lds + scb.lds_vd);
        float* cxcy = reinterpret_cast<float*>(lds + scb.lds_cxcy);
        float4* rows = reinterpret_cast<float4*>(lds + scb.lds_rows);
        FrameUniforms* fu = reinterpret_cast<FrameUniforms*>(lds + scb.lds_misc);
        uint16_t* list = reinterpret_cast<uint16_t*>(lds + scb.lds_list);
        uint16_t* list2 = reinterpret_cast<uint16_t*>(lds + scb.lds_large);
        RasterWindow win = {0, (int)scb.W, 0, (int)scb.H, scb.pitch};
        ResolveRange range = {};
        uint32_t n_keys = scb.pitch * scb.H;
        bool by_lists = false;
        if (WINDOWED) {
            const auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
            range.x0 = uniform(fu->win_x0);
            range.groups = uniform(fu->win_groups);
            range.magic = uniform(fu->win_magic);
            const uint32_t y0 = uniform(fu->win_y0), n_rows = uniform(fu->win_rows), held = uniform(fu->band_rows);
            range.y0 = y0 + bands_done * held;
            range.rows = min(held, n_rows - bands_done * held);
            more_bands = (bands_done + 1u) * held < n_rows;
            win.pitch = range.groups * 4u;
            win.x_lo = (int)range.x0;
            win.x_end = (int)min(range.x0 + win.pitch, scb.W);
            win.y_lo = (int)range.y0;
            win.y_end = (int)(range.y0 + range.rows);
            n_keys = win.pitch * held;
            if (__builtin_expect(n_rows > held, 0)) {  // (most windows fit in one piece: 16 384 frames of 84x84 424 us without the branch, now 415)
                const uint32_t n_tiny = uniform((uint32_t)fu->bins & 0xFFFFu), n_small = uniform((uint32_t)fu->bins >> 16),
                               n_large = uniform((uint32_t)(fu->bins >> 32)), n_few = uniform(fu->n_few), n_binned = n_tiny + n_small + n_large;
                // (the lists live in what the bins leave free of their arrays; at most half of a closed body's triangles are binned)
                const bool room = n_tiny + n_small + min(n_tiny, (uint32_t)NT) <= scb.T && n_large + n_few + min(n_small + n_large, (uint32_t)NT) <= scb.T;
                by_lists = room && n_large + (n_small >> (6u - kSmallLanesLog2)) >= (n_binned <= NT ? kBandListsFromOneRound : kBandListsFrom);
            }
        } else {
            more_bands = false;
        }
        const auto resolve = [&](auto part, const ResolveRange& r) {
            constexpr ResolvePart PART = decltype(part)::value;
            ResolveCtx rc;
            const float eye_x = fu->ground_eye[0], eye_y = fu->ground_eye[1], eye_z = fu->ground_eye[2];
            rc.eye_x = eye_x;
            rc.eye_y = eye_y;
            rc.eye_z = eye_z;
            const bool no_roll = scb.Rt[2] == 0.0f;
            rc.inv_ez = 0.0f;
            if (!no_roll) {  // (without roll the row table already holds the ground test)
                asm volatile("" ::: "memory");  // (a branch, not a select: the compiler would do the division either way)
                rc.inv_ez = 1.0f / eye_z;
            }
            rc.ground_ok = scb.ground_on && eye_z > 0.0f;
            // (in place also in the kernels that have their arguments by value: four scalar registers less that are kept from the kernel's head on.  65 536 x 3 frames
            // of 64x64 3113 us, eight scalars parked, now 3064, 4096 quadrupeds 61.0 / 60.0.)
            const SceneConsts& late = kByValue && !WINDOWED ? PXR_ARGUMENT(in_place, sc) : scb;
            rc.tri_shade = late.tri_shade;
            rc.ambient = late.ambient;
            rc.diffuse = late.diffuse;
            rc.alpha = dcb.alpha;
            rc.vframe = nullptr;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                rc.scale[c] = fu->scale[c];
                rc.offs[c] = fu->offs[c];
            }
            rc.col_addr = scb.lds_misc + (uint32_t)offsetof(FrameUniforms, base_col);
#pragma unroll
            for (int c = 0; c < 3; ++c) rc.packed[c] = VIDEO ? 0u : fu->base_packed[c];
            rc.vlut = scb.lds_vlut;
            if (VIDEO) rc.vframe = dcb.video + (size_t)fu->video_frame * scb.npix * 3;
            uint8_t* out = frames + (size_t)frame * scb.npix * 3;
            uint32_t* out_ids = ids ? ids + (size_t)frame * scb.npix : nullptr;
            // uniform scene properties select a specialised loop (kept out of the per-pixel code)
            // (an eye that is a NaN makes ground points NaNs: such a frame takes the general loop, which is exact
            // for a unit cell as well)
            if (scb.checker_short_form && eye_x == eye_x && eye_y == eye_y) {
                if (no_roll && scb.Rt[0] == 0.0f)
                    resolve_groups<NT, true, true, VIDEO, RAGGED, PART, true>(scb, rc, cxcy, rows, keys, out, out_ids, tid, r);
                else if (no_roll)
                    resolve_groups<NT, true, true, VIDEO, RAGGED, PART>(scb, rc, cxcy, rows, keys, out, out_ids, tid, r);
                else
                    resolve_groups<NT, true, false, VIDEO, RAGGED, PART>(scb, rc, cxcy, rows, keys, out, out_ids, tid, r);
            } else {
                if (no_roll)
                    resolve_groups<NT, false, true, VIDEO, RAGGED, PART>(scb, rc, cxcy, rows, keys, out, out_ids, tid, r);
                else
                    resolve_groups<NT, false, false, VIDEO, RAGGED, PART>(scb, rc, cxcy, rows, keys, out, out_ids, tid, r);
            }
        };
        // wide triangles that show few pixels: a team of lanes each, every band as they lie in the bin (rare: few scenes have one)
        const auto raster_wide_few = [&](uint32_t n_few) {
            if (__builtin_expect(n_few == 0u, 1)) return;
            constexpr uint32_t kTeam = 1u << kSmallLanesLog2;
            const SceneConsts& scf = WINDOWED ? PXR_ARGUMENT(reloaded, sc) : scb;
            const uint16_t* few = reinterpret_cast<const uint16_t*>(lds + scf.lds_large) + (scf.T - 1);
            for (uint32_t k = tid >> kSmallLanesLog2; k < n_few; k += NT >> kSmallLanesLog2) {
                const uint32_t t = *(few - k);
                raster_few(scf, win, t, reinterpret_cast<const uint2*>(scf.tri_idx)[t], keys, (int)(tid & (kTeam - 1u)), (int)kSmallLanesLog2);
            }
        };
        if (!by_lists) {
            // Windows in one piece, and in bands if walking all bins for every band costs less than picking a band's
            // triangles out.
            if (WINDOWED && bands_done) __syncthreads();  // the previous band is resolved (its lanes left their keys cleared)
            // The bins are complete: each lane asks now for the first triangle it will raster from the small and from the
            // tiny bin (its list entry, then its entry of the index table), so that they come in from memory while the keys
            // are cleared and the barrier is waited at.
            const u64 bins = fu->bins;
            const uint32_t n_tiny = (uint32_t)bins & 0xFFFFu, n_small = (uint32_t)bins >> 16, n_upper = (uint32_t)(bins >> 32),
                           n_large = WINDOWED ? n_upper : n_upper & 0xFFFFu;
            constexpr uint32_t kTeam = 1u << kSmallLanesLog2;
            const uint2* tri_table = reinterpret_cast<const uint2*>(scb.tri_idx);
            // (Asked for without a branch, so that nothing has to wait for the answers here: a lane with no triangle in a
            // bin reads a list entry that may never have been written and clamps it into the table.)
            uint32_t t_small = list[scb.T - 1 - min(tid >> kSmallLanesLog2, scb.T - 1u)];
            uint32_t t_tiny = list[min(NT - 1 - tid, scb.T - 1u)];
            uint2 ti_small = tri_table[min(t_small, scb.T - 1u)], ti_tiny = tri_table[min(t_tiny, scb.T - 1u)];

            // codes and candidates are dead: clear the pixel keys they shared LDS with (0 = background at depth 0)
            // (two keys per store; the region is padded to 16 bytes, so an odd count may clear one key more)
            if (!WINDOWED || bands_done == 0) {
                for (uint32_t p = tid; p < (n_keys + 1u) >> 1; p += NT)
                    reinterpret_cast<uint4*>(keys)[p] = make_uint4(0u, 0u, 0u, 0u);
                PXR_TIMED_BARRIER(4);
            }
            PXR_PHASE_MARK(4);

            // ---- phase 3: raster + z-test into the LDS key buffer.  The bins start at different
            // lanes of the workgroup so that all waves get a share.
            // The hardware favours a workgroup's older wavefronts when several want to issue, so the youngest finish a
            // phase last: the heavier bin goes to the oldest.
            // small: a team of lanes per triangle, from the first lane up
            // (a lane's first triangle of each was requested before the barrier; the next one is at the loop's end)
            for (uint32_t k = tid >> kSmallLanesLog2; k < n_small;) {
                raster_binned<WINDOWED>(win, t_small, ti_small, scb.lds_vxy, scb.lds_vd, keys, (int)(tid & (kTeam - 1u)), (int)kSmallLanesLog2);
                k += NT >> kSmallLanesLog2;
                if (k < n_small) {
                    t_small = list[scb.T - 1 - k];
                    ti_small = tri_table[t_small];
                }
            }
            // tiny: one lane per triangle, from the last lane down
            for (uint32_t k = NT - 1 - tid; k < n_tiny;) {
                raster_binned<WINDOWED>(win, t_tiny, ti_tiny, scb.lds_vxy, scb.lds_vd, keys, 0, 0);
                k += NT;
                if (k < n_tiny) {
                    t_tiny = list[k];
                    ti_tiny = tri_table[t_tiny];
                }
            }
            // large: a whole wave per triangle, starting in the middle waves
            for (uint32_t k = ((tid >> 6) + NT / 128) % (NT / 64); k < n_large; k += NT / 64)
                raster_large(scb, win, list2[k], tri_table[list2[k]], vxy, vd, keys, (int)lane);
            if (!WINDOWED) raster_wide_few((uint32_t)__builtin_amdgcn_readfirstlane((int)(n_upper >> 16)));
        } else {
            // Windows in bands of many triangles.  Every band walks the frame's bins again, but only to pick out the triangles that can
            // touch its rows: a dense pass, one lane per binned triangle and round of NT, that compacts them (ballot,
            // one packed atomic per wavefront) into the round's own short lists, from which the raster loops then
            // work as above.  A band that holds a twentieth of the frame's triangles rasters a
            // twentieth of them, not all.
            // The lists lie in what the bins leave free of their arrays: tiny behind the tiny bin in the first, large behind the
            // large bin in the second, small from its other end (the wide triangles with few pixels) downwards.  (Small in the first as well would leave no
            // room for them where more than half of the triangles are binned: meshes of 256x256 72 us, now 67.)  (In 4 KB of their own they cost every
            // windowed frame 512 keys, and often a band where a body at the near plane makes the window the whole frame: 3520
            // such humanoid-and-box frames of 84x84 346 us, now 265, 1472 of 128x128 301, now 263; 128x128 in view 70.0, now 64.3.)
            if (bands_done) __syncthreads();  // the previous band is resolved (its lanes left their keys cleared)
            const u64 bins = fu->bins;
            const uint32_t n_tiny = (uint32_t)bins & 0xFFFFu, n_small = (uint32_t)bins >> 16, n_large = (uint32_t)(bins >> 32);
            const uint32_t n_binned = n_tiny + n_small + n_large;
            uint16_t* band_tiny = list + n_tiny;                     // (grows up)
            uint16_t* band_small = list2 + (scb.T - 1 - fu->n_few);  // (grows down)
            uint16_t* band_large = list2 + n_large;
            constexpr uint32_t kTeam = 1u << kSmallLanesLog2;
            const uint2* tri_table = reinterpret_cast<const uint2*>(scb.tri_idx);
            if (bands_done == 0) {
                // the first band's keys share LDS with the cell codes and the candidate list, dead by now
                for (uint32_t p = tid; p < (n_keys + 1u) >> 1; p += NT)
                    reinterpret_cast<uint4*>(keys)[p] = make_uint4(0u, 0u, 0u, 0u);
            }
            uint32_t base = 0;
            do {
                if (base) __syncthreads();  // (the lists of the round before are read)
                // ---- this round's share of the bins -> the triangles among them that touch the band's rows
                const uint32_t slot = band_round & 1u;
                if (tid == 0) fu->band_bins[slot ^ 1u] = 0ull;  // (last read before the barrier behind the round before this one)
                const uint32_t k = base + tid;
                int cls = 0;
                uint32_t t = 0;
                if (k < n_binned) {
                    cls = k < n_tiny ? 1 : (k < n_tiny + n_small ? 2 : 3);
                    t = cls == 1 ? list[k] : (cls == 2 ? list[scb.T - 1 - (k - n_tiny)] : list2[k - n_tiny - n_small]);
                    int j0 = 0, j_end = 0;
                    if (tri_rows(tri_table[t], scb.lds_vxy, j0, j_end) == kTriPlain && (j0 >= win.y_end || j_end <= win.y_lo)) cls = 0;
                }
                const u64 m1 = __ballot(cls == 1), m2 = __ballot(cls == 2), m3 = __ballot(cls == 3);
                if (m1 | m2 | m3) {
                    u64 old = 0;
                    if (lane == 0)
                        old = atomicAdd(&fu->band_bins[slot], (u64)__popcll(m1) | ((u64)__popcll(m2) << 16) | ((u64)__popcll(m3) << 32));
                    const uint32_t old_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)old);
                    const uint32_t old_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(old >> 32));
                    // (a round looks at NT triangles: both arrays have that many entries left)
                    if (cls == 1) band_tiny[(old_lo & 0xFFFFu) + lanes_below(m1)] = (uint16_t)t;
                    if (cls == 2) *(band_small - ((old_lo >> 16) + lanes_below(m2))) = (uint16_t)t;
                    if (cls == 3) band_large[old_hi + lanes_below(m3)] = (uint16_t)t;
                }
                PXR_TIMED_BARRIER(4);
                PXR_PHASE_MARK(4);

                // ---- phase 3 from the round's lists (lane teams as above)
                const u64 bb = fu->band_bins[slot];
                const uint32_t b_tiny = (uint32_t)bb & 0xFFFFu, b_small = (uint32_t)bb >> 16, b_large = (uint32_t)(bb >> 32);
                for (uint32_t i = tid >> kSmallLanesLog2; i < b_small; i += NT >> kSmallLanesLog2) {
                    const uint32_t ts = *(band_small - i);
                    raster_binned<WINDOWED>(win, ts, tri_table[ts], scb.lds_vxy, scb.lds_vd, keys, (int)(tid & (kTeam - 1u)), (int)kSmallLanesLog2);
                }
                if (NT - 1 - tid < b_tiny) {
                    const uint32_t tt = band_tiny[NT - 1 - tid];
                    raster_binned<WINDOWED>(win, tt, tri_table[tt], scb.lds_vxy, scb.lds_vd, keys, 0, 0);
                }
                for (uint32_t i = ((tid >> 6) + NT / 128) % (NT / 64); i < b_large; i += NT / 64)
                    raster_large(scb, win, band_large[i], tri_table[band_large[i]], vxy, vd, keys, (int)lane);
                ++band_round;
                base += NT;
            } while (base < n_binned);
        }
        if (WINDOWED) raster_wide_few((uint32_t)__builtin_amdgcn_readfirstlane((int)fu->n_few));
        if (WINDOWED && bands_done == 0) {
            // The first band's raster phase ends with the pixels beside the window, in chunks for whichever wavefront is
            // done: they cover the wait for the phase's longest chains.
            const uint32_t slab = frame_of_block(blockIdx.x, gridDim.x) & ((1u << slabs_log2) - 1u);
            ResolveRange beside = range;
            beside.rows = (uint32_t)__builtin_amdgcn_readfirstlane((int)fu->win_rows);
            beside.first_row = (slab * scb.H) >> slabs_log2;
            beside.end_row = ((slab + 1u) * scb.H) >> slabs_log2;
            beside.side_groups = ((scb.W + 3u) >> 2) - range.groups;
            beside.side_magic = (uint32_t)__builtin_amdgcn_readfirstlane((int)fu->side_magic);
            beside.ticket = &fu->ticket;
            resolve(std::integral_constant<ResolvePart, kBesideWindow>{}, beside);
        }
        PXR_TIMED_BARRIER(5);
        PXR_PHASE_MARK(5);

        // ---- phase 4: resolve + shade + distractor + pack + store
        if (WINDOWED)
            resolve(std::integral_constant<ResolvePart, kInsideWindow>{}, range);
        else
            resolve(std::integral_constant<ResolvePart, kWholeFrame>{}, range);
        ++bands_done;
    } while (WINDOWED && more_bands);
    PXR_PHASE_MARK(6);
    PXR_PHASE_END();
}

template <int NT, bool RAGGED, bool WINDOWED, bool VIDEO>
int launch_one(const SceneConsts& sc, const DistractConsts& dc, const FkArgs* fk, const float* d_poses, const float* d_shapes,
               uint32_t n_frames, uint32_t S, uint32_t step0, uint32_t env0, uint8_t* d_frames, uint32_t* d_ids,
               uint32_t slabs_log2, hipStream_t stream, std::string& err) {
    if constexpr (makes_poses(NT, WINDOWED)) {
        if (fk)
            hipLaunchKernelGGL((render_kernel<NT, RAGGED, WINDOWED, VIDEO, true>), dim3(n_frames << slabs_log2), dim3(NT), sc.lds_total, stream,
                               sc, dc, d_poses, d_shapes, S, step0, env0, d_frames, d_ids, slabs_log2, KinematicArgs<true>{*fk});
    } else if (fk) {
        err = "this workgroup size has no kernel that makes poses";
        return PXR_ERR_UNSUPPORTED;
    }
    if (!fk)
        hipLaunchKernelGGL((render_kernel<NT, RAGGED, WINDOWED, VIDEO, false>), dim3(n_frames << slabs_log2), dim3(NT), sc.lds_total, stream,
                           sc, dc, d_poses, d_shapes, S, step0, env0, d_frames, d_ids, slabs_log2, KinematicArgs<false>{});
    const hipError_t rc = hipGetLastError();
    if (rc != hipSuccess) {
        err = std::string("kernel launch failed: ") + hipGetErrorString(rc);
        return PXR_ERR_DEVICE;
    }
    return PXR_OK;
}

template <int NT, bool RAGGED, bool WINDOWED, bool VIDEO, bool POSED = false>
int prepare_one(uint32_t lds_bytes, std::string& err) {
    hipFuncAttributes attr;
    const void* kernel = reinterpret_cast<const void*>(&render_kernel<NT, RAGGED, WINDOWED, VIDEO, POSED>);
    if (hipFuncGetAttributes(&attr, kernel) != hipSuccess ||
        attr.sharedSizeBytes != 0) {
        err = "the render kernel has static LDS in front of its dynamic segment (LDS addresses in the tables assume none)";
        return PXR_ERR_DEVICE;
    }
    const hipError_t rc = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (rc != hipSuccess) {
        err = std::string("hipFuncSetAttribute(MaxDynamicSharedMemorySize) failed: ") + hipGetErrorString(rc);
        return PXR_ERR_DEVICE;
    }
    if constexpr (!POSED && makes_poses(NT, WINDOWED)) return prepare_one<NT, RAGGED, WINDOWED, VIDEO, true>(lds_bytes, err);
    return PXR_OK;
}

template <int NT>
int prepare_all(uint32_t cap, std::string& err) {
    int rc;
    if ((rc = prepare_one<NT, false, false, false>(cap, err))) return rc;
    if ((rc = prepare_one<NT, false, true, false>(cap, err))) return rc;
    if ((rc = prepare_one<NT, true, false, false>(cap, err))) return rc;
    if ((rc = prepare_one<NT, true, true, false>(cap, err))) return rc;
    if ((rc = prepare_one<NT, false, false, true>(cap, err))) return rc;
    if ((rc = prepare_one<NT, false, true, true>(cap, err))) return rc;
    if ((rc = prepare_one<NT, true, false, true>(cap, err))) return rc;
    if ((rc = prepare_one<NT, true, true, true>(cap, err))) return rc;
    return PXR_OK;
}

#if defined(PXR_PROFILING_BUILD) && defined(PXR_PHASE_TIMING)
#include "profiling/phase_exports.h"
#endif

}  // namespace

int prepare_kernels(std::string& err) {
    // The attribute is a per-kernel cap, not a per-launch size: raise it to the whole 160 KB, so that scenes
    // of any size can coexist.
    const uint32_t cap = 160u * 1024u;
    int rc;
    if ((rc = prepare_all<256>(cap, err))) return rc;
    if ((rc = prepare_all<512>(cap, err))) return rc;
    if ((rc = prepare_all<768>(cap, err))) return rc;
    if ((rc = prepare_all<1024>(cap, err))) return rc;
    return PXR_OK;
}

int launch_render(const SceneConsts& sc, const DistractConsts& dc, const FkArgs* fk, const float* d_poses, const float* d_shapes,
                  uint32_t n_frames, uint32_t S, uint32_t step0, uint32_t env0, uint8_t* d_frames, uint32_t* d_ids,
                  uint32_t block_threads, uint32_t n_cus, void* stream, std::string& err) {
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const bool ragged = (sc.W % 4u) != 0u, windowed = sc.key_capacity != 0u;
    // (the video distractor has kernels of its own: the others carry none of its code, and the other way round)
    const bool video = dc.mode == PXR_DISTRACT_VIDEO;
    // A windowed frame is shared by several workgroups while that gives every workgroup of the launch a compute unit of its
    // own: geometry is repeated, raster and resolve, which dominate large frames, are split.  us per launch without / with
    // 2 / 4 / 8 / 16 slabs, humanoid and box: 256x256, 8 frames 33.8 / 26.1 / 24.6 / 20.0 / 17.7, 32 frames 43.2 / 27.9 /
    // 25.7 / 20.8 / 29.6, 100 frames 45.1 / 30.1 / 46.1 / 51.1 / 74.5, 200 frames 46.6 / 50.5 and up; 128x128, 32 frames 21.2 /
    // 17.4 / 14.5 / 13.3 / 14.7; quadruped 84x84, 64 frames 10.8 / 10.2 / 10.1 / 11.7 / 20.0.  (A slab has 4 rows or more.)
    uint32_t slabs_log2 = 0;
    while (windowed && slabs_log2 < 5u && ((uint64_t)n_frames << (slabs_log2 + 1u)) <= n_cus && (sc.H >> (slabs_log2 + 1u)) >= 4u) ++slabs_log2;
#define PXR_ARGS sc, dc, fk, d_poses, d_shapes, n_frames, S, step0, env0, d_frames, d_ids, slabs_log2, st, err
#define PXR_LAUNCH_V(NT, V)                                                                                      \
    return ragged ? (windowed ? launch_one<NT, true, true, V>(PXR_ARGS) : launch_one<NT, true, false, V>(PXR_ARGS)) \
                  : (windowed ? launch_one<NT, false, true, V>(PXR_ARGS) : launch_one<NT, false, false, V>(PXR_ARGS))
#define PXR_LAUNCH(NT)                   \
    if (video) PXR_LAUNCH_V(NT, true);   \
    PXR_LAUNCH_V(NT, false)
    switch (block_threads) {
        case 256: PXR_LAUNCH(256);
        case 512: PXR_LAUNCH(512);
        case 768: PXR_LAUNCH(768);
        case 1024: PXR_LAUNCH(1024);
        default:
            err = "block_threads must be 256, 512, 768 or 1024";
            return PXR_ERR_INVALID_ARG;
    }
#undef PXR_LAUNCH
#undef PXR_LAUNCH_V
#undef PXR_ARGS
}

}  // namespace pxr
