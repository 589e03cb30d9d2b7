// Ray casting of the imaging sonar's returns on gfx950 (Sec. III-A.2 of
// arXiv 2503.01074 obtains the returns by ray tracing the scene): closest
// hits of a beam x elevation ray pattern against a triangle mesh in a binary
// bounding-volume hierarchy (built on the host, bvh.cpp).
//
//   k_raycast_packet  (patterns of angular steps that are fine against the
//              scene's triangles) a wave traverses the
//              hierarchy once for an 8 x 8 patch of beams and rays: node and
//              triangle records come through scalar loads, each lane tests the
//              boxes for its own ray, and the wave's stack holds references
//              with the mask of the lanes that met the box.
//   k_raycast  (the others) each lane traverses for itself, with a stack
//              of its own in LDS (thread-minor, so a wave's stack accesses are
//              conflict-free); over dense scenes a wave takes the rays of one
//              beam.
//
// Both are ordered: an inner node holds both child boxes (one 64-byte record),
// the nearer child is taken first and the other deferred; leaves hold at most
// 8 triangles, each tested with the Moller-Trumbore algorithm in single
// precision; the first triangle visited by a ray's own ordered traversal wins
// a tie.  The hit point is written as t times the sensor-frame direction, the
// normal as R^T of the hit triangle's unit normal: the return buffers the
// sonar image formation reads.
//
// Several poses go in one launch (grid.y = pose); their descriptors travel in
// the kernel arguments, so a cast allocates nothing.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>

#include "../../include/oceansim.h"
#include "device.hpp"
#include "host.hpp"
#include "launch.hpp"
#include "scene.hpp"

struct oceansim_scene {
    int device = 0;
    osim::BvhNode *nodes = nullptr;
    osim::BvhTri *tris = nullptr;
    int root = 0;
    int empty = 1;
    double lo[3], hi[3], tri_area;   // see BvhBuild
    oceansim_scene_info info{};
};

namespace osim {
namespace {

constexpr int kRayThreads = 256;
constexpr int kRayLineThreads = 128;   // of a workgroup whose waves take lines of rays (see ray_shape)
constexpr int kRayXcdRun = 16;         // consecutive tiles one XCD takes
constexpr int kRayFramesPerLaunch = 16;
constexpr float kSlabWiden = 1.00000036f;   // 1 + 2 gamma_3, gamma_n = n eps / (1 - n eps), eps = 2^-24

struct RayFrameDev {
    float o[3];
    float R[9];
    float az0, daz, el0, del, t_max;
    int nb, nr;
    int br_log2;      // rays of a beam in a workgroup's tile (see RayTile), log2
    int wr_log2;      // and in a wave's patch
    int tiles_r;      // tiles along the rays of a beam
    int n_tiles;      // tiles in all
    gptr<float> x, y, z, nx, ny, nz;
    gptr<int> mat;
};

struct RayGroup {
    RayFrameDev f[kRayFramesPerLaunch];
};
static_assert(sizeof(RayGroup) <= 3072, "ray-cast kernel arguments");

__device__ __forceinline__ float4 ld4(gptr<const float4> p) { return gload(p); }

// Node and triangle records read with a wave-uniform index, through scalar
// loads (the constant address space; a scene does not change once uploaded).
template <class T>
using cptr = const __attribute__((address_space(4))) T *;

// A workgroup of NT threads casts a tile of NT rays: 2^br neighbouring rays of
// NT / 2^br neighbouring beams, each wave a patch of 2^wr rays of 2^(6 - wr)
// beams (ray_shape).  The waves of a tile lie side by side along the rays up
// to 32 of them, so that a beam's rays fill whole cache lines of the output.
// Neighbouring tiles meet the same nodes and triangles, so runs of 16 go to one
// XCD, rotated (a beam's tiles divide a round, and its elevations differ in
// cost): 8 x (2048 x 1024) rays on a seabed of 130,242 triangles 517 -> 411 us by
// one traversal per wave, on one of 2 M triangles 1614 -> 1178 us by lanes.
struct RayTile {
    int beams, rays;          // tile size
    int b0, r0;               // its first beam and ray
    int b, r;                 // this thread's, within the tile
};
template <int NT>
__device__ __forceinline__ RayTile ray_tile(const RayFrameDev &f, int block, int tid) {
    RayTile t;
    const int tile = xcd_rotated_id<kRayXcdRun>(block, f.n_tiles);
    const int br = f.br_log2, wr = f.wr_log2;
    t.rays = 1 << br;
    t.beams = NT >> br;
    const int tb = tile / f.tiles_r;
    t.b0 = tb * t.beams;
    t.r0 = (tile - tb * f.tiles_r) << br;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int per_row = br - wr;                       // log2 wave patches along a tile row
    t.r = ((wave & ((1 << per_row) - 1)) << wr) + (lane & ((1 << wr) - 1));
    t.b = ((wave >> per_row) << (6 - wr)) + (lane >> wr);
    return t;
}

// a b + c d + e f and a b - c d, the rounding of each step fixed: which
// product of a sum is fused is the compiler's choice, and rays along a
// triangle's edge would hit or miss it, or one neighbour or the other, by the
// kernel that casts them.
__device__ __forceinline__ float sum3(float a, float b, float c, float d, float e, float f) {
    return __builtin_fmaf(e, f, __builtin_fmaf(a, b, c * d));
}
__device__ __forceinline__ float diff2(float a, float b, float c, float d) {
    return __builtin_fmaf(a, b, -(c * d));
}

// One ray: its directions (sensor and world frame) and slab reciprocals.
struct Ray {
    float s0, s1, s2, d0, d1, d2, i0, i1, i2;
};

// The rays of the tile: one sine and cosine per beam and per ray of the tile,
// shared through LDS (trig holds the beams', then the rays').  Contains a barrier.
template <int NT>
__device__ __forceinline__ Ray ray_of(const RayFrameDev &f, const RayTile &t, int tid, float2 *trig) {
    for (int k = tid; k < t.beams + t.rays; k += NT) {
        const bool beam = k < t.beams;
        const float a = beam ? __builtin_fmaf((float)(t.b0 + k) + 0.5f, f.daz, f.az0)
                             : __builtin_fmaf((float)(t.r0 + k - t.beams) + 0.5f, f.del, f.el0);
        float sn, cs;
        sincosf(a, &sn, &cs);
        trig[k] = make_float2(sn, cs);
    }
    __syncthreads();
    const float2 az = trig[t.b], el = trig[t.beams + t.r];
    const float sa = az.x, ca = az.y, se = el.x, ce = el.y;
    Ray q;
    q.s0 = ce * ca, q.s1 = ce * sa, q.s2 = se;
    q.d0 = sum3(f.R[0], q.s0, f.R[1], q.s1, f.R[2], q.s2);
    q.d1 = sum3(f.R[3], q.s0, f.R[4], q.s1, f.R[5], q.s2);
    q.d2 = sum3(f.R[6], q.s0, f.R[7], q.s1, f.R[8], q.s2);
    // reciprocal direction; a zero component becomes a tiny one of its sign
    // (the box margins make that harmless), keeping the slab products finite
    auto safe = [](float v) { return fabsf(v) > kMinDirComponent ? v : copysignf(kMinDirComponent, v); };
    q.i0 = 1.0f / safe(q.d0), q.i1 = 1.0f / safe(q.d1), q.i2 = 1.0f / safe(q.d2);
    return q;
}

// Entry distance tn of a box and whether the ray meets it before tbest.  The
// slab distances are (plane - origin) / direction, each off by at most about
// two roundings; widening the far end by 1 + 2 gamma_3 (Ize, Robust BVH Ray
// Traversal, JCGT 2013) keeps the test conservative, including for boxes of
// zero thickness.
__device__ __forceinline__ bool slab(const Ray &q, float o0, float o1, float o2, float lx, float ly, float lz,
                                     float hx, float hy, float hz, float tbest, float &tn) {
#pragma clang fp contract(off)
    const float ax = (lx - o0) * q.i0, bx = (hx - o0) * q.i0;
    const float ay = (ly - o1) * q.i1, by = (hy - o1) * q.i1;
    const float az = (lz - o2) * q.i2, bz = (hz - o2) * q.i2;
    tn = fmaxf(fmaxf(fminf(ax, bx), fminf(ay, by)), fmaxf(fminf(az, bz), 0.0f));
    const float tf = fminf(fminf(fmaxf(ax, bx), fmaxf(ay, by)), fminf(fmaxf(az, bz), tbest));
    return tn <= tf * kSlabWiden;
}
// The same with the nearer planes n and the farther f of the ray's direction
// signs given: bit for bit the minima and maxima above, so that a traversal
// that a wave shares visits for each ray what the ray's own would.
__device__ __forceinline__ bool slab_sorted(const Ray &q, float o0, float o1, float o2, float nx, float ny, float nz,
                                            float fx, float fy, float fz, float tbest, float &tn) {
#pragma clang fp contract(off)
    tn = fmaxf(fmaxf((nx - o0) * q.i0, (ny - o1) * q.i1), fmaxf((nz - o2) * q.i2, 0.0f));
    const float tf = fminf(fminf((fx - o0) * q.i0, (fy - o1) * q.i1), fminf((fz - o2) * q.i2, tbest));
    return tn <= tf * kSlabWiden;
}

// Moller-Trumbore: p = d x e2, det = e1 . p; t, and whether the ray meets the
// triangle (edges included) at 0 < t <= tbest.
__device__ __forceinline__ bool triangle(const Ray &q, float o0, float o1, float o2, float4 A, float4 E1, float4 E2,
                                         float tbest, float &t) {
#pragma clang fp contract(off)
    const float d0 = q.d0, d1 = q.d1, d2 = q.d2;
    const float p0 = diff2(d1, E2.z, d2, E2.y);
    const float p1 = diff2(d2, E2.x, d0, E2.z);
    const float p2 = diff2(d0, E2.y, d1, E2.x);
    const float det = sum3(E1.x, p0, E1.y, p1, E1.z, p2);
    const float inv = 1.0f / det;
    const float q0 = o0 - A.x, q1 = o1 - A.y, q2 = o2 - A.z;
    const float u = sum3(q0, p0, q1, p1, q2, p2) * inv;
    const float c0 = diff2(q1, E1.z, q2, E1.y);
    const float c1 = diff2(q2, E1.x, q0, E1.z);
    const float c2 = diff2(q0, E1.y, q1, E1.x);
    const float v = sum3(d0, c0, d1, c1, d2, c2) * inv;
    t = sum3(E2.x, c0, E2.y, c1, E2.z, c2) * inv;
    return det != 0.0f && u >= 0.0f && v >= 0.0f && u + v <= 1.0f && t > 0.0f && t <= tbest;
}

// Whether a ray's own ordered traversal visits triangle slot a before slot b:
// at the deepest node above both, the child with the nearer entry comes
// first; within a leaf, the lower slot.  Used where both lie at exactly the
// same distance, so that the hit does not depend on how rays share a
// traversal.  (A child's triangles are consecutive slots, child 1's from
// split on.)
__device__ bool visited_before(const Ray &q, float o0, float o1, float o2, gptr<const float4> nodes, int root, int a,
                               int b, float t_max) {
    int ref = root;
    while (ref >= 0) {
        const gptr<const float4> nd = nodes + 4LL * ref;
        const int4 rr = gload((gptr<const int4>)(nd + 3));
        const bool a1 = a >= rr.z, b1 = b >= rr.z;
        if (a1 != b1) {
            const float4 v0 = ld4(nd), v1 = ld4(nd + 1), v2 = ld4(nd + 2);
            float t0, t1;
            (void)slab(q, o0, o1, o2, v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, t_max, t0);
            (void)slab(q, o0, o1, o2, v1.z, v1.w, v2.x, v2.y, v2.z, v2.w, t_max, t1);
            return (t1 < t0) == a1;
        }
        ref = a1 ? rr.y : rr.x;
    }
    return a < b;
}

// The return of one ray: the hit point and normal in the sensor frame and the
// material, or a miss.
__device__ __forceinline__ void write_return(const RayFrameDev &f, const Ray &q, gptr<const float4> tris, int k,
                                             int hit, float tbest) {
    float px = 0.0f, py = 0.0f, pz = 0.0f, wx = 0.0f, wy = 0.0f, wz = 0.0f;
    int m = -1;
    if (hit >= 0) {
        const gptr<const float4> tp = tris + 3LL * hit;
        const float4 A = ld4(tp), E1 = ld4(tp + 1), E2 = ld4(tp + 2);
        const float n0 = diff2(E1.y, E2.z, E1.z, E2.y);
        const float n1 = diff2(E1.z, E2.x, E1.x, E2.z);
        const float n2 = diff2(E1.x, E2.y, E1.y, E2.x);
        const float il = 1.0f / sqrtf(sum3(n0, n0, n1, n1, n2, n2));
        const float w0 = n0 * il, w1 = n1 * il, w2 = n2 * il;
        wx = sum3(f.R[0], w0, f.R[3], w1, f.R[6], w2);
        wy = sum3(f.R[1], w0, f.R[4], w1, f.R[7], w2);
        wz = sum3(f.R[2], w0, f.R[5], w1, f.R[8], w2);
        px = tbest * q.s0;
        py = tbest * q.s1;
        pz = tbest * q.s2;
        m = __float_as_int(A.w);
    }
    if (f.x) f.x[k] = px;
    if (f.y) f.y[k] = py;
    if (f.z) f.z[k] = pz;
    if (f.nx) f.nx[k] = wx;
    if (f.ny) f.ny[k] = wy;
    if (f.nz) f.nz[k] = wz;
    f.mat[k] = m;
}

template <int NT>
__global__ __launch_bounds__(NT) void k_raycast(RayGroup g, gptr<const float4> nodes, gptr<const float4> tris,
                                                int root, int empty) {
    extern __shared__ int stk[];   // [depth of the scene][NT]: a deferred child per level at most
    __shared__ float2 trig[NT + 1];
    const RayFrameDev &f = g.f[blockIdx.y];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= f.n_tiles) return;
    const RayTile tl = ray_tile<NT>(f, blockIdx.x, tid);
    const Ray q = ray_of<NT>(f, tl, tid, trig);
    const int b = tl.b0 + tl.b, r = tl.r0 + tl.r;
    if (b >= f.nb || r >= f.nr) return;
    const float o0 = f.o[0], o1 = f.o[1], o2 = f.o[2];
    float tbest = f.t_max;
    int hit = -1;
    int ref = root;
    int sp = 0;
    if (!empty) {
        while (true) {
            if (ref >= 0) {
                const gptr<const float4> nd = nodes + 4LL * ref;
                const float4 a = ld4(nd), bq = ld4(nd + 1), c = ld4(nd + 2);
                const int4 rr = gload((gptr<const int4>)(nd + 3));
                float t0, t1;
                const bool h0 = slab(q, o0, o1, o2, a.x, a.y, a.z, a.w, bq.x, bq.y, tbest, t0);
                const bool h1 = slab(q, o0, o1, o2, bq.z, bq.w, c.x, c.y, c.z, c.w, tbest, t1);
                if (h0 && h1) {
                    const bool swap = t1 < t0;
                    ref = swap ? rr.y : rr.x;
                    stk[sp * NT + tid] = swap ? rr.x : rr.y;
                    ++sp;
                    continue;
                }
                if (h0 || h1) {
                    ref = h0 ? rr.x : rr.y;
                    continue;
                }
            } else {
                const int code = ~ref;
                const int first = code >> kLeafShift;
                const int cnt = (code & (kLeafMax - 1)) + 1;
                for (int i = 0; i < cnt; ++i) {
                    const gptr<const float4> tp = tris + 3LL * (first + i);
                    float t;
                    if (triangle(q, o0, o1, o2, ld4(tp), ld4(tp + 1), ld4(tp + 2), tbest, t) &&
                        (hit < 0 || t < tbest)) {
                        tbest = t;
                        hit = first + i;
                    }
                }
            }
            if (sp == 0) break;
            --sp;
            ref = stk[sp * NT + tid];
        }
    }
    write_return(f, q, tris, b * f.nr + r, hit, tbest);
}

// Lane `at` of v (uniform) set to the uniform value x.
__device__ __forceinline__ void set_lane(int &v, int x, int at) {
    asm("s_mov_b32 m0, %2\n\tv_writelane_b32 %0, %1, m0" : "+v"(v) : "s"(x), "s"(at) : "m0");
}

typedef int i32x16_t __attribute__((ext_vector_type(16)));

// The wave's traversal: hit and tbest of each live lane's ray.  OCT 0 to 7:
// the rays' directions have these signs (bit a: negative along axis a), so
// near and far planes are known when compiling; 8: the signs differ.  (One
// traversal that picks the planes by scalar selects spends two scalar
// instructions a plane, and the scalar unit, which issues no faster than the
// vector unit, was then the bound: 25 more of them a node.)
template <int OCT>
__device__ __forceinline__ void packet_traverse(const Ray &q, float o0, float o1, float o2, float t_max,
                                                gptr<const float4> nodes, gptr<const float4> tris, int root,
                                                unsigned long long live_m, float &tbest, int &hit) {
    constexpr bool X = (OCT & 1) != 0, Y = (OCT & 2) != 0, Z = (OCT & 4) != 0;
    const cptr<char> cn = (cptr<char>)(uintptr_t)nodes;
    const cptr<char> ct = (cptr<char>)(uintptr_t)tris;
    int ref = root;                    // uniform
    unsigned long long m = live_m;     // lanes that met the current box
    int sp = 0;
    int s_ref = 0, s_lo = 0, s_hi = 0;   // stack entry e in lane e: reference and lanes
    auto push = [&](int r, unsigned long long mo) __attribute__((always_inline)) {
        set_lane(s_ref, r, sp);
        set_lane(s_lo, (int)(unsigned)mo, sp);
        set_lane(s_hi, (int)(unsigned)(mo >> 32), sp);
        ++sp;
    };
    while (true) {
        if (ref >= 0) {
            const i32x16_t nd = *(cptr<i32x16_t>)(cn + ((uint32_t)ref << 6));   // below 2^32 (kPacketNodes)
            auto pl = [&](int k) __attribute__((always_inline)) { return __int_as_float(nd[k]); };
            float t0, t1;
            bool h0, h1;
            if (OCT < 8) {
                h0 = slab_sorted(q, o0, o1, o2, pl(X ? 3 : 0), pl(Y ? 4 : 1), pl(Z ? 5 : 2), pl(X ? 0 : 3),
                                 pl(Y ? 1 : 4), pl(Z ? 2 : 5), tbest, t0);
                h1 = slab_sorted(q, o0, o1, o2, pl(X ? 9 : 6), pl(Y ? 10 : 7), pl(Z ? 11 : 8), pl(X ? 6 : 9),
                                 pl(Y ? 7 : 10), pl(Z ? 8 : 11), tbest, t1);
            } else {
                h0 = slab(q, o0, o1, o2, pl(0), pl(1), pl(2), pl(3), pl(4), pl(5), tbest, t0);
                h1 = slab(q, o0, o1, o2, pl(6), pl(7), pl(8), pl(9), pl(10), pl(11), tbest, t1);
            }
            const unsigned long long m0 = __ballot(h0) & m, m1 = __ballot(h1) & m;
            const int c0 = __popcll(m0), c1 = __popcll(m1);   // compared as integers: scalar branches
            if (c0 != 0) {
                if (c1 != 0) {
                    // first the child that is nearer for most of the lanes that meet both
                    const unsigned long long both = m0 & m1;
                    if (2 * __popcll(__ballot(t1 < t0) & both) > __popcll(both)) {
                        push(nd[12], m0);
                        ref = nd[13];
                        m = m1;
                    } else {
                        push(nd[13], m1);
                        ref = nd[12];
                        m = m0;
                    }
                } else {
                    ref = nd[12];
                    m = m0;
                }
                continue;
            }
            if (c1 != 0) {
                ref = nd[13];
                m = m1;
                continue;
            }
        } else {
            const int code = ~ref;
            const int first = code >> kLeafShift;
            const int cnt = (code & (kLeafMax - 1)) + 1;
            for (int i = 0; i < cnt; ++i) {
                const cptr<f32x4_t> tp = (cptr<f32x4_t>)(ct + (uint32_t)(first + i) * (uint32_t)sizeof(BvhTri));
                const f32x4_t A = tp[0], E1 = tp[1], E2 = tp[2];
                float t;
                const bool met = triangle(q, o0, o1, o2, make_float4(A.x, A.y, A.z, A.w),
                                          make_float4(E1.x, E1.y, E1.z, 0.0f), make_float4(E2.x, E2.y, E2.z, 0.0f),
                                          tbest, t);
                const unsigned long long mm = __ballot(met) & m;
                if (mm == 0ull) continue;
                if (__builtin_amdgcn_inverse_ballot_w64(mm)) {
                    if (hit < 0 || t < tbest || visited_before(q, o0, o1, o2, nodes, root, first + i, hit, t_max)) {
                        tbest = t;
                        hit = first + i;
                    }
                }
            }
        }
        if (sp == 0) break;
        --sp;
        ref = __builtin_amdgcn_readlane(s_ref, sp);
        m = (unsigned long long)(unsigned)__builtin_amdgcn_readlane(s_lo, sp) |
            (unsigned long long)(unsigned)__builtin_amdgcn_readlane(s_hi, sp) << 32;
    }
}

// One traversal per wave.  Bound by instruction issue, vector and scalar in
// about equal parts (a node is about 42 vector instructions, the cheap kind
// mostly, against 66 for a lane of its own, and 25 scalar ones); no vector loads, the
// stack's entries live in the lanes of three registers.  8 x (2048 x 1024)
// rays on a seabed of 130,242 triangles: 985 us with a traversal per lane over
// 64 rays of one beam, 640 us with one per wave over 8 x 8 patches and planes
// picked by scalar selects, 476 us with the octants, 411 us with runs of tiles per
// XCD (41 G rays/s).
__global__ __launch_bounds__(kRayThreads) void k_raycast_packet(RayGroup g, gptr<const float4> nodes,
                                                                gptr<const float4> tris, int root, int empty) {
    static_assert(kBvhMaxDepth <= kWave, "a stack entry per lane");
    __shared__ float2 trig[kRayThreads + 1];
    const RayFrameDev &f = g.f[blockIdx.y];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= f.n_tiles) return;
    const RayTile tl = ray_tile<kRayThreads>(f, blockIdx.x, tid);
    const Ray q = ray_of<kRayThreads>(f, tl, tid, trig);
    const int b = tl.b0 + tl.b, r = tl.r0 + tl.r;
    const bool live = b < f.nb && r < f.nr;
    const unsigned long long live_m = __ballot(live);
    if (live_m == 0ull) return;
    const float o0 = f.o[0], o1 = f.o[1], o2 = f.o[2];
    float tbest = f.t_max;
    int hit = -1;
    if (!empty) {
        const unsigned long long n0 = __ballot(q.i0 < 0.0f) & live_m, n1 = __ballot(q.i1 < 0.0f) & live_m,
                                 n2 = __ballot(q.i2 < 0.0f) & live_m;
        int oct = 8;
        if ((n0 == 0ull || n0 == live_m) && (n1 == 0ull || n1 == live_m) && (n2 == 0ull || n2 == live_m))
            oct = (n0 ? 1 : 0) | (n1 ? 2 : 0) | (n2 ? 4 : 0);
        switch (oct) {
#define OSIM_OCT(O) \
    case O: packet_traverse<O>(q, o0, o1, o2, f.t_max, nodes, tris, root, live_m, tbest, hit); break
            OSIM_OCT(0);
            OSIM_OCT(1);
            OSIM_OCT(2);
            OSIM_OCT(3);
            OSIM_OCT(4);
            OSIM_OCT(5);
            OSIM_OCT(6);
            OSIM_OCT(7);
            default: packet_traverse<8>(q, o0, o1, o2, f.t_max, nodes, tris, root, live_m, tbest, hit);
#undef OSIM_OCT
        }
    }
    if (live) write_return(f, q, tris, b * f.nr + r, hit, tbest);
}

int ceil_log2(int v) {
    int e = 0;
    while (e < 30 && (1 << e) < v) ++e;
    return e;
}

// The wave's patch: 2^wr rays of 2^(6 - wr) beams, no more rays or beams than
// the pattern has.  Its angular height is about half its width (elevation
// steps are stretched on the ground by the grazing incidence), so that its rays
// meet nearly the same nodes: on a seabed, 64 rays of one beam step through a
// third more.  With `line` it is such a line of 64 rays all the same: over
// triangles smaller than the rays' spacing nothing is shared, and a square
// patch only puts the costly rays into few waves.
// The tile of 2^threads_log2 rays: waves along the rays up to 32 rays, the rest
// along the beams, again within the pattern.
void ray_shape(int n_beams, int n_rays, float daz, float del, bool line, int threads_log2, int &wr, int &br) {
    const int nb2 = ceil_log2(n_beams), nr2 = ceil_log2(n_rays);
    wr = line ? 6 : 3;
    if (!line && daz > 0.0f && del > 0.0f)
        wr = (int)std::lround(0.5 * (5.0 + std::log2((double)daz / (double)del)));
    wr = std::min(std::max(wr, 0), 6);
    wr = std::max(std::min(wr, nr2), std::min(6, 6 - nb2));   // few rays, then few beams
    br = wr;
    while (br < wr + threads_log2 - 6 && br < nr2 && (br < 5 || threads_log2 - br > nb2)) ++br;
}

// Triangles in a wave's patch, roughly: its footprint half way to what the
// cast can reach (or where the scene begins), across the ray, over the area
// that a quarter of the triangles do not exceed: rather too many than too few
// where a dense object stands on a coarse floor.
double patch_triangles(const oceansim_scene &s, const oceansim_ray_frame &q, float daz, float del) {
    if (s.empty) return 0.0;
    double near2 = 0.0, far2 = 0.0;
    for (int a = 0; a < 3; ++a) {
        const double below = s.lo[a] - (double)q.pos[a], above = (double)q.pos[a] - s.hi[a];
        const double n = std::max({below, above, 0.0});
        const double f = std::max(std::fabs(below), std::fabs(above));
        near2 += n * n;
        far2 += f * f;
    }
    const double r = std::max(std::sqrt(near2), 0.5 * std::min((double)q.t_max, std::sqrt(far2)));
    return (double)kWave * daz * del * r * r / s.tri_area;
}

// Which traversal.  One per wave pays where its patch is narrow (64 daz del, in
// steradians, within 5e-4), holds few triangles and the launch fills the
// chip (2^18 rays: 4 waves a SIMD): its steps are cheaper but more, since a wave
// visits what any of its rays meets, and in a small launch only their number
// counts.  Seabed of 130,242 triangles, t_max 50, one traversal per wave
// against one per lane: 9 x (2048 x 256) rays 162 / 304 us, 1 x (2048 x 256)
// 34 / 49, 9 x (2048 x 64) 86 / 111, 4 x (1024 x 128) 54 / 61; but 9 x (1024 x 64),
// 7.6e-4 sr, 78 / 69, and 1 x (1024 x 128) 40 / 33.
// Triangles in a patch, per wave / per lane, over seabeds of 1,250 to 8 M
// triangles: 0.7 (1 x (2048 x 256) rays) 38 / 52 us, 0.75 (8 x (2048 x 1024)) 1108 /
// 1609, 1.5 (1 x (512 x 512)) 37 / 32, 2.0 (9 x (2048 x 256)) 344 / 430, 2.2 (16 x (512
// x 512)) 124 / 130, 3 (4 x (1024 x 128)) 103 / 67, 12 (the same) 228 / 82; over a
// hull of 320,000 triangles on a floor of two 558 / 223.  Inside a closed tank,
// where no ray grazes a wall, one per wave would pay up to 20 of them and more
// (165 / 298 us at 5): the scene's numbers do not tell it from the others.
// Lanes take lines instead of square patches from six triangles on: square / line
// over the hull 223 / 146 us, before waves took patches 158, and 9 x (1024 x 64)
// rays on 2 M triangles 222 / 178 (182), though 4 x (1024 x 128) there 82 / 101 (98).
// kPacketNodes: the packet's 32-bit offsets into the node and triangle arrays.
constexpr double kPacketSteradians = 5e-4;
constexpr double kPacketTriangles = 1.25, kPacketTrianglesLarge = 2.5;   // below and from kPacketLargeRays on
constexpr double kSquareTriangles = 6.0;
constexpr long long kPacketRays = 1LL << 18, kPacketLargeRays = 1LL << 20;
constexpr long long kPacketNodes = 1LL << 26;

bool finite_all(const float *v, int n) {
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(v[i])) return false;
    return true;
}

bool aligned4(const void *p) { return ((uintptr_t)p & 3u) == 0; }

}  // namespace
}  // namespace osim

using namespace osim;
using host::fail;
using host::hip_fail;
using host::ok;

extern "C" {

int oceansim_scene_create(const float *vertices, int64_t n_vertices, const int32_t *triangles,
                          const int32_t *tri_mat, int64_t n_triangles, oceansim_scene **scene) {
    if (!scene) return fail(OCEANSIM_E_INVALID_ARG, "scene is NULL");
    *scene = nullptr;
    BvhBuild B;
    int rc = build_bvh(vertices, n_vertices, triangles, tri_mat, n_triangles, B);
    if (rc != OCEANSIM_OK) return rc;
    oceansim_scene *s = new (std::nothrow) oceansim_scene();
    if (!s) {
        free_bvh(B);
        return fail(OCEANSIM_E_HIP, "host memory for the scene");
    }
    hipError_t e = hipGetDevice(&s->device);
    s->root = B.root;
    s->empty = B.empty ? 1 : 0;
    s->info = B.info;
    s->tri_area = B.tri_area;
    for (int a = 0; a < 3; ++a) {
        s->lo[a] = B.lo[a];
        s->hi[a] = B.hi[a];
    }
    if (e == hipSuccess && !B.empty) {
        e = hipMalloc((void **)&s->nodes, sizeof(BvhNode) * (size_t)std::max(1LL, B.n_nodes));
        if (e == hipSuccess) e = hipMalloc((void **)&s->tris, sizeof(BvhTri) * (size_t)B.n_tris);
        if (e == hipSuccess && B.n_nodes)
            e = hipMemcpy(s->nodes, B.nodes, sizeof(BvhNode) * (size_t)B.n_nodes, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(s->tris, B.tris, sizeof(BvhTri) * (size_t)B.n_tris, hipMemcpyHostToDevice);
    }
    free_bvh(B);
    if (e != hipSuccess) {
        if (s->nodes) (void)hipFree(s->nodes);
        if (s->tris) (void)hipFree(s->tris);
        delete s;
        return hip_fail(e, "scene upload");
    }
    *scene = s;
    return ok();
}

int oceansim_scene_measure(const float *vertices, int64_t n_vertices, const int32_t *triangles,
                           const int32_t *tri_mat, int64_t n_triangles, oceansim_scene_info *info) {
    if (!info) return fail(OCEANSIM_E_INVALID_ARG, "info is NULL");
    BvhBuild B;
    const int rc = build_bvh(vertices, n_vertices, triangles, tri_mat, n_triangles, B);
    if (rc == OCEANSIM_OK) *info = B.info;
    free_bvh(B);
    return rc;
}

int oceansim_scene_get_info(const oceansim_scene *scene, oceansim_scene_info *info) {
    if (!scene || !info) return fail(OCEANSIM_E_INVALID_ARG, "scene or info is NULL");
    *info = scene->info;
    return ok();
}

int oceansim_scene_destroy(oceansim_scene *scene) {
    if (!scene) return ok();
    hipError_t e = hipSuccess;
    if (scene->nodes || scene->tris) {
        int cur = 0;
        e = hipGetDevice(&cur);
        if (e == hipSuccess && cur != scene->device) e = hipSetDevice(scene->device);
        if (e == hipSuccess) e = hipDeviceSynchronize();
        if (scene->nodes) (void)hipFree(scene->nodes);
        if (scene->tris) (void)hipFree(scene->tris);
        if (cur != scene->device) (void)hipSetDevice(cur);
    }
    delete scene;
    return e == hipSuccess ? ok() : hip_fail(e, "scene destroy");
}

int oceansim_raycast(const oceansim_scene *scene, const oceansim_ray_frame *frames, int32_t n_frames,
                     void *stream) {
    if (!scene) return fail(OCEANSIM_E_INVALID_ARG, "scene is NULL");
    if (n_frames < 0) return fail(OCEANSIM_E_SHAPE, "n_frames < 0");
    if (n_frames == 0) return ok();
    if (!frames) return fail(OCEANSIM_E_INVALID_ARG, "frames is NULL");
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev != scene->device)
        return fail(OCEANSIM_E_INVALID_ARG, "the scene lives on device %d, the current device is %d", scene->device,
                    dev);
    std::vector<RayFrameDev> fd;
    std::vector<double> dense;   // triangles in a patch
    fd.reserve((size_t)n_frames);
    dense.reserve((size_t)n_frames);
    for (int i = 0; i < n_frames; ++i) {
        const oceansim_ray_frame &q = frames[i];
        if (q.n_beams < 0 || q.n_rays < 0) return fail(OCEANSIM_E_SHAPE, "frame %d: negative beam or ray count", i);
        const long long n = (long long)q.n_beams * q.n_rays;
        if (n > 0x7fffffffLL) return fail(OCEANSIM_E_UNSUPPORTED, "frame %d: more than 2^31 - 1 rays", i);
        if (!(q.fov_az >= 0.0f && q.fov_az <= 6.2831855f))
            return fail(OCEANSIM_E_INVALID_ARG, "frame %d: fov_az must be in [0, 2pi]", i);
        if (!(q.fov_el >= 0.0f && q.fov_el < 3.1415927f))
            return fail(OCEANSIM_E_INVALID_ARG, "frame %d: fov_el must be in [0, pi)", i);
        if (!(q.t_max > 0.0f && std::isfinite(q.t_max)))
            return fail(OCEANSIM_E_INVALID_ARG, "frame %d: t_max must be finite and > 0", i);
        if (!finite_all(q.pos, 3) || !finite_all(q.rot, 9))
            return fail(OCEANSIM_E_INVALID_ARG, "frame %d: non-finite pose", i);
        for (int a = 0; a < 3; ++a)
            if (std::fabs(q.pos[a]) > kMaxCoord)
                return fail(OCEANSIM_E_UNSUPPORTED, "frame %d: sensor position beyond 2^40", i);
        if (n == 0) continue;
        if (!q.mat) return fail(OCEANSIM_E_INVALID_ARG, "frame %d: mat is NULL", i);
        const void *outs[7] = {q.x, q.y, q.z, q.nx, q.ny, q.nz, q.mat};
        for (auto p : outs)
            if (!aligned4(p)) return fail(OCEANSIM_E_INVALID_ARG, "frame %d: misaligned output", i);
        RayFrameDev d;
        for (int a = 0; a < 3; ++a) d.o[a] = q.pos[a];
        for (int a = 0; a < 9; ++a) d.R[a] = q.rot[a];
        d.az0 = -0.5f * q.fov_az;
        d.daz = (float)((double)q.fov_az / q.n_beams);
        d.el0 = -0.5f * q.fov_el;
        d.del = (float)((double)q.fov_el / q.n_rays);
        d.t_max = q.t_max;
        d.nb = q.n_beams;
        d.nr = q.n_rays;
        d.x = gcast(q.x);
        d.y = gcast(q.y);
        d.z = gcast(q.z);
        d.nx = gcast(q.nx);
        d.ny = gcast(q.ny);
        d.nz = gcast(q.nz);
        d.mat = gcast(q.mat);
        fd.push_back(d);
        dense.push_back(patch_triangles(*scene, q, d.daz, d.del));
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const gptr<const float4> nodes = gcast(reinterpret_cast<const float4 *>(scene->nodes));
    const gptr<const float4> tris = gcast(reinterpret_cast<const float4 *>(scene->tris));
    for (size_t g0 = 0; g0 < fd.size(); g0 += kRayFramesPerLaunch) {
        RayGroup grp;
        std::memset(&grp, 0, sizeof grp);
        const int cnt = (int)std::min<size_t>(kRayFramesPerLaunch, fd.size() - g0);
        long long rays = 0;
        bool packet = scene->info.n_triangles < kPacketNodes;   // more triangles than nodes
        double most = 0.0;   // triangles in a patch
        for (int j = 0; j < cnt; ++j) {
            const RayFrameDev &d = fd[g0 + j];
            rays += (long long)d.nb * d.nr;
            packet = packet && (double)kWave * d.daz * d.del <= kPacketSteradians;
            most = std::max(most, dense[g0 + j]);
        }
        packet = packet && rays >= kPacketRays &&
                 most <= (rays >= kPacketLargeRays ? kPacketTrianglesLarge : kPacketTriangles);
        const bool line = most > kSquareTriangles;
        const int nt = line ? kRayLineThreads : kRayThreads;
        int tiles = 0;
        for (int j = 0; j < cnt; ++j) {
            RayFrameDev &d = grp.f[j] = fd[g0 + j];
            ray_shape(d.nb, d.nr, d.daz, d.del, line, ceil_log2(nt), d.wr_log2, d.br_log2);
            const int beams = nt >> d.br_log2;
            const long long tr = ((long long)d.nr + (1 << d.br_log2) - 1) >> d.br_log2;
            const long long tb = ((long long)d.nb + beams - 1) / beams;
            d.tiles_r = (int)tr;
            d.n_tiles = (int)(tr * tb);   // padded to less than twice the rays where these near 2^31: a valid grid
            tiles = std::max(tiles, d.n_tiles);
        }
        const dim3 grid((unsigned)tiles, (unsigned)cnt);
        const size_t stack = (size_t)std::max(1, scene->info.depth) * nt * sizeof(int);
        if (packet)
            OSIM_LAUNCH("k_raycast", k_raycast_packet, grid, dim3(kRayThreads), 0, st, grp, nodes, tris, scene->root,
                        scene->empty);
        else if (line)
            OSIM_LAUNCH("k_raycast", k_raycast<kRayLineThreads>, grid, dim3(kRayLineThreads), stack, st, grp, nodes,
                        tris, scene->root, scene->empty);
        else
            OSIM_LAUNCH("k_raycast", k_raycast<kRayThreads>, grid, dim3(kRayThreads), stack, st, grp, nodes, tris,
                        scene->root, scene->empty);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "ray-cast launch");
    }
    return ok();
}

}  // extern "C"
