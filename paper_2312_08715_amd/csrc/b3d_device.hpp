// Device-side building blocks shared by the gfx950 kernels: camera and pose
// helpers, packed depth/id keys, the cluster-based triangle rasteriser that
// fills an LDS depth buffer, and fixed-order block reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace b3d {

constexpr int kBlock = 256;          // threads per workgroup (4 wave64)
constexpr int kWaves = kBlock / 64;
constexpr int kCUs = 256;            // compute units of an MI355X
constexpr size_t kLdsPerCU = 160 * 1024;
constexpr int kClusterPrims = 64;    // max primitives (triangles or quads) per cluster, one per lane of a wave
constexpr uint32_t kNoTri = 0xFFFFFFFFu;  // second id of a primitive that is a single triangle
// The key of a pixel with no surface: depth 1e15 m (bits 0x58635FA9), id all
// ones.  It compares above every surface nearer than that, and its depth is
// finite, so a window term against an empty slot evaluates to exactly 0
// (exp of minus a huge distance) without a test, provided rays stay within
// |x/z|, |y/z| <= 1e3 (checked when a scene is created).
constexpr unsigned long long kEmptyKey = (0x58635FA9ull << 32) | 0xFFFFFFFFull;

// A workgroup barrier that orders LDS only: global loads and stores stay in
// flight across it, where __syncthreads would first wait for all of them.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Pinhole camera and image size.
struct Cam {
  float fx, fy, cx, cy, znear;
  int H, W;
};

// Row-major rotation and translation of an object-to-camera pose.
struct Pose {
  float r[9];
  float t[3];
};

// A group of up to kClusterPrims primitives of one orientation class that
// are close in space: primitives [pfirst, pfirst + np).  A primitive is the
// triangle (a, b, c) and, when its second id is not kNoTri, the triangle
// (a, c, d) sharing the edge a-c (a convex planar quad).  sphere = centre and
// radius of a ball holding them; cone = unit axis of a cone holding their face
// normals and the sine of its half-angle plus a margin (above 1: no bound).
// `alike` clusters hold parallelograms a, a + ab, a + ab + ad, a + ad that
// share their edge vectors up to the rounding of the vertices: the faces of
// equal voxels.  ab.w is how far from one of their corners that puts it at most.
struct ClusterDev {
  int pfirst, np, alike, pad;
  float4 sphere;
  float4 cone;
  float4 ab, ad;  // alike: the edge vectors b - a and d - a
};

// Device view of an uploaded mesh.
struct MeshDev {
  const ClusterDev* clusters;  // [0, n_visible) drawn; [n_visible, n_clusters) only near the near plane
  const float4* pverts;        // [primitives][4] object-frame corners a, b, c, d (d = c for a triangle)
  const float4* pfirsts;       // [primitives] corner a alone (all that an alike cluster's primitives need)
  const uint2* pids;           // [primitives] caller's ids of triangles (a, b, c) and (a, c, d) or kNoTri
  const float4* verts;         // caller's vertices
  const int4* tris;            // caller's triangles (w unused)
  const float4* normals;       // object-frame (v1 - v0) x (v2 - v0)
  const double4* planes;       // the same in double, and its product with v0
  int n_clusters, n_visible;
  int has_big;                 // some primitive spans over 1/8 of the bounds' diagonal (table tops, walls)
  int T;                       // triangles
  float sphere[4];             // bounding sphere centre and radius
  float lo[3], hi[3];          // axis-aligned bounds
};

__device__ __forceinline__ Pose load_pose(const float* __restrict__ p) {
  Pose P;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    P.r[3 * i + 0] = p[4 * i + 0];
    P.r[3 * i + 1] = p[4 * i + 1];
    P.r[3 * i + 2] = p[4 * i + 2];
    P.t[i] = p[4 * i + 3];
  }
  return P;
}

__device__ __forceinline__ float3 xform(const Pose& P, float x, float y, float z) {
  return make_float3(P.r[0] * x + P.r[1] * y + P.r[2] * z + P.t[0], P.r[3] * x + P.r[4] * y + P.r[5] * z + P.t[1],
                     P.r[6] * x + P.r[7] * y + P.r[8] * z + P.t[2]);
}

__device__ __forceinline__ float3 rotate(const Pose& P, float x, float y, float z) {
  return make_float3(P.r[0] * x + P.r[1] * y + P.r[2] * z, P.r[3] * x + P.r[4] * y + P.r[5] * z,
                     P.r[6] * x + P.r[7] * y + P.r[8] * z);
}

// Ray direction components of pixel column c / row r (the z component is 1).
// Correctly rounded division, so every kernel gets bit-identical rays.
__device__ __forceinline__ float ray_x(const Cam& cam, int c) { return ((float)c + 0.5f - cam.cx) / cam.fx; }
__device__ __forceinline__ float ray_y(const Cam& cam, int r) { return ((float)r + 0.5f - cam.cy) / cam.fy; }

// Packed depth/id key: positive float bits are monotone, so the smallest key
// is the nearest surface and, at equal depth, the smallest triangle id.
__device__ __forceinline__ unsigned long long pack_key(float z, uint32_t id) {
  return ((unsigned long long)__float_as_uint(z) << 32) | (unsigned long long)id;
}
__device__ __forceinline__ float key_depth(unsigned long long k) { return __uint_as_float((uint32_t)(k >> 32)); }
__device__ __forceinline__ uint32_t key_id(unsigned long long k) { return (uint32_t)(k & 0xffffffffull); }

// Integer rectangle [x0, x1) x [y0, y1).
struct Rect {
  int x0, x1, y0, y1;
  __device__ __forceinline__ int w() const { return x1 - x0; }
  __device__ __forceinline__ int h() const { return y1 - y0; }
  __device__ __forceinline__ bool empty() const { return x1 <= x0 || y1 <= y0; }
};

__device__ __forceinline__ Rect grow(const Rect& r, int m) {
  Rect o;
  o.x0 = r.x0 - m;
  o.x1 = r.x1 + m;
  o.y0 = r.y0 - m;
  o.y1 = r.y1 + m;
  return o;
}

__device__ __forceinline__ Rect grow_clip(const Rect& r, int m, int W, int H) {
  Rect o;
  o.x0 = max(r.x0 - m, 0);
  o.x1 = min(r.x1 + m, W);
  o.y0 = max(r.y0 - m, 0);
  o.y1 = min(r.y1 + m, H);
  return o;
}

// Minimum and maximum of v over the lanes of each group of eight, in all of them.
template <int CTRL>
__device__ __forceinline__ float lane_swap(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float min8(float v) {
  v = fminf(v, lane_swap<0xB1>(v));     // lanes 1 apart
  v = fminf(v, lane_swap<0x4E>(v));     // lanes 2 apart
  return fminf(v, lane_swap<0x141>(v));  // the other quad of the eight
}
__device__ __forceinline__ float max8(float v) {
  v = fmaxf(v, lane_swap<0xB1>(v));
  v = fmaxf(v, lane_swap<0x4E>(v));
  return fmaxf(v, lane_swap<0x141>(v));
}

// Range of x/z over a sphere (centre c, radius r) in front of the camera:
// the planes x = k z through the camera that touch the sphere have
// (c_x - k c_z)^2 = r^2 (1 + k^2), i.e.
// k = (c_x c_z -+ r sqrt(c_x^2 + c_z^2 - r^2)) / (c_z^2 - r^2).
__device__ __forceinline__ void sphere_slopes(float cx, float cz, float r, float& k0, float& k1) {
  const float iden = __builtin_amdgcn_rcpf(cz * cz - r * r);
  const float root = r * __builtin_amdgcn_sqrtf(fmaxf(cx * cx + cz * cz - r * r, 0.0f));
  k0 = (cx * cz - root) * iden;
  k1 = (cx * cz + root) * iden;
}

// Conservative pixel rectangle of the object under pose P: the projection of
// the mesh's posed bounding box intersected with the exact projection bounds
// of its bounding sphere (slightly enlarged against rounding), widened by one
// pixel, clipped to the image.  The whole image when neither bound applies
// (the box reaches the near plane and the sphere reaches the camera plane).
// Every wave computes it with all lanes, eight of them sharing the box's
// corners; the result is uniform.
__device__ __forceinline__ Rect object_rect(const MeshDev& m, const Pose& P, const Cam& cam) {
  const int k8 = threadIdx.x & 7;
  const float3 q = xform(P, (k8 & 1) ? m.hi[0] : m.lo[0], (k8 & 2) ? m.hi[1] : m.lo[1], (k8 & 4) ? m.hi[2] : m.lo[2]);
  const bool aok = __ballot(!(q.z > cam.znear)) == 0ull;
  const float iz = __builtin_amdgcn_rcpf(q.z);
  const float u = cam.fx * q.x * iz + cam.cx, v = cam.fy * q.y * iz + cam.cy;
  const float a[4] = {min8(u), max8(u), min8(v), max8(v)};
  const float3 c = xform(P, m.sphere[0], m.sphere[1], m.sphere[2]);
  const float rad = m.sphere[3] * 1.0001f + 1e-6f;
  const bool sok = c.z - rad > cam.znear;
  Rect r;
  if (!aok && !sok) {
    r.x0 = 0;
    r.x1 = cam.W;
    r.y0 = 0;
    r.y1 = cam.H;
    return r;
  }
  float b[4];
  if (sok) {
    float k0, k1;
    sphere_slopes(c.x, c.z, rad, k0, k1);
    b[0] = cam.fx * k0 + cam.cx - 0.01f;
    b[1] = cam.fx * k1 + cam.cx + 0.01f;
    sphere_slopes(c.y, c.z, rad, k0, k1);
    b[2] = cam.fy * k0 + cam.cy - 0.01f;
    b[3] = cam.fy * k1 + cam.cy + 0.01f;
    if (aok) {
      b[0] = fmaxf(a[0], b[0]);
      b[1] = fminf(a[1], b[1]);
      b[2] = fmaxf(a[2], b[2]);
      b[3] = fminf(a[3], b[3]);
    }
  } else {
    for (int k = 0; k < 4; ++k) b[k] = a[k];
  }
  // pixel centres c + 1/2 in [umin, umax], widened by one pixel each side
  const float fx0 = fmaxf(ceilf(b[0] - 0.5f) - 1.0f, 0.0f);
  const float fx1 = fminf(floorf(b[1] - 0.5f) + 2.0f, (float)cam.W);
  const float fy0 = fmaxf(ceilf(b[2] - 0.5f) - 1.0f, 0.0f);
  const float fy1 = fminf(floorf(b[3] - 0.5f) + 2.0f, (float)cam.H);
  r.x0 = __builtin_amdgcn_readfirstlane((int)fminf(fx0, (float)cam.W));
  r.x1 = __builtin_amdgcn_readfirstlane((int)fmaxf(fx1, fx0));
  r.y0 = __builtin_amdgcn_readfirstlane((int)fminf(fy0, (float)cam.H));
  r.y1 = __builtin_amdgcn_readfirstlane((int)fmaxf(fy1, fy0));
  if (r.x1 > cam.W) r.x1 = cam.W;
  if (r.y1 > cam.H) r.y1 = cam.H;
  return r;
}

// What the plane depth of a pixel needs of a pose and a camera, in double:
// the cofactors of R (normals turn with them, whatever R's rounding), det R,
// t, and the reciprocal focal lengths.  The kernels that rasterise keep it in
// LDS (kPlaneViewBytes): 34 registers less across the rasteriser.
struct PlaneView {
  double c[9], det, t[3], ifx, ify, cx, cy;
};
constexpr size_t kPlaneViewBytes = sizeof(PlaneView);

__device__ __forceinline__ PlaneView plane_view(const Pose& P, const Cam& cam) {
  PlaneView v;
  const double r[9] = {P.r[0], P.r[1], P.r[2], P.r[3], P.r[4], P.r[5], P.r[6], P.r[7], P.r[8]};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double *a = r + 3 * ((i + 1) % 3), *b = r + 3 * ((i + 2) % 3);
    v.c[3 * i] = a[1] * b[2] - a[2] * b[1];
    v.c[3 * i + 1] = a[2] * b[0] - a[0] * b[2];
    v.c[3 * i + 2] = a[0] * b[1] - a[1] * b[0];
    v.t[i] = P.t[i];
  }
  v.det = r[0] * v.c[0] + r[1] * v.c[1] + r[2] * v.c[2];
  v.ifx = 1.0 / (double)cam.fx;
  v.ify = 1.0 / (double)cam.fy;
  v.cx = (double)cam.cx - 0.5;
  v.cy = (double)cam.cy - 0.5;
  return v;
}

// Depth of pixel (r, c) on the plane of triangle `id`: the ray z d meets the
// plane n.(x - c0) = 0 at z = (n.c0)/(n.d), with c_k = R v_k + t and
// n = (c1 - c0) x (c2 - c0) = cof(R) n_o, n.c0 = det(R) n_o.v0 + n.t, all in
// double precision.  The rasteriser's interpolated 1/z decides visibility;
// this value is the depth reported and scored.  (For a triangle seen nearly
// edge-on the depth is ill-conditioned in the vertex coordinates, and single
// precision would put errors of several micrometres into the point and its
// gradient.)  The quotient takes the hardware reciprocal and two Newton steps,
// far below the rounding of the result to single precision.
__device__ __forceinline__ float plane_depth(const MeshDev& m, const PlaneView& v, uint32_t id, int r, int c) {
  const double4 o = m.planes[id];
  const double nx = v.c[0] * o.x + v.c[1] * o.y + v.c[2] * o.z;
  const double ny = v.c[3] * o.x + v.c[4] * o.y + v.c[5] * o.z;
  const double nz = v.c[6] * o.x + v.c[7] * o.y + v.c[8] * o.z;
  const double top = v.det * o.w + nx * v.t[0] + ny * v.t[1] + nz * v.t[2];
  const double den = nx * (((double)c - v.cx) * v.ifx) + ny * (((double)r - v.cy) * v.ify) + nz;
  double y = __builtin_amdgcn_rcp(den);
  y = __builtin_fma(y, __builtin_fma(-den, y, 1.0), y);
  y = __builtin_fma(y, __builtin_fma(-den, y, 1.0), y);
  return (float)(top * y);
}

// Whether a cluster can draw into `band` under pose P: false when its
// sphere lies behind the near plane, when every normal of its cone faces away
// from every point of its sphere, or when the sphere's screen box misses the
// band.  With th the angle between the cone's axis a and the direction to the
// sphere's centre s (at distance d) and ph = asin(r/d) the sphere's angular
// radius, all face away when th + ph + half-angle stays below a right angle:
// cos(th + ph) > sin(half-angle), times d^2.
__device__ __forceinline__ bool cluster_may_draw(const ClusterDev& c, const Pose& P, const Cam& cam,
                                                 const Rect& band) {
  const float3 s = xform(P, c.sphere.x, c.sphere.y, c.sphere.z);
  const float r = c.sphere.w;
  const float znear = s.z - r, zfar = s.z + r;
  if (zfar <= cam.znear) return false;
  const float d2 = s.x * s.x + s.y * s.y + s.z * s.z;
  const float g2 = d2 - r * r;
  if (c.cone.w < 1.0f && g2 > 0.0f) {
    const float3 a = rotate(P, c.cone.x, c.cone.y, c.cone.z);
    const float as = a.x * s.x + a.y * s.y + a.z * s.z;
    if (as * __builtin_amdgcn_sqrtf(g2) - r * __builtin_amdgcn_sqrtf(fmaxf(d2 - as * as, 0.0f)) > c.cone.w * d2)
      return false;
  }
  if (znear > cam.znear) {
    // the box around the sphere, its nearer or farther face whichever bounds
    const float in = __builtin_amdgcn_rcpf(znear), ifr = __builtin_amdgcn_rcpf(zfar);
    const float x0 = s.x - r, x1 = s.x + r, y0 = s.y - r, y1 = s.y + r;
    const float u0 = cam.fx * x0 * (x0 < 0.0f ? in : ifr) + cam.cx, u1 = cam.fx * x1 * (x1 > 0.0f ? in : ifr) + cam.cx;
    const float v0 = cam.fy * y0 * (y0 < 0.0f ? in : ifr) + cam.cy, v1 = cam.fy * y1 * (y1 > 0.0f ? in : ifr) + cam.cy;
    if (u1 < (float)band.x0 - 1.0f || u0 > (float)band.x1 + 1.0f || v1 < (float)band.y0 - 1.0f ||
        v0 > (float)band.y1 + 1.0f)
      return false;
  }
  return true;
}

// Coverage of pixel (r, c) by triangle `id` decided in double precision with
// exactly the operations, in the same order, of the plain definition
// (transform, near-plane drop, back-face test on ((c1-c0)x(c2-c0)).c0,
// projection, edge functions at the pixel centre, inclusive).  Used only for
// pixel centres that single precision cannot place on one side of an edge.
__device__ __forceinline__ bool covered_exact(const MeshDev& m, const Pose& P, const Cam& cam, uint32_t id,
                                                        int r, int col) {
#pragma clang fp contract(off)
  const int4 tr = m.tris[id];
  const float4 v[3] = {m.verts[tr.x], m.verts[tr.y], m.verts[tr.z]};
  double c[3][3];
  for (int k = 0; k < 3; ++k)
    for (int i = 0; i < 3; ++i)
      c[k][i] = (double)P.r[3 * i] * (double)v[k].x + (double)P.r[3 * i + 1] * (double)v[k].y +
                (double)P.r[3 * i + 2] * (double)v[k].z + (double)P.t[i];
  const double zn = (double)cam.znear;
  if (c[0][2] <= zn || c[1][2] <= zn || c[2][2] <= zn) return false;
  const double e1[3] = {c[1][0] - c[0][0], c[1][1] - c[0][1], c[1][2] - c[0][2]};
  const double e2[3] = {c[2][0] - c[0][0], c[2][1] - c[0][1], c[2][2] - c[0][2]};
  const double n0 = e1[1] * e2[2] - e1[2] * e2[1];
  const double n1 = e1[2] * e2[0] - e1[0] * e2[2];
  const double n2 = e1[0] * e2[1] - e1[1] * e2[0];
  const double nc0 = n0 * c[0][0] + n1 * c[0][1] + n2 * c[0][2];
  if (!(nc0 < 0.0)) return false;
  const double fx = cam.fx, fy = cam.fy, cx = cam.cx, cy = cam.cy;
  const double u0 = fx * c[0][0] / c[0][2] + cx, v0 = fy * c[0][1] / c[0][2] + cy;
  const double u1 = fx * c[1][0] / c[1][2] + cx, v1 = fy * c[1][1] / c[1][2] + cy;
  const double u2 = fx * c[2][0] / c[2][2] + cx, v2 = fy * c[2][1] / c[2][2] + cy;
  const double px = col + 0.5, py = r + 0.5;
  const double w0 = (u2 - u1) * (py - v1) - (v2 - v1) * (px - u1);
  const double w1 = (u0 - u2) * (py - v2) - (v0 - v2) * (px - u2);
  const double w2 = (u1 - u0) * (py - v0) - (v1 - v0) * (px - u0);
  return !(w0 > 0.0 || w1 > 0.0 || w2 > 0.0);
}

// How a launch takes part: alone; first, leaving the hypotheses beyond its
// depth buffer; or second, scoring those that were left.
enum Part { kAlone = 0, kFirst = 1, kRest = 2 };

// What a deferred hypothesis leaves in its result for the second launch: a NaN
// that no arithmetic makes (were an input's NaN to carry it here, the
// hypothesis would be taken twice, with one result).
constexpr uint32_t kDeferred = 0x7fcb3d5eu;

// Images above which objects often exceed the 256-thread block's depth buffer,
// and the 512-thread block's (an object takes about a tenth to a quarter of
// its image); hypotheses above which a second launch costs at most a few per cent.
constexpr int kBandedPixels = 24000, kWholeCuPixels = 56000;
constexpr int kBandedCount = 2048;

// LDS scratch of the rasteriser (free again once raster_mesh returns; the
// fused kernel then reuses it for the window weights, which sets its size).
struct RasterLds {
  uint2* queue;  // (band pixel, triangle id) pairs left for the exact test
  int* list;     // drawable clusters of the current group of one per thread
  int* counts;   // [0] queue fill, [1..waves] per-wave drawable counts, [waves + 1] next list entry
  int qcap;
};

// The scratch of a block of BS threads: the queue, the list, the counts.
constexpr int kQueueCap = 1536;
constexpr size_t raster_lds_bytes(int bs) {
  return sizeof(uint2) * kQueueCap + sizeof(int) * bs + sizeof(int) * (bs > 256 ? 32 : 16);
}
constexpr size_t kRasterLdsBytes = raster_lds_bytes(kBlock);

constexpr int kBigCentres = 64;  // a box of more centres than this is walked by the whole wave
constexpr int kBigSlots = 2;     // such boxes a wave takes together per cluster
constexpr int kStageWords = 36;  // words of one staged box
// the staged boxes take the queue's last entries
constexpr int stage_queue_entries(int bs) {
  return (int)((sizeof(float) * (bs / 64) * kBigSlots * kStageWords + 7) / 8);
}
static_assert(stage_queue_entries(1024) < kQueueCap / 2, "staging area too large for the exact-test queue");

template <int BS>
__device__ __forceinline__ RasterLds carve_raster_lds(unsigned char* p) {
  RasterLds r;
  r.queue = reinterpret_cast<uint2*>(p);
  r.list = reinterpret_cast<int*>(r.queue + kQueueCap);
  r.counts = r.list + BS;
  r.qcap = kQueueCap;
  return r;
}

// Staging slots of the large-box walk (only meshes with large primitives use
// them, with the queue shortened by their entries).
template <int BS>
__device__ __forceinline__ float* raster_stage(const RasterLds& r) {
  return reinterpret_cast<float*>(r.queue + (kQueueCap - stage_queue_entries(BS)));
}

// Work counters of the counting instantiation (indices into a per-block
// array): vertices transformed, triangles tested, triangles set up, covered
// pixel centres, window pairs, observed pixels that saw a point, object pixels
// of the adjoint, centres decided by the exact test.
enum { kCntVert = 0, kCntTri, kCntSetup, kCntFrag, kCntPair, kCntObs, kCntAdj, kCntExact, kCntN };

// Pixel position, depth and 1/depth of an object-frame point under pose P.
__device__ __forceinline__ float4 project_corner(const Pose& P, const Cam& cam, const float4 o) {
  const float3 p = xform(P, o.x, o.y, o.z);
  // hardware reciprocal (1 ulp): far inside the rasteriser's edge margin
  const float iz = __builtin_amdgcn_rcpf(p.z);
  return make_float4(cam.fx * p.x * iz + cam.cx, cam.fy * p.y * iz + cam.cy, p.z, iz);
}

// A centre of one triangle: queued for the exact test when within the
// margin of an edge (or the triangle is nearly edge-on), else written.  Beyond
// the queue's end it is only counted: the caller draws the band again in parts.
// (x0, x1, x2) are its edge functions, (m0, m1, m2) their margins, (i0, i1,
// i2) the corners' 1/z and ia 1/area.
template <bool COUNT>
__device__ __forceinline__ void emit_centre(int pix, bool eon, float x0, float x1, float x2, float m0, float m1,
                                            float m2, float i0, float i1, float i2, float ia, uint32_t tid,
                                            uint32_t id_base, unsigned long long* zbuf, const RasterLds& lds,
                                            unsigned& c_frag) {
  if (eon || x0 >= -m0 || x1 >= -m1 || x2 >= -m2) {
    const int slot = atomicAdd(&lds.counts[0], 1);
    if (slot < lds.qcap) lds.queue[slot] = make_uint2((uint32_t)pix, tid);
    return;
  }
  // 1/z is affine in screen space: interpolate with barycentrics x_k/area
  const float z = __builtin_amdgcn_rcpf((x0 * i0 + x1 * i1 + x2 * i2) * ia);
  if (!(z > 0.0f)) return;
  if (COUNT) ++c_frag;
  atomicMin(&zbuf[pix], pack_key(z, id_base + tid));
}

// Word layout of a staged box: edge vectors e0, e1, e2, f0, f1 (x, y), edge
// margins t0, t1, t2, s0, s1, 1/area of both triangles, the edge functions at
// the box's first centre, the corners' 1/z, then (as ints) the box, the two
// triangle ids and the flags act1 | act2 << 1 | eon1 << 2 | eon2 << 3.
enum { kStE = 0, kStT = 10, kStIa = 15, kStW = 17, kStIz = 22, kStBox = 26, kStIds = 30, kStFlags = 32 };

// The whole wave walks a staged box, lane l taking centres l, l + 64, ...;
// each centre gets the coverage tests of the single-lane walk from the same
// values (which walk a box takes depends only on the mesh and the pose).
template <bool COUNT>
__device__ __forceinline__ void walk_staged(const float* __restrict__ st, int lane, const Rect& buf, int pitch,
                                            uint32_t id_base, unsigned long long* zbuf, const RasterLds& lds,
                                            unsigned& c_frag) {
  const int* si = reinterpret_cast<const int*>(st);
  const int c0 = si[kStBox], c1 = si[kStBox + 1], r0 = si[kStBox + 2], r1 = si[kStBox + 3];
  const uint32_t id1 = (uint32_t)si[kStIds], id2 = (uint32_t)si[kStIds + 1];
  const int flags = si[kStFlags];
  const bool act1 = flags & 1, act2 = flags & 2, eon1 = flags & 4, eon2 = flags & 8;
  const float e0x = st[kStE], e0y = st[kStE + 1], e1x = st[kStE + 2], e1y = st[kStE + 3];
  const float e2x = st[kStE + 4], e2y = st[kStE + 5], f0x = st[kStE + 6], f0y = st[kStE + 7];
  const float f1x = st[kStE + 8], f1y = st[kStE + 9];
  const float t0 = st[kStT], t1 = st[kStT + 1], t2 = st[kStT + 2], s0 = st[kStT + 3], s1 = st[kStT + 4];
  const float ia1 = st[kStIa], ia2 = st[kStIa + 1];
  const float w0b = st[kStW], w1b = st[kStW + 1], w2b = st[kStW + 2], v0b = st[kStW + 3], v1b = st[kStW + 4];
  const float izA = st[kStIz], izB = st[kStIz + 1], izC = st[kStIz + 2], izD = st[kStIz + 3];
  const int wc = c1 - c0 + 1, n_cent = wc * (r1 - r0 + 1);
  for (int k = lane; k < n_cent; k += 64) {
    const int dri = k / wc;
    const int r = r0 + dri, col = c0 + (k - dri * wc);
    const float dr = (float)dri, dc = (float)(col - c0);
    const float w0 = __builtin_fmaf(-e0y, dc, __builtin_fmaf(e0x, dr, w0b));
    const float w1 = __builtin_fmaf(-e1y, dc, __builtin_fmaf(e1x, dr, w1b));
    const float w2 = __builtin_fmaf(-e2y, dc, __builtin_fmaf(e2x, dr, w2b));
    const float v0 = __builtin_fmaf(-f0y, dc, __builtin_fmaf(f0x, dr, v0b));
    const float v1 = __builtin_fmaf(-f1y, dc, __builtin_fmaf(f1x, dr, v1b));
    const bool out1 = !act1 || w0 > t0 || w1 > t1 || w2 > t2;
    const bool out2 = !act2 || v0 > s0 || v1 > s1 || -w1 > t1;
    if (out1 && out2) continue;
    const int pix = (r - buf.y0) * pitch + (col - buf.x0);
    if (!out1) emit_centre<COUNT>(pix, eon1, w0, w1, w2, t0, t1, t2, izA, izB, izC, ia1, id1, id_base, zbuf, lds, c_frag);
    if (!out2) emit_centre<COUNT>(pix, eon2, v0, v1, -w1, s0, s1, t1, izA, izC, izD, ia2, id2, id_base, zbuf, lds, c_frag);
  }
}

// Boxes of at most this many rows and columns are walked by a whole wave in
// step; larger ones by each lane on its own.
constexpr int kStepBox = 16;

// An alike cluster (see ClusterDev), one parallelogram per lane.  What bounds
// it is VALU issue: a voxel face covers two or three pixels at the sizes the
// searches run at, so setting a face up costs more than filling it.  Hence
// one corner is transformed and the other three follow from the edge vectors
// (18 multiply-adds and additions for four corners instead of 36, 16 bytes
// read instead of 64); one 1/z plane serves both triangles; and the wave steps
// through the rows and columns of its largest box together, which keeps the
// walk free of per-lane bookkeeping (the boxes of equal faces differ by at
// most a row and a column).  A centre beyond every side by the largest margin
// tq is outside or written at once, on the triangle that the diagonal's sign
// picks; the few between, and every centre of a face seen nearly edge-on, go
// to the queue of the exact test.  Measured against the general path on blobs
// of 1 cm voxels: 429 against 495 us for 5,000 hypotheses of 2,000 voxels at
// 160x120 with the adjoint, 3,086 against 4,177 us for 10,000 of 1,500 voxels at
// 320x240.
// Returns false, for the whole wave, when the general path has to take the
// cluster: a corner behind the near plane (or so near that 1/z is in doubt) or a
// box beyond kStepBox.
template <bool COUNT>
__device__ __forceinline__ bool raster_alike(const ClusterDev& cl, const MeshDev& m, const Pose& P, const Cam& cam,
                                             uint32_t id_base, const Rect& buf, int pitch, float bx0, float bx1,
                                             float by0, float by1, unsigned long long* zbuf, const RasterLds& lds,
                                             int lane, unsigned* c_work) {
  // camera coordinates with x and y scaled by the focal lengths; pixel
  // coordinates with the centres on the integers
  const float cu = cam.cx - 0.5f, cv = cam.cy - 0.5f;
  const bool in = lane < cl.np;
  const size_t pi = (size_t)cl.pfirst + (in ? lane : 0);
  const float4 a = m.pfirsts[pi];
  const uint2 ids = m.pids[pi];
  const float3 oa = xform(P, a.x, a.y, a.z);
  const float3 rb = rotate(P, cl.ab.x, cl.ab.y, cl.ab.z), rd = rotate(P, cl.ad.x, cl.ad.y, cl.ad.z);
  const float bX = cam.fx * rb.x, bY = cam.fy * rb.y, dX = cam.fx * rd.x, dY = cam.fy * rd.y;
  const float aX = cam.fx * oa.x, aY = cam.fy * oa.y;
  const float Bz = oa.z + rb.z, Dz = oa.z + rd.z, Cz = Bz + rd.z;
  const float zmin = fminf(fminf(oa.z, Bz), fminf(Cz, Dz));
  if (__ballot(in && !(zmin > fmaxf(cam.znear, 256.0f * cl.ab.w))) != 0ull) return false;
  const float iA = __builtin_amdgcn_rcpf(oa.z), iB = __builtin_amdgcn_rcpf(Bz);
  const float iC = __builtin_amdgcn_rcpf(Cz), iD = __builtin_amdgcn_rcpf(Dz);
  const float Au = __builtin_fmaf(aX, iA, cu), Av = __builtin_fmaf(aY, iA, cv);
  const float Bu = __builtin_fmaf(aX + bX, iB, cu), Bv = __builtin_fmaf(aY + bY, iB, cv);
  const float Cu = __builtin_fmaf(aX + bX + dX, iC, cu), Cv = __builtin_fmaf(aY + bY + dY, iC, cv);
  const float Du = __builtin_fmaf(aX + dX, iD, cu), Dv = __builtin_fmaf(aY + dY, iD, cv);
  // edges as in the general path: e of (a, b, c), f of (a, c, d), diagonal e1
  const float e0x = Cu - Bu, e0y = Cv - Bv, e1x = Au - Cu, e1y = Av - Cv, e2x = Bu - Au, e2y = Bv - Av;
  const float f0x = Du - Cu, f0y = Dv - Cv, f1x = Au - Du, f1y = Av - Dv;
  const float area1 = e1x * e2y - e2x * e1y, area2 = e1x * f1y - f1x * e1y;
  const float mag = fmaxf(fmaxf(fmaxf(fabsf(Au), fabsf(Av)), fmaxf(fabsf(Bu), fabsf(Bv))),
                          fmaxf(fmaxf(fabsf(Cu), fabsf(Cv)), fmaxf(fabsf(Du), fabsf(Dv))));
  // rounding, and what a corner ab.w away from its place moves on the screen
  // (the projection's slopes are f/z and (u - cx)/z)
  const float wide = fmaxf(cam.fx, cam.fy) + fmaxf(fabsf(cam.cx), fabsf(cam.cy)) + 1.0f;
  const float off = 1.01f * cl.ab.w * fmaxf(fmaxf(iA, iB), fmaxf(iC, iD));
  const float tau = __builtin_fmaf(off, mag + wide, 2e-6f * fmaxf(mag + 0.5f, 256.0f));
  const float len = fmaxf(fmaxf(fmaxf(fabsf(e0x) + fabsf(e0y), fabsf(e1x) + fabsf(e1y)),
                                fmaxf(fabsf(e2x) + fabsf(e2y), fabsf(f0x) + fabsf(f0y))),
                          fabsf(f1x) + fabsf(f1y));
  const float tm = tau * len, amb = 4.0f * tm;
  const bool act = in && !(fminf(area1, area2) > amb);
  const bool eon = !(fmaxf(area1, area2) < -amb);
  const float umin = fminf(fminf(Au, Bu), fminf(Cu, Du)), umax = fmaxf(fmaxf(Au, Bu), fmaxf(Cu, Du));
  const float vmin = fminf(fminf(Av, Bv), fminf(Cv, Dv)), vmax = fmaxf(fmaxf(Av, Bv), fmaxf(Cv, Dv));
  const float c0 = ceilf(fmaxf(umin - tau, bx0)), c1 = floorf(fminf(umax + tau, bx1));
  const float r0 = ceilf(fmaxf(vmin - tau, by0)), r1 = floorf(fminf(vmax + tau, by1));
  const bool has = act && c0 <= c1 && r0 <= r1;
  const float nc = has ? c1 - c0 : -1.0f, nr = has ? r1 - r0 : -1.0f;  // columns and rows less one
  if (__ballot(fmaxf(nr, nc) >= (float)kStepBox) != 0ull) return false;
  if (COUNT && in) {
    c_work[kCntVert] += 4;
    c_work[kCntTri] += 2;
    c_work[kCntSetup] += has ? 2u : 0u;
  }
  // edge functions at the box's first centre, positive outside
  const float w0b = e0x * (r0 - Bv) - e0y * (c0 - Bu), w1b = e1x * (r0 - Cv) - e1y * (c0 - Cu);
  const float w2b = e2x * (r0 - Av) - e2y * (c0 - Au), v0b = f0x * (r0 - Cv) - f0y * (c0 - Cu);
  const float v1b = f1x * (r0 - Dv) - f1y * (c0 - Du);
  // 1/z is affine on the screen: its value at that centre and its gradient
  const float ia = __builtin_amdgcn_rcpf(area1);
  const float zb = (w0b * iA + w1b * iB + w2b * iC) * ia;
  const float zr = (e0x * iA + e1x * iB + e2x * iC) * ia;
  const float zc = (e0y * iA + e1y * iB + e2y * iC) * ia;
  const float tq = eon ? 3.0e38f : tm;
  const uint32_t id1 = id_base + ids.x, id2 = id_base + ids.y;
  const int first = (int)((r0 - (float)buf.y0) * (float)pitch + (c0 - (float)buf.x0));  // exact below 2^24
  for (int r = 0;; ++r) {
    const float dr = (float)r;
    const bool row = dr <= nr;
    if (__ballot(row) == 0ull) break;
    const float w0r = __builtin_fmaf(e0x, dr, w0b), w1r = __builtin_fmaf(e1x, dr, w1b);
    const float w2r = __builtin_fmaf(e2x, dr, w2b), v0r = __builtin_fmaf(f0x, dr, v0b);
    const float v1r = __builtin_fmaf(f1x, dr, v1b), izr = __builtin_fmaf(zr, dr, zb);
    const float ncr = row ? nc : -1.0f;
    const int pixr = first + r * pitch;
    for (int c = 0;; ++c) {
      const float dc = (float)c;
      const bool col = dc <= ncr;
      if (__ballot(col) == 0ull) break;
      const float w0 = __builtin_fmaf(-e0y, dc, w0r), w1 = __builtin_fmaf(-e1y, dc, w1r);
      const float w2 = __builtin_fmaf(-e2y, dc, w2r), v0 = __builtin_fmaf(-f0y, dc, v0r);
      const float v1 = __builtin_fmaf(-f1y, dc, v1r);
      const float side = fmaxf(fmaxf(fmaxf(w0, w2), v0), v1);
      if (col && !(side > tq)) {
        const int pix = pixr + c;
        if (fmaxf(side, -fabsf(w1)) < -tq) {
          if (COUNT) ++c_work[kCntFrag];
          const float z = __builtin_amdgcn_rcpf(__builtin_fmaf(-zc, dc, izr));
          atomicMin(&zbuf[pix], pack_key(z, w1 > 0.0f ? id2 : id1));
        } else {
          // within the margin of an edge or the diagonal: both triangles that may hold it
          for (int k = 0; k < 2; ++k) {
            const float x0 = k ? v0 : w0, x1 = k ? v1 : w1, x2 = k ? -w1 : w2;
            const float top = fmaxf(fmaxf(x0, x1), x2);
            if (top > tm) continue;
            const int slot = atomicAdd(&lds.counts[0], 1);
            if (slot < lds.qcap) lds.queue[slot] = make_uint2((uint32_t)pix, k ? ids.y : ids.x);
          }
        }
      }
    }
  }
  return true;
}

// Rasterise the mesh under pose P into the pixels of the image rectangle
// `band` of an LDS key buffer that covers the rectangle `buf` (row pitch
// buf.w(); band inside buf).  Triangle ids written are
// id_base + the caller's triangle index.  Clusters are tested for drawing,
// one per thread at a time, and the drawable ones compacted into a list; the
// waves then take clusters from the list independently: each lane takes one
// primitive (a quad or a triangle), projects its corners and walks the pixel
// centres of its screen box (alike clusters: see raster_alike); with BIG, up to kBigSlots boxes of more than kBigCentres centres per
// wave and cluster are walked by the whole wave instead (with the same
// coverage tests from the same values).  A centre that single
// precision places clearly inside all three edges is written at once (64-bit
// atomicMin of the packed depth/id key); one that lies within a rounding
// margin of an edge, or any centre of a triangle seen nearly edge-on, is
// queued and decided afterwards by covered_exact (its depth from *view, the
// pose's plane view in LDS).  Returns true, in every thread, when more centres
// came up than the queue holds: those are not decided, and the caller has to
// draw the band again in smaller parts (what is drawn already is right, and
// drawing it again changes nothing).  A band of one pixel tests every triangle
// instead.  Must be called by the whole block; its barriers order LDS alone; ends
// after a barrier.
template <bool COUNT, bool BIG, int BS>
__device__ __forceinline__ bool raster_mesh(const MeshDev& m, const Pose& P, const Cam& cam, uint32_t id_base,
                                            const Rect& band, const Rect& buf, unsigned long long* zbuf,
                                            const RasterLds& lds, const PlaneView* view, unsigned* cnt = nullptr) {
  unsigned c_vert = 0, c_tri = 0, c_setup = 0, c_frag = 0, c_exact = 0;
  unsigned c_alike[kCntN] = {};  // raster_alike's share
  const int pitch = buf.w();
  const float bx0 = (float)band.x0, bx1 = (float)(band.x1 - 1);
  const float by0 = (float)band.y0, by1 = (float)(band.y1 - 1);
  if (threadIdx.x == 0) lds.counts[0] = 0;
  // the hidden-pair clusters matter only when the object reaches the near
  // plane: the z of the box's corners, eight lanes sharing them
  const int k8 = threadIdx.x & 7;
  const float3 corner =
      xform(P, (k8 & 1) ? m.hi[0] : m.lo[0], (k8 & 2) ? m.hi[1] : m.lo[1], (k8 & 4) ? m.hi[2] : m.lo[2]);
  const int n_clusters = __ballot(!(corner.z > cam.znear)) != 0ull ? m.n_clusters : m.n_visible;
  constexpr int kW = BS / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int base = 0; base < n_clusters; base += BS) {
    // each thread tests one cluster; the drawable ones are compacted into `list`
    const int mine = base + threadIdx.x;
    const bool draw = mine < n_clusters && cluster_may_draw(m.clusters[mine], P, cam, band);
    const unsigned long long mask = __ballot(draw);
    lds_barrier();  // the previous group's list is no longer read
    if (lane == 0) lds.counts[1 + wave] = __popcll(mask);
    if (threadIdx.x == 0) lds.counts[1 + kW] = 0;
    lds_barrier();
    int off = 0, total = 0;
    for (int w = 0; w < kW; ++w) {
      off += (w < wave) ? lds.counts[1 + w] : 0;
      total += lds.counts[1 + w];
    }
    if (draw) lds.list[off + __popcll(mask & ((1ull << lane) - 1ull))] = mine;
    lds_barrier();
    for (;;) {
      int q = 0;
      if (lane == 0) q = atomicAdd(&lds.counts[1 + kW], 1);
      q = __shfl(q, 0, 64);
      if (q >= total) break;
      const ClusterDev cl = m.clusters[__builtin_amdgcn_readfirstlane(lds.list[q])];
      if (__builtin_amdgcn_readfirstlane(cl.alike) && raster_alike<COUNT>(cl, m, P, cam, id_base, buf, pitch, bx0, bx1, by0, by1, zbuf, lds, lane, c_alike))
        continue;
      bool staged = false;
      if (lane < cl.np) {
        const size_t pi = (size_t)cl.pfirst + lane;
        const uint2 ids = m.pids[pi];
        const bool quad = ids.y != kNoTri;
        // corners as (u, v, z, 1/z); triangle 1 = (a, b, c), triangle 2 = (a, c, d)
        const float4* pv = m.pverts + 4 * pi;
        const float4 A = project_corner(P, cam, pv[0]), B = project_corner(P, cam, pv[1]);
        const float4 C = project_corner(P, cam, pv[2]), D = project_corner(P, cam, pv[3]);
        if (COUNT) {
          c_vert += 4;
          c_tri += quad ? 2 : 1;
        }
        const float zn = cam.znear;
        const bool near1 = A.z <= zn || B.z <= zn || C.z <= zn;
        const bool near2 = A.z <= zn || C.z <= zn || D.z <= zn;
        // edges of triangle 1 (e_k opposite corner k) and of triangle 2 (f_k); the
        // diagonal a-c is e1 (c -> a) for triangle 1 and -e1 for triangle 2
        const float e0x = C.x - B.x, e0y = C.y - B.y;
        const float e1x = A.x - C.x, e1y = A.y - C.y;
        const float e2x = B.x - A.x, e2y = B.y - A.y;
        const float f0x = D.x - C.x, f0y = D.y - C.y;
        const float f1x = A.x - D.x, f1y = A.y - D.y;
        // rounding margin (pixels) from the magnitudes of the corners in use
        float mag = fmaxf(fmaxf(fabsf(A.x), fabsf(A.y)), fmaxf(fabsf(C.x), fabsf(C.y)));
        const float area1 = e2x * (C.y - A.y) - (C.x - A.x) * e2y;
        const float area2 = -e1x * (D.y - A.y) + (D.x - A.x) * e1y;
        // preliminary activity (near plane) decides which corners set the margin
        const bool use1 = !near1, use2 = quad && !near2;
        mag = fmaxf(mag, use1 ? fmaxf(fabsf(B.x), fabsf(B.y)) : 0.0f);
        mag = fmaxf(mag, use2 ? fmaxf(fabsf(D.x), fabsf(D.y)) : 0.0f);
        const float tau = 2e-6f * fmaxf(mag, 256.0f);
        const float amb1 = 2.0f * tau * (fabsf(e1x) + fabsf(e1y) + fabsf(e2x) + fabsf(e2y));
        const float amb2 = 2.0f * tau * (fabsf(f1x) + fabsf(f1y) + fabsf(e1x) + fabsf(e1y));
        // drawn unless behind the near plane or facing away
        const bool act1 = use1 && !(area1 > amb1);
        const bool act2 = use2 && !(area2 > amb2);
        // box of the active triangles' corners (a and c belong to both)
        const float bxu = act1 ? B.x : A.x, bxv = act1 ? B.y : A.y;
        const float dxu = act2 ? D.x : A.x, dxv = act2 ? D.y : A.y;
        const float umin = fminf(fminf(A.x, C.x), fminf(bxu, dxu)), umax = fmaxf(fmaxf(A.x, C.x), fmaxf(bxu, dxu));
        const float vmin = fminf(fminf(A.y, C.y), fminf(bxv, dxv)), vmax = fmaxf(fmaxf(A.y, C.y), fmaxf(bxv, dxv));
        const float fc0 = ceilf(fmaxf(umin - 0.5f - tau, bx0)), fc1 = floorf(fminf(umax - 0.5f + tau, bx1));
        const float fr0 = ceilf(fmaxf(vmin - 0.5f - tau, by0)), fr1 = floorf(fminf(vmax - 0.5f + tau, by1));
        if ((act1 || act2) && fc0 <= fc1 && fr0 <= fr1) {
          const int c0 = (int)fc0, c1 = (int)fc1, r0 = (int)fr0, r1 = (int)fr1;
          if (COUNT) c_setup += (act1 ? 1u : 0u) + (act2 ? 1u : 0u);
          const bool eon1 = area1 >= -amb1, eon2 = area2 >= -amb2;
          const float ia1 = __builtin_amdgcn_rcpf(area1), ia2 = __builtin_amdgcn_rcpf(area2);
          const float t0 = tau * (fabsf(e0x) + fabsf(e0y)), t1 = tau * (fabsf(e1x) + fabsf(e1y)),
                      t2 = tau * (fabsf(e2x) + fabsf(e2y));
          const float s0 = tau * (fabsf(f0x) + fabsf(f0y)), s1 = tau * (fabsf(f1x) + fabsf(f1y));
          // a centre of triangle k: queued for the exact test when within the
          // margin of an edge (or the triangle is nearly edge-on), else written
          // edge functions (each the negative area at the opposite corner) at the
          // box's first centre; at a centre dr rows and dc columns further they
          // are w + e_x dr - e_y dc with exact small integers dr, dc: two FMAs
          // each, and the rounding stays far below the margin for any box size
          const float py0 = (float)r0 + 0.5f, px0 = (float)c0 + 0.5f;
          const float w0b = e0x * (py0 - B.y) - e0y * (px0 - B.x);
          const float w1b = e1x * (py0 - C.y) - e1y * (px0 - C.x);
          const float w2b = e2x * (py0 - A.y) - e2y * (px0 - A.x);
          const float v0b = f0x * (py0 - C.y) - f0y * (px0 - C.x);
          const float v1b = f1x * (py0 - D.y) - f1y * (px0 - D.x);
          // one flat walk over the box's centres: a wave then iterates max(rows x cols)
          // times over its lanes, not max(rows) x max(cols)
          int n_cent = (c1 - c0 + 1) * (r1 - r0 + 1);
          // a large box (a table top, a wall) would keep this lane walking long
          // after the others are done: the first kBigSlots of them are staged in
          // the wave's LDS slots and walked by the whole wave below
          const unsigned long long bigm = BIG ? __ballot(n_cent > kBigCentres) : 0ull;
          if (BIG && bigm != 0ull && n_cent > kBigCentres && __popcll(bigm & ((1ull << lane) - 1ull)) < kBigSlots) {
            const int rank = __popcll(bigm & ((1ull << lane) - 1ull));
            float* st = raster_stage<BS>(lds) + (wave * kBigSlots + rank) * kStageWords;
            int* si = reinterpret_cast<int*>(st);
            const float vals[26] = {e0x, e0y, e1x, e1y, e2x, e2y, f0x, f0y, f1x, f1y, t0,  t1,  t2,
                                    s0,  s1,  ia1, ia2, w0b, w1b, w2b, v0b, v1b, A.w, B.w, C.w, D.w};
#pragma unroll
            for (int k = 0; k < 26; ++k) st[k] = vals[k];
            si[kStBox] = c0;
            si[kStBox + 1] = c1;
            si[kStBox + 2] = r0;
            si[kStBox + 3] = r1;
            si[kStIds] = (int)ids.x;
            si[kStIds + 1] = (int)ids.y;
            si[kStFlags] = (act1 ? 1 : 0) | (act2 ? 2 : 0) | (eon1 ? 4 : 0) | (eon2 ? 8 : 0);
            staged = true;
            n_cent = 0;
          }
          // the offsets from the box's first centre as exact small floats,
          // stepped along the row and wrapped to the next one
          const float dcmax = (float)(c1 - c0), drmax = n_cent > 0 ? (float)(r1 - r0) : -1.0f;
          float dr = 0.0f, dc = 0.0f;
          while (dr <= drmax) {
            const float drn = dc < dcmax ? dr : dr + 1.0f;
            const float dcn = dc < dcmax ? dc + 1.0f : 0.0f;
            const float w0 = __builtin_fmaf(-e0y, dc, __builtin_fmaf(e0x, dr, w0b));
            const float w1 = __builtin_fmaf(-e1y, dc, __builtin_fmaf(e1x, dr, w1b));
            const float w2 = __builtin_fmaf(-e2y, dc, __builtin_fmaf(e2x, dr, w2b));
            const float v0 = __builtin_fmaf(-f0y, dc, __builtin_fmaf(f0x, dr, v0b));
            const float v1 = __builtin_fmaf(-f1y, dc, __builtin_fmaf(f1x, dr, v1b));
            const bool out1 = !act1 || w0 > t0 || w1 > t1 || w2 > t2;
            const bool out2 = !act2 || v0 > s0 || v1 > s1 || -w1 > t1;
            const float drc = dr, dcc = dc;
            dr = drn;
            dc = dcn;
            if (out1 && out2) continue;  // clearly outside both
            const int r = r0 + (int)drc, col = c0 + (int)dcc;
            const int pix = (r - buf.y0) * pitch + (col - buf.x0);
            if (!out1)
              emit_centre<COUNT>(pix, eon1, w0, w1, w2, t0, t1, t2, A.w, B.w, C.w, ia1, ids.x, id_base, zbuf, lds,
                                 c_frag);
            if (!out2)
              emit_centre<COUNT>(pix, eon2, v0, v1, -w1, s0, s1, t1, A.w, C.w, D.w, ia2, ids.y, id_base, zbuf, lds,
                                 c_frag);
          }
        }
      }
      if constexpr (BIG) {
        __builtin_amdgcn_wave_barrier();
        const unsigned long long sm = __ballot(staged);
        if (sm != 0ull) {
          const int n_staged = __popcll(sm);
          for (int j = 0; j < n_staged; ++j)
            walk_staged<COUNT>(raster_stage<BS>(lds) + (wave * kBigSlots + j) * kStageWords, lane, buf, pitch, id_base,
                               zbuf, lds, c_frag);
        }
      }
    }
  }
  lds_barrier();
  // centres near an edge: the exact test, then the plane depth
  const int found = __builtin_amdgcn_readfirstlane(lds.counts[0]);
  const bool over = found > lds.qcap, one = band.h() * band.w() == 1;
  const int nq = !over ? found : one ? m.T : 0;
  for (int k = threadIdx.x; k < nq; k += BS) {
    uint2 e = make_uint2((uint32_t)((band.y0 - buf.y0) * pitch + (band.x0 - buf.x0)), (uint32_t)k);
    if (!over) e = lds.queue[k];
    const int r = buf.y0 + (int)e.x / pitch, col = buf.x0 + (int)e.x % pitch;
    if (COUNT) ++c_exact;
    if (!covered_exact(m, P, cam, e.y, r, col)) continue;
    const float z = plane_depth(m, *view, e.y, r, col);
    if (!(z > 0.0f)) continue;
    if (COUNT) ++c_frag;
    atomicMin(&zbuf[e.x], pack_key(z, id_base + e.y));
  }
  if (COUNT) {
    atomicAdd(&cnt[kCntVert], c_vert + c_alike[kCntVert]);
    atomicAdd(&cnt[kCntTri], c_tri + c_alike[kCntTri]);
    atomicAdd(&cnt[kCntSetup], c_setup + c_alike[kCntSetup]);
    atomicAdd(&cnt[kCntFrag], c_frag + c_alike[kCntFrag]);
    atomicAdd(&cnt[kCntExact], c_exact);
  }
  lds_barrier();
  return over && !one;
}

// raster_mesh over the band, whole or, where the exact test's queue does not
// hold its centres, in strips of rows and at last of columns.  That takes a view
// along the axes of a regular mesh, with pixel centres on its edges: a quarter of
// the centres of a plate of 8-pixel voxels seen from the front.  (Deciding what the
// queue does not hold in single precision left holes of hundreds of pixels in such
// an image.  Where no part is needed, the loop costs 0 to 1 %: 1,838 against 1,816
// us for 10,000 hypotheses of 1,500 voxels at 320x240; 0.4 us where a launch
// lasts as long as one workgroup.)
template <bool COUNT, bool BIG, int BS>
__device__ __forceinline__ void raster_parts(const MeshDev& m, const Pose& P, const Cam& cam, uint32_t id_base,
                                             const Rect& band, const Rect& buf, unsigned long long* zbuf,
                                             const RasterLds& lds, const PlaneView* view, unsigned* cnt) {
  Rect part = band;
  int rows = band.h(), cols = band.w();  // of a strip
  while (part.y0 < band.y1) {
    part.y1 = min(part.y0 + rows, band.y1);
    part.x1 = min(part.x0 + cols, band.x1);
    if (raster_mesh<COUNT, BIG, BS>(m, P, cam, id_base, part, buf, zbuf, lds, view, cnt)) {
      if (rows > 1)
        rows = (part.h() + 1) / 2;
      else
        cols = (part.w() + 1) / 2;
    } else if (part.x1 < band.x1) {
      part.x0 = part.x1;
    } else {
      part.x0 = band.x0;
      part.y0 = part.y1;
    }
  }
}

// Which rasteriser a kernel holds: the plain one, the one with the wave walk
// of large boxes, or both behind a test of the mesh's has_big (the large-box
// walk costs meshes without large primitives a few per cent).
enum RasterMode { kRasterSmall = 0, kRasterBig = 1, kRasterAny = 2 };

template <bool COUNT, int MODE, int BS>
__device__ __forceinline__ void raster_mesh_mode(const MeshDev& m, const Pose& P, const Cam& cam, uint32_t id_base,
                                                 const Rect& band, const Rect& buf, unsigned long long* zbuf,
                                                 const RasterLds& lds, const PlaneView* view,
                                                 unsigned* cnt = nullptr) {
  if (MODE == kRasterBig || (MODE == kRasterAny && m.has_big)) {
    RasterLds shorter = lds;
    shorter.qcap = kQueueCap - stage_queue_entries(BS);
    raster_parts<COUNT, true, BS>(m, P, cam, id_base, band, buf, zbuf, shorter, view, cnt);
  } else {
    raster_parts<COUNT, false, BS>(m, P, cam, id_base, band, buf, zbuf, lds, view, cnt);
  }
}

// Row r and column c of slot k (0 <= k < 2^20) of a rectangle of width w,
// given inv_w = 1/w correctly rounded: (k + 1/2) inv_w is formed with one
// rounding, a relative error below 2^-22, so it lies within 1/(4w) of
// (k + 1/2)/w, whose fractional part is in [1/(2w), 1 - 1/(2w)]: truncating it
// gives floor(k/w) exactly, with no integer division.
__device__ __forceinline__ void row_col(int k, int w, float inv_w, int& r, int& c) {
  r = (int)__builtin_fmaf((float)k, inv_w, 0.5f * inv_w);
  c = k - __mul24(r, w);
}

// Work compaction inside a wave: of the items 0 .. n - 1 (64 consecutive ones
// per wave and turn, wave w of NW taking turns w, w + NW, ...) those that are
// `wanted` are processed 64 at a time, one per lane, so that a wave does not
// run long work for a few lanes.  Indices wait in the wave's own LDS queue q
// (kWaveQueue entries): no barrier.  Called by whole waves; `wanted` and
// process(index, active) run with all lanes.
constexpr int kWaveQueue = 128;

__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

template <int NW, class W, class F>
__device__ __forceinline__ void wave_compacted(int n, unsigned short* q, W&& wanted, F&& process) {
  const int lane = threadIdx.x & 63;
  int base = __builtin_amdgcn_readfirstlane(((int)threadIdx.x >> 6) * 64);
  int head = 0, fill = 0;  // the ring's first entry and its number of entries
  for (;;) {
    while (fill < 64 && base < n) {
      const int item = base + lane;
      const bool want = item < n && wanted(item);
      const unsigned long long m = __ballot(want);
      if (want) q[(head + fill + lanes_below(m)) & (kWaveQueue - 1)] = (unsigned short)item;
      fill += __popcll(m);
      base += NW * 64;
    }
    if (fill <= 0) break;
    __builtin_amdgcn_wave_barrier();
    const int item = q[(head + lane) & (kWaveQueue - 1)];
    const bool act = lane < fill;
    head += 64;
    fill -= 64;
    __builtin_amdgcn_wave_barrier();
    process(item, act);
  }
}

// One Adam ascent step on logL for pose P (row-major 4x4), on the tangent
// (dt, dw): m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2,
// s = lr * mhat / (sqrt(vhat) + eps), then t <- t + s[0:3], R <- exp([s[3:6]]x) R.
__device__ __forceinline__ void adam_update(float* P, const float* g, float* m, float* v, int iter, float lr_t,
                                            float lr_r, float b1, float b2, float eps) {
  const float c1 = 1.0f - powf(b1, (float)iter), c2 = 1.0f - powf(b2, (float)iter);
  float s[6];
  for (int k = 0; k < 6; ++k) {
    m[k] = b1 * m[k] + (1.0f - b1) * g[k];
    v[k] = b2 * v[k] + (1.0f - b2) * g[k] * g[k];
    const float mh = m[k] / c1, vh = v[k] / c2;
    s[k] = (k < 3 ? lr_t : lr_r) * mh / (sqrtf(vh) + eps);
  }
  for (int k = 0; k < 3; ++k) P[4 * k + 3] += s[k];
  const float wx = s[3], wy = s[4], wz = s[5];
  const float th = sqrtf(wx * wx + wy * wy + wz * wz);
  if (th > 0.0f) {
    const float kx = wx / th, ky = wy / th, kz = wz / th;
    const float sn = sinf(th), cs = 1.0f - cosf(th);
    const float E[9] = {1.0f + cs * (kx * kx - 1.0f), -sn * kz + cs * kx * ky,       sn * ky + cs * kx * kz,
                        sn * kz + cs * kx * ky,       1.0f + cs * (ky * ky - 1.0f), -sn * kx + cs * ky * kz,
                        -sn * ky + cs * kx * kz,      sn * kx + cs * ky * kz,       1.0f + cs * (kz * kz - 1.0f)};
    float R[9];
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) R[3 * i + j] = E[3 * i] * P[j] + E[3 * i + 1] * P[4 + j] + E[3 * i + 2] * P[8 + j];
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) P[4 * i + j] = R[3 * i + j];
  }
}

// Fixed-order sum over the 64 lanes of a wave (butterfly), result in all lanes.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Fixed-order block sum of NV floats; the result is valid in thread 0.
// `red` must hold kWaves * NV floats of LDS.
template <int NV>
__device__ __forceinline__ void block_sum(float (&v)[NV], float* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wave * NV + k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      float s = red[k];
      for (int w = 1; w < kWaves; ++w) s += red[w * NV + k];
      v[k] = s;
    }
  }
  __syncthreads();
}

}  // namespace b3d
