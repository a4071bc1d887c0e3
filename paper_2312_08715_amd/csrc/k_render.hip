// Split-path rendering kernels: batched point-image render (one workgroup
// per hypothesis, LDS depth buffer over the object's pixel rectangle),
// depth-to-point conversion, the frozen-visibility pose adjoint, and the
// global-memory rasteriser used once per scene for static objects.
#include "b3d_launch.hpp"

namespace b3d {

static size_t render_lds_bytes(int bs, int zcap) {
  return raster_lds_bytes(bs) + sizeof(unsigned long long) * (size_t)zcap + kPlaneViewBytes;
}

// Rows [y0, y1) of an image written empty, as 16-byte words where the image is
// made of them (VEC: rows of 4 k pixels in 16-byte aligned buffers).
template <bool VEC, int BS>
__device__ __forceinline__ void write_empty_rows(int W, int y0, int y1, float* __restrict__ xyz, int* __restrict__ tri) {
  const size_t first = (size_t)y0 * W;
  const int np = (y1 - y0) * W;
  if constexpr (VEC) {
    float4* x4 = reinterpret_cast<float4*>(xyz + 3 * first);
    for (int k = threadIdx.x; k < 3 * (np / 4); k += BS) x4[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (tri) {
      int4* t4 = reinterpret_cast<int4*>(tri + first);
      for (int k = threadIdx.x; k < np / 4; k += BS) t4[k] = make_int4(-1, -1, -1, -1);
    }
  } else {
    float* x = xyz + 3 * first;
    for (int k = threadIdx.x; k < 3 * np; k += BS) x[k] = 0.0f;
    if (tri) {
      int* t = tri + first;
      for (int k = threadIdx.x; k < np; k += BS) t[k] = -1;
    }
  }
}

// Rows of the band: pixels inside it come from the LDS key buffer, others are
// empty.  Four pixels per lane (VEC), or one.
template <bool VEC, int BS>
__device__ __forceinline__ void write_band_rows(const Cam& cam, const Rect& band, const unsigned long long* zbuf,
                                                float* __restrict__ xyz, int* __restrict__ tri) {
  constexpr int V = VEC ? 4 : 1;
  const int W = cam.W, per_row = W / V, n_rows = band.h(), bw = band.w();
  // row and column stepped, not found from an index: a narrow object's band can
  // hold more pixels of the image than row_col is exact for
  const int step_r = BS / per_row, step_c = BS - step_r * per_row;
  int dr = (int)threadIdx.x / per_row, qc = (int)threadIdx.x - dr * per_row;
  while (dr < n_rows) {
    const int r = band.y0 + dr, c0 = V * qc;
    float x[V], y[V], z[V];
    int id[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      x[u] = y[u] = z[u] = 0.0f;
      id[u] = -1;
    }
    if (c0 + V > band.x0 && c0 < band.x1) {
      const float ry = ray_y(cam, r);
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const int c = c0 + u;
        if (c < band.x0 || c >= band.x1) continue;
        const unsigned long long k = zbuf[dr * bw + (c - band.x0)];
        if (k == kEmptyKey) continue;
        z[u] = key_depth(k);
        x[u] = z[u] * ray_x(cam, c);
        y[u] = z[u] * ry;
        id[u] = (int)key_id(k);
      }
    }
    const size_t p = (size_t)r * W + c0;
    if constexpr (VEC) {
      float4* o = reinterpret_cast<float4*>(xyz + 3 * p);
      o[0] = make_float4(x[0], y[0], z[0], x[1]);
      o[1] = make_float4(y[1], z[1], x[2], y[2]);
      o[2] = make_float4(z[2], x[3], y[3], z[3]);
      if (tri) *reinterpret_cast<int4*>(tri + p) = make_int4(id[0], id[1], id[2], id[3]);
    } else {
      xyz[3 * p] = x[0];
      xyz[3 * p + 1] = y[0];
      xyz[3 * p + 2] = z[0];
      if (tri) tri[p] = id[0];
    }
    dr += step_r;
    qc += step_c;
    if (qc >= per_row) {
      qc -= per_row;
      ++dr;
    }
  }
}

// One workgroup per hypothesis.  What bounds it is writing the images (16 bytes
// a pixel) and, before its rows can be written, rasterising: the rows that the
// object does not reach come last, so that their stores drain while the next
// workgroup on the CU rasterises, and the barriers in between order LDS alone.
// (Writing the whole image empty first and the drawn pixels after their depths
// took 214 us for 2,000 images of 160x120: every workgroup of the first wave then
// waits on the same stores.)
// Block sizes and the second launch as for the fused kernel; a hypothesis left
// to it is marked in its image's first word, which it rewrites.
template <int RM, bool VEC, int BS, int PART>
__global__ __launch_bounds__(BS, 4) void k_render_batch(MeshDev m, Cam cam, const float* __restrict__ poses, int N,
                                                         float* __restrict__ xyz, int* __restrict__ tri, int zcap) {
  extern __shared__ __align__(16) unsigned char smem[];
  const RasterLds rl = carve_raster_lds<BS>(smem);
  unsigned long long* zbuf = reinterpret_cast<unsigned long long*>(smem + raster_lds_bytes(BS));
  const int n = blockIdx.x;
  if (n >= N) return;
  const Pose P = load_pose(poses + 16 * (size_t)n);
  const int H = cam.H, W = cam.W;
  float* xn = xyz + (size_t)n * H * W * 3;
  int* tn = tri ? tri + (size_t)n * H * W : nullptr;
  if (PART == kRest && __float_as_uint(xn[0]) != kDeferred) return;
  const Rect obj = object_rect(m, P, cam);
  if (PART == kFirst && obj.w() * obj.h() > zcap) {
    if (threadIdx.x == 0) xn[0] = __uint_as_float(kDeferred);
    return;
  }
  if (obj.empty()) {
    write_empty_rows<VEC, BS>(W, 0, H, xn, tn);
    return;
  }
  const int band_rows = max(zcap / obj.w(), 1);
  PlaneView* view = reinterpret_cast<PlaneView*>(zbuf + zcap);
  if (threadIdx.x == 0) *view = plane_view(P, cam);
  const float inv_w = 1.0f / (float)obj.w();
  for (int a = obj.y0; a < obj.y1; a += band_rows) {
    Rect band = obj;
    band.y0 = a;
    band.y1 = min(a + band_rows, obj.y1);
    const int nk = band.h() * band.w();
    for (int k = threadIdx.x; k < nk; k += BS) zbuf[k] = kEmptyKey;
    lds_barrier();
    raster_mesh_mode<false, RM, BS>(m, P, cam, 0u, band, band, zbuf, rl, view);
    // the drawn slots' depths on their triangles' planes
    wave_compacted<(BS / 64)>(
        nk, reinterpret_cast<unsigned short*>(smem) + (threadIdx.x >> 6) * kWaveQueue,
        [&](int k) { return zbuf[k] != kEmptyKey; },
        [&](int k, bool act) {
          if (!act) return;
          const uint32_t id = key_id(zbuf[k]);
          int r, c;
          row_col(k, band.w(), inv_w, r, c);
          zbuf[k] = pack_key(plane_depth(m, *view, id, band.y0 + r, band.x0 + c), id);
        });
    lds_barrier();
    write_band_rows<VEC, BS>(cam, band, zbuf, xn, tn);
    lds_barrier();
  }
  write_empty_rows<VEC, BS>(W, 0, obj.y0, xn, tn);
  write_empty_rows<VEC, BS>(W, obj.y1, H, xn, tn);
}

template <int BS, int PART = kAlone>
static void launch_render_bs(const MeshDev& m, const Cam& cam, const float* poses, int N, float* xyz, int* tri,
                             int zcap, hipStream_t st) {
  const size_t lds = render_lds_bytes(BS, zcap);
  // whole 16-byte words: rows of 4 k pixels in 16-byte aligned buffers
  const bool vec = cam.W % 4 == 0 && (((uintptr_t)xyz | (uintptr_t)tri) & 15) == 0;
  auto k = m.has_big ? (vec ? k_render_batch<kRasterBig, true, BS, PART> : k_render_batch<kRasterBig, false, BS, PART>)
                     : (vec ? k_render_batch<kRasterSmall, true, BS, PART>
                            : k_render_batch<kRasterSmall, false, BS, PART>);
  hipLaunchKernelGGL(k, dim3(N), dim3(BS), lds, st, m, cam, poses, N, xyz, tri, zcap);
}

// Depth keys for a block of bs threads: its share of a CU's LDS, no more than
// the image needs (slots are listed as 16-bit indices).
static int render_zcap(const Cam& cam, int bs) {
  const int fit = (int)((kLdsPerCU / (1024 / bs) - render_lds_bytes(bs, 0)) / 8);
  return min(fit, cam.W * cam.H);
}

// Block sizes and the second launch as for the fused kernel, but that images
// large enough for it go by 512 threads alone up to two rounds of them: each
// launch drains its own stores, and which hypotheses are left is a matter of a few
// rows (1,024 spheres of 12,000 triangles at 320x240: 278 us against 373).
hipError_t launch_render_batch(const MeshDev& m, const Cam& cam, const float* poses, int N, float* xyz, int* tri,
                               hipStream_t st) {
  const int small = max(render_zcap(cam, kBlock), cam.W);
  if (N <= kCUs) {
    launch_render_bs<1024>(m, cam, poses, N, xyz, tri, render_zcap(cam, 1024), st);
  } else if (N <= 2 * kCUs || (N <= 4 * kCUs && cam.W * cam.H > kBandedPixels)) {
    launch_render_bs<512>(m, cam, poses, N, xyz, tri, render_zcap(cam, 512), st);
  } else if (cam.W * cam.H > max(small, kBandedPixels) || (cam.W * cam.H > small && N >= kBandedCount)) {
    launch_render_bs<kBlock, kFirst>(m, cam, poses, N, xyz, tri, small, st);
    if (cam.W * cam.H > kWholeCuPixels)
      launch_render_bs<1024, kRest>(m, cam, poses, N, xyz, tri, render_zcap(cam, 1024), st);
    else
      launch_render_bs<512, kRest>(m, cam, poses, N, xyz, tri, render_zcap(cam, 512), st);
  } else {
    launch_render_bs<kBlock>(m, cam, poses, N, xyz, tri, small, st);
  }
  return hipGetLastError();
}

__global__ void k_unproject(const float* __restrict__ depth, int B, Cam cam, float* __restrict__ xyz) {
  const size_t total = (size_t)B * cam.H * cam.W;
  for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < total; p += (size_t)gridDim.x * blockDim.x) {
    const int pix = (int)(p % ((size_t)cam.H * cam.W));
    const int r = pix / cam.W, c = pix - r * cam.W;
    const float z = depth[p] > 0.0f ? depth[p] : 0.0f;
    xyz[3 * p + 0] = z * ray_x(cam, c);
    xyz[3 * p + 1] = z * ray_y(cam, r);
    xyz[3 * p + 2] = z;
  }
}

hipError_t launch_unproject(const float* depth, int B, const Cam& cam, float* xyz, hipStream_t st) {
  const size_t total = (size_t)B * cam.H * cam.W;
  const int blocks = (int)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
  hipLaunchKernelGGL(k_unproject, dim3(blocks), dim3(256), 0, st, depth, B, cam, xyz);
  return hipGetLastError();
}

// d_pose[n] = sum_j g_j (n/(n.d), n x (t - q)/(n.d)), g_j = d_rend_j . d_j,
// with the depth of pixel j taken on the plane of its triangle.  The ids are
// read as 16-byte words of four pixels where the image allows it (VEC); a
// wave's drawn pixels wait in its LDS queue and are processed 64 at a time, so
// that the few drawn pixels of an image do not each hold a wave (2,000 images
// of 160x120 with one lane per pixel: 134 us).
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_render_backward(MeshDev m, Cam cam, const float* __restrict__ poses,
                                                            int N, const int* __restrict__ tri,
                                                            const float* __restrict__ d_rend,
                                                            float* __restrict__ d_pose) {
  __shared__ double red[kWaves * 6];
  __shared__ PlaneView view;
  __shared__ int queues[kWaves][kWaveQueue];
  const int n = blockIdx.x;
  if (n >= N) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Pose P = load_pose(poses + 16 * (size_t)n);
  if (threadIdx.x == 0) view = plane_view(P, cam);
  __syncthreads();
  const int HW = cam.H * cam.W;
  const int* tn = tri + (size_t)n * HW;
  const float* dn = d_rend + (size_t)n * HW * 3;
  int* q = queues[wave];
  double acc[6] = {0, 0, 0, 0, 0, 0};
  int head = 0, fill = 0;
  auto drain = [&](int least) {
    while (fill >= least && fill > 0) {
      __builtin_amdgcn_wave_barrier();
      const int p = q[(head + lane) & (kWaveQueue - 1)];
      const bool act = lane < fill;
      __builtin_amdgcn_wave_barrier();
      head += 64;
      fill -= 64;
      if (!act) continue;
      const int id = tn[p];
      const int r = p / cam.W, c = p - r * cam.W;
      const float dx = ray_x(cam, c), dy = ray_y(cam, r);
      const float g = dn[3 * (size_t)p] * dx + dn[3 * (size_t)p + 1] * dy + dn[3 * (size_t)p + 2];
      if (g == 0.0f) continue;
      const float4 no = m.normals[id];
      const float3 nn = rotate(P, no.x, no.y, no.z);
      const float nd = nn.x * dx + nn.y * dy + nn.z;
      const float z = plane_depth(m, view, (uint32_t)id, r, c);
      const float tx = P.t[0] - z * dx, ty = P.t[1] - z * dy, tz = P.t[2] - z;
      const float s = g / nd;
      acc[0] += (double)(s * nn.x);
      acc[1] += (double)(s * nn.y);
      acc[2] += (double)(s * nn.z);
      acc[3] += (double)(s * (nn.y * tz - nn.z * ty));
      acc[4] += (double)(s * (nn.z * tx - nn.x * tz));
      acc[5] += (double)(s * (nn.x * ty - nn.y * tx));
    }
  };
  auto push = [&](bool drawn, int p) {
    const unsigned long long mask = __ballot(drawn);
    if (mask == 0ull) return;
    if (drawn) q[(head + fill + lanes_below(mask)) & (kWaveQueue - 1)] = p;
    fill += __popcll(mask);
    drain(64);
  };
  if constexpr (VEC) {
    const int4* t4 = reinterpret_cast<const int4*>(tn);
    const int nq = HW / 4;
    constexpr int kTurn = 4;
    for (int base = wave * 64; base < nq; base += kTurn * kBlock) {
      int4 v[kTurn];
#pragma unroll
      for (int u = 0; u < kTurn; ++u) v[u] = t4[min(base + u * kBlock + lane, nq - 1)];
#pragma unroll
      for (int u = 0; u < kTurn; ++u) {
        const int w = base + u * kBlock + lane;
        const bool in = w < nq;
        auto drawn = [&](int id) { return in && (unsigned)id < (unsigned)m.T; };
        if (__ballot(drawn(v[u].x) || drawn(v[u].y) || drawn(v[u].z) || drawn(v[u].w)) == 0ull) continue;
        push(drawn(v[u].x), 4 * w);
        push(drawn(v[u].y), 4 * w + 1);
        push(drawn(v[u].z), 4 * w + 2);
        push(drawn(v[u].w), 4 * w + 3);
      }
    }
  } else {
    for (int base = wave * 64; base < HW; base += kBlock) {
      const int p = base + lane;
      push(p < HW && (unsigned)tn[min(p, HW - 1)] < (unsigned)m.T, p);
    }
  }
  drain(1);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double v = wave_sum(acc[k]);
    if (lane == 0) red[wave * 6 + k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    double t = red[threadIdx.x];
    for (int w = 1; w < kWaves; ++w) t += red[w * 6 + threadIdx.x];
    d_pose[6 * (size_t)n + threadIdx.x] = (float)t;
  }
}

hipError_t launch_render_backward(const MeshDev& m, const Cam& cam, const float* poses, int N, const int* tri,
                                  const float* d_rend, float* d_pose, hipStream_t st) {
  const bool vec = (cam.H * cam.W) % 4 == 0 && ((uintptr_t)tri & 15) == 0;
  hipLaunchKernelGGL((vec ? k_render_backward<true> : k_render_backward<false>), dim3(N), dim3(kBlock), 0, st, m, cam,
                     poses, N, tri, d_rend, d_pose);
  return hipGetLastError();
}

__global__ void k_fill_keys(unsigned long long* keys, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    keys[i] = kEmptyKey;
}

hipError_t launch_fill_keys(unsigned long long* keys, size_t n, hipStream_t st) {
  const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(k_fill_keys, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, st, keys, n);
  return hipGetLastError();
}

// The static objects drawn into a full-image key buffer with global 64-bit
// atomicMin: mesh blockIdx.z, one lane per triangle.  A lane walks a small box
// itself; a box of more than kBigCentres centres (a table top, a wall) is walked
// by its whole wave, and for meshes with large primitives the rows of such
// boxes are dealt over kRasterSlices blocks, so that a triangle that spans the
// image does not serialise on one thread (with the rows dealt over blocks but
// one thread per row, a table top at 320x240 took 240 us).  The minimum does
// not depend on the order.
constexpr int kRasterSlices = 32;

__global__ __launch_bounds__(256) void k_raster_statics(StaticsDev G, Cam cam, unsigned long long* keys) {
  const MeshDev m = G.m[blockIdx.z];
  const int slice = blockIdx.y, slices = m.has_big ? kRasterSlices : 1;
  if (slice >= slices || (int)blockIdx.x * 256 >= m.T) return;
  const uint32_t id_base = G.id_base[blockIdx.z];
  const Pose P = G.dev_pose[blockIdx.z] ? load_pose(G.dev_pose[blockIdx.z]) : G.pose[blockIdx.z];
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int4 tr = m.tris[min(i, m.T - 1)];
  float u[3], v[3], iz[3], zmin = 3.0e38f;
  const int vi[3] = {tr.x, tr.y, tr.z};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float4 o = m.verts[vi[k]];
    const float3 p = xform(P, o.x, o.y, o.z);
    iz[k] = 1.0f / p.z;
    u[k] = cam.fx * p.x * iz[k] + cam.cx;
    v[k] = cam.fy * p.y * iz[k] + cam.cy;
    zmin = fminf(zmin, p.z);
  }
  const float area = (u[1] - u[0]) * (v[2] - v[0]) - (u[2] - u[0]) * (v[1] - v[0]);
  const float fc0 = ceilf(fmaxf(fminf(u[0], fminf(u[1], u[2])) - 0.5f, 0.0f));
  const float fc1 = floorf(fminf(fmaxf(u[0], fmaxf(u[1], u[2])) - 0.5f, (float)(cam.W - 1)));
  const float fr0 = ceilf(fmaxf(fminf(v[0], fminf(v[1], v[2])) - 0.5f, 0.0f));
  const float fr1 = floorf(fminf(fmaxf(v[0], fmaxf(v[1], v[2])) - 0.5f, (float)(cam.H - 1)));
  const bool draw = i < m.T && zmin > cam.znear && area < 0.0f && fc0 <= fc1 && fr0 <= fr1;
  int box[4] = {0, -1, 0, -1};
  if (draw) {
    box[0] = (int)fc0;
    box[1] = (int)fc1;
    box[2] = (int)fr0;
    box[3] = (int)fr1;
  }
  const float inv_area = 1.0f / area;
  auto centre = [&](int r, int c, uint32_t id, const float(&a)[3], const float(&b)[3], const float(&w)[3], float ia) {
    const float py = (float)r + 0.5f, px = (float)c + 0.5f;
    const float e0x = a[2] - a[1], e0y = b[2] - b[1];
    const float e1x = a[0] - a[2], e1y = b[0] - b[2];
    const float e2x = a[1] - a[0], e2y = b[1] - b[0];
    const float w0 = e0x * (py - b[1]) - e0y * (px - a[1]);
    const float w1 = e1x * (py - b[2]) - e1y * (px - a[2]);
    const float w2 = e2x * (py - b[0]) - e2y * (px - a[0]);
    if (w0 > 0.0f || w1 > 0.0f || w2 > 0.0f) return;
    const float z = __builtin_amdgcn_rcpf((w0 * w[0] + w1 * w[1] + w2 * w[2]) * ia);
    if (!(z > 0.0f)) return;
    atomicMin(&keys[(size_t)r * cam.W + c], pack_key(z, id));
  };
  const bool large = (box[1] - box[0] + 1) * (box[3] - box[2] + 1) > kBigCentres;
  if (slice == 0 && !large)
    for (int r = box[2]; r <= box[3]; ++r)
      for (int c = box[0]; c <= box[1]; ++c) centre(r, c, id_base + (uint32_t)i, u, v, iz, inv_area);
  unsigned long long left = __ballot(large);
  while (left != 0ull) {
    const int b = __ffsll(left) - 1;
    left &= left - 1ull;
    float bu[3], bv[3], bw[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      bu[k] = __shfl(u[k], b, 64);
      bv[k] = __shfl(v[k], b, 64);
      bw[k] = __shfl(iz[k], b, 64);
    }
    const float bi = __shfl(inv_area, b, 64);
    const int c0 = __shfl(box[0], b, 64), c1 = __shfl(box[1], b, 64);
    const int q0 = __shfl(box[2], b, 64), q1 = __shfl(box[3], b, 64);
    const uint32_t id = id_base + (uint32_t)(i - lane + b);
    for (int r = q0 + slice; r <= q1; r += slices)
      for (int c = c0 + lane; c <= c1; c += 64) centre(r, c, id, bu, bv, bw, bi);
  }
}

// Exact plane depth for every pixel of a full-image key buffer drawn by one of
// these meshes (see plane_depth).
__global__ void k_refine_statics(StaticsDev G, Cam cam, unsigned long long* keys) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= cam.H * cam.W) return;
  const unsigned long long key = keys[p];
  if (key == kEmptyKey) return;
  for (int j = 0; j < G.n; ++j) {
    const uint32_t id = key_id(key) - G.id_base[j];
    if (id >= (uint32_t)G.m[j].T) continue;
    const Pose Q = G.dev_pose[j] ? load_pose(G.dev_pose[j]) : G.pose[j];
    const int r = p / cam.W, c = p - r * cam.W;
    keys[p] = pack_key(plane_depth(G.m[j], plane_view(Q, cam), id, r, c), key_id(key));
  }
}

hipError_t launch_raster_statics(const StaticsDev& G, const Cam& cam, unsigned long long* keys, hipStream_t st) {
  int T = 1, slices = 1;
  for (int j = 0; j < G.n; ++j) {
    T = max(T, G.m[j].T);
    if (G.m[j].has_big) slices = kRasterSlices;
  }
  hipLaunchKernelGGL(k_raster_statics, dim3((T + 255) / 256, slices, G.n), dim3(256), 0, st, G, cam, keys);
  return hipGetLastError();
}

hipError_t launch_refine_statics(const StaticsDev& G, const Cam& cam, unsigned long long* keys, hipStream_t st) {
  hipLaunchKernelGGL(k_refine_statics, dim3((cam.H * cam.W + 255) / 256), dim3(256), 0, st, G, cam, keys);
  return hipGetLastError();
}

}  // namespace b3d
