// Fused render + windowed likelihood (+ adjoint), one workgroup per pose
// hypothesis.  Nothing but the per-hypothesis results leaves the CU:
//   1. the object's conservative pixel rectangle under the pose is found;
//   2. an LDS depth/id buffer covering that rectangle plus twice the window
//      half-width is initialised from the static background and the mesh is
//      rasterised into it (cluster by cluster, a primitive per lane, 64-bit
//      atomicMin on packed (depth, id) keys);
//   3. every observed pixel whose window can see the object evaluates eq. (1)
//      over its window, reading rendered depths from LDS and turning them into
//      points on their pixel rays;
//   4. (adjoint) the window weights b/L_i are kept in LDS and every object
//      pixel gathers d logL/d z_j over its window, then maps it through the
//      ray/plane intersection of its triangle onto (dt, dw);
//   5. pixels whose window cannot see the object contribute their
//      background-only terms, read from double-precision summed-area tables.
// When the rectangle does not fit the LDS budget it is left to a second launch
// of larger blocks, or processed in bands of rows, re-rasterising per band.
#include "b3d_launch.hpp"
#include <algorithm>
#include <type_traits>

namespace b3d {

__device__ __forceinline__ float f_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float f_ln(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }

__device__ __forceinline__ double rect_sum(const double* sat, int W, const Rect& r) {
  if (r.empty()) return 0.0;
  const int p = W + 1;
  return sat[(size_t)r.y1 * p + r.x1] - sat[(size_t)r.y0 * p + r.x1] - sat[(size_t)r.y1 * p + r.x0] +
         sat[(size_t)r.y0 * p + r.x0];
}

// LDS of a block of bs threads: rasteriser scratch (once the depth buffer is
// complete: the window weights and the waves' queues) | depth keys [zcap] |
// plane view (64 floats) | ray tables of columns [-2h, W + 2h) and rows [-2h, H + 2h).
static size_t fused_lds_bytes(const SceneDev& s, int bs, int zcap) {
  return raster_lds_bytes(bs) + sizeof(float) * (64 + s.cam.W + s.cam.H + 8 * s.sc.h) + kFusedBytesPerKey * (size_t)zcap;
}
size_t fused_lds_bytes(const SceneDev& s) { return fused_lds_bytes(s, kBlock, s.zcap); }

// LDS of block_total over nv values (below), which reuses all of the block's.
static size_t total_lds_bytes(int nv, int bs) { return sizeof(double) * (size_t)nv * (bs / 4); }

// Two rows of the widest depth buffer (image width plus 2h each side).
int min_zcap(const SceneDev& s) { return (4 * s.sc.h + 2) * (s.cam.W + 4 * s.sc.h); }

// Bytes beyond these that the adjoint needs: blocks of more than kBlock threads
// keep the window weights in an area of their own, as many as depth keys; and
// the weights of one row and the halo together with the waves' queues exceed
// the scratch for a wide image.
__host__ __device__ __forceinline__ int weight_bytes(int bs, int W, int h) {
  return 4 * (2 * h + 1) * W + 2 * kWaveQueue * (bs / 64);
}
static size_t launch_lds_bytes(const SceneDev& s, int bs, int zcap, bool grad) {
  size_t bytes = fused_lds_bytes(s, bs, zcap);
  if (grad && bs > kBlock) bytes += 4 * (size_t)zcap;
  if (grad && bs == kBlock && weight_bytes(bs, s.cam.W, s.sc.h) > (int)raster_lds_bytes(bs))
    bytes += 2 * kWaveQueue * (bs / 64);
  return std::max(bytes, total_lds_bytes(grad ? 9 : 1, bs));
}

// Sums over the block of NV doubles per thread, in a fixed order: quads of
// lanes, then 16 lanes per value.  Afterwards thread t < 16 NV holds the total
// of value t / 16.  `red`: NV * BS / 4 doubles of LDS.  Whole block; starts
// with a barrier.  (The terms are single precision; summed in double, their
// grouping over threads, bands and block sizes moves a total by parts in 2^50,
// which its rounding to single precision does not show.)
template <int CTRL>
__device__ __forceinline__ double lane_swap(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}

template <int NV, int BS>
__device__ __forceinline__ double block_total(const double (&v)[NV], double* red) {
  static_assert(16 * NV <= BS, "one group of 16 threads per value");
  const int t = threadIdx.x;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double x = v[k];
    x += lane_swap<0xB1>(x);
    x += lane_swap<0x4E>(x);
    if ((t & 3) == 0) red[k * (BS / 4) + (t >> 2)] = x;
  }
  __syncthreads();
  double x = 0.0;
  if (t < 16 * NV) {
    const double* p = red + (t >> 4) * (BS / 4) + (t & 15);
#pragma unroll
    for (int i = 0; i < BS / 64; ++i) x += p[16 * i];
  }
  x += lane_swap<0xB1>(x);
  x += lane_swap<0x4E>(x);
  x += lane_swap<0x141>(x);
  x += lane_swap<0x140>(x);
  return x;
}

// Window sums for observed point (ox, oy, oz) at pixel (r, c) over the LDS
// depth rectangle L (pitch lw), which holds the whole window (positions
// outside the image are empty slots): S = sum_j exp(-D_ij/(2 sigma^2)) and
// T = sum_j exp(-D_ij/(2 sigma^2)) D_ij over the rendered points of the
// window.  HH > 0: the window half-width known at compile time, each row
// unrolled and branch-free: an empty slot's far depth makes its term exactly 0.
// With the adjoint the rows of windows up to 5 x 5 are unrolled as well (397
// against 400 us for 5,000 hypotheses at 160x120; without it that costs 2 %: 529
// against 519 us for 729 of a solid mesh at 200x200, by its instructions alone).
// HH = 0: any h.  From 7 x 7 on the terms of empty slots are selected away
// instead, so that an observed point at infinity beside the object adds 0 and
// not infinity times 0.  A loop that branches around empty slots is bound by
// the latency of one pair after the other: 2,000 hypotheses at 160x120 with 11 x
// 11 windows take 363 us without the branch against 509 us, 3,000 with 7 x 7
// windows and the adjoint 477 us against 660 us.
template <int HH, bool GRAD, bool COUNT>
__device__ __forceinline__ void window_sums(const unsigned long long* __restrict__ zbuf, const Rect& L, int lw,
                                            const float* __restrict__ dxt, const float* __restrict__ dyt, int r,
                                            int c, int h, float ox, float oy, float oz, float c2, float& S, float& T,
                                            unsigned& pairs) {
  S = 0.0f;
  T = 0.0f;
  if (HH > 0) {
    constexpr int n = 2 * HH + 1;
    float dxs[n];
#pragma unroll
    for (int k = 0; k < n; ++k) dxs[k] = dxt[c - HH + k];
    const unsigned long long* zr = zbuf + (r - HH - L.y0) * lw + (c - HH - L.x0);
#pragma unroll (GRAD && HH < 3 ? 2 * HH + 1 : 1)
    for (int j = 0; j < n; ++j, zr += lw) {
      const float dy = dyt[r - HH + j];
#pragma unroll
      for (int k = 0; k < n; ++k) {
        const unsigned long long key = zr[k];
        const float z = key_depth(key);
        const float ex = ox - z * dxs[k], ey = oy - z * dy, ez = oz - z;
        const float D = ex * ex + ey * ey + ez * ez;
        const float e = f_exp2(-D * c2);
        const bool drawn = z != key_depth(kEmptyKey);
        S += HH < 3 || drawn ? e : 0.0f;
        if (GRAD) T += HH < 3 || drawn ? e * D : 0.0f;
        if (COUNT) pairs += drawn ? 1u : 0u;
      }
    }
  } else {
    const int n = 2 * h + 1;
    const float* dxw = dxt + c - h;
    const float* dyw = dyt + r - h;
    const unsigned long long* zr = zbuf + (r - h - L.y0) * lw + (c - h - L.x0);
#pragma unroll 1
    for (int j = 0; j < n; ++j, zr += lw) {
      const float dy = dyw[j];
#pragma unroll 4
      for (int k = 0; k < n; ++k) {
        const unsigned long long key = zr[k];
        const float z = key_depth(key);
        const bool drawn = z != key_depth(kEmptyKey);
        const float ex = ox - z * dxw[k], ey = oy - z * dy, ez = oz - z;
        const float D = ex * ex + ey * ey + ez * ez;
        const float e = f_exp2(-D * c2);
        S += drawn ? e : 0.0f;
        if (GRAD) T += drawn ? e * D : 0.0f;
        if (COUNT) pairs += drawn ? 1u : 0u;
      }
    }
  }
}

// d logL / d z_j of an object pixel (r, c) with point q = z (dx, dy, 1):
// sum over observed i in its window of w_i exp(-D_ij/(2 sigma^2)) (q~_i - q).d,
// with w_i = b/L_i from the LDS buffer of observed rows [wa, ...) and region
// columns (0 for invalid observed pixels).  Returns the sum before the
// 1/sigma^2 factor.  HH > 0: the half-width known at compile time, for windows
// inside the weights' rows and the region's columns (every pixel away from the
// image border), each row unrolled; the rest, and HH = 0, in a loop over the
// clipped window.  A weight of 0 adds nothing, whatever the point it belongs to,
// but in 3 x 3 and 5 x 5 windows off the border, whose terms are not selected: x
// and y of a pixel without a measurement have to be finite there.
// Border rows unrolled with clamped columns took 96 bytes of spilled registers
// a thread against 28, and 408 us against 398 us for 5,000 hypotheses at 160x120
// with 5 x 5 windows.
template <int HH>
__device__ __forceinline__ float window_grad(const float* __restrict__ wbuf, int wa, int wb, const Rect& region,
                                             const float* __restrict__ obs, int W, int r, int c, int h, float qx,
                                             float qy, float qz, float dx, float dy, float c2) {
  const int rw = region.w();
  float g = 0.0f;
  if (HH > 0) {
    constexpr int n = 2 * HH + 1;
    if (r - HH >= wa && r + HH < wb && c - HH >= region.x0 && c + HH < region.x1) {
      const float* wr = wbuf + (r - HH - wa) * rw + (c - HH - region.x0);
      const float* orow = obs + 3 * ((size_t)(r - HH) * W + (c - HH));
#pragma unroll 1
      for (int j = 0; j < n; ++j, wr += rw, orow += 3 * (size_t)W) {
#pragma unroll
        for (int k = 0; k < n; ++k) {
          const float wv = wr[k];
          const float* q = orow + 3 * k;
          const float ex = q[0] - qx, ey = q[1] - qy, ez = q[2] - qz;
          const float e = f_exp2(-(ex * ex + ey * ey + ez * ez) * c2);
          const float v = wv * e * __builtin_fmaf(ex, dx, __builtin_fmaf(ey, dy, ez));
          g += HH < 3 || wv != 0.0f ? v : 0.0f;
        }
      }
      return g;
    }
  }
  const int r0 = max(r - h, wa), r1 = min(r + h, wb - 1);
  const int c0 = max(c - h, region.x0), c1 = min(c + h, region.x1 - 1);
  for (int ri = r0; ri <= r1; ++ri) {
    const float* wr = wbuf + (ri - wa) * rw - region.x0;
#pragma unroll 4
    for (int ci = c0; ci <= c1; ++ci) {
      const float wv = wr[ci];
      const float* q = obs + 3 * ((size_t)ri * W + ci);
      const float ex = q[0] - qx, ey = q[1] - qy, ez = q[2] - qz;
      const float e = f_exp2(-(ex * ex + ey * ey + ez * ez) * c2);
      const float v = wv * e * __builtin_fmaf(ex, dx, __builtin_fmaf(ey, dy, ez));
      g += wv != 0.0f ? v : 0.0f;
    }
  }
  return g;
}

// The depth buffer of one band: the LDS rectangle L (pitch L.w(), rows and
// columns possibly beyond the image, which stay empty) initialised from the
// background keys, the mesh rasterised into its image part, then the depth of
// every slot the mesh drew recomputed on its triangle's plane.  Whole block.
template <bool COUNT, int RM, int BS>
__device__ __forceinline__ void raster_band(const SceneDev& s, const Pose& P, const Rect& L,
                                            unsigned long long* zbuf, unsigned char* smem, unsigned* cnt) {
  const PlaneView* view = reinterpret_cast<const PlaneView*>(zbuf + s.zcap);
  const Cam& cam = s.cam;
  const int H = cam.H, W = cam.W, lw = L.w();
  const int nk = L.h() * lw;
  const float inv_lw = 1.0f / (float)lw;
  if (s.bg) {
    for (int k = threadIdx.x; k < nk; k += BS) {
      int r, c;
      row_col(k, lw, inv_lw, r, c);
      r += L.y0;
      c += L.x0;
      const bool in = r >= 0 && r < H && c >= 0 && c < W;
      zbuf[k] = in ? s.bg[(size_t)r * W + c] : kEmptyKey;
    }
  } else {
    ulonglong2* z2 = reinterpret_cast<ulonglong2*>(zbuf);
    for (int k = threadIdx.x; k < nk / 2; k += BS) z2[k] = make_ulonglong2(kEmptyKey, kEmptyKey);
    if ((nk & 1) && threadIdx.x == 0) zbuf[nk - 1] = kEmptyKey;
  }
  __syncthreads();
  raster_mesh_mode<COUNT, RM, BS>(s.mesh, P, cam, 0u, grow_clip(L, 0, W, H), L, zbuf, carve_raster_lds<BS>(smem), view,
                                  cnt);
  // the slots this mesh drew, compacted wave by wave (their queues in the free
  // scratch): their depths on the triangles' planes
  const uint32_t T = (uint32_t)s.mesh.T;
  wave_compacted<BS / 64>(
      nk, reinterpret_cast<unsigned short*>(smem) + (threadIdx.x >> 6) * kWaveQueue,
      [&](int k) { return key_id(zbuf[k]) < T; },
      [&](int k, bool act) {
        if (!act) return;
        const unsigned long long key = zbuf[k];
        int r, c;
        row_col(k, lw, inv_lw, r, c);
        zbuf[k] = pack_key(plane_depth(s.mesh, *view, key_id(key), L.y0 + r, L.x0 + c), key_id(key));
      });
  __syncthreads();
}

// One hypothesis: pose16 (16 floats), writes *logL_out and, when GRAD,
// grad_out[0..8).  DEFER: one whose depth buffer exceeds the block's writes
// kDeferred instead, and nothing else.  Must be called by the whole block of BS
// threads; `smem` is at least the fused LDS size for BS and s.zcap.  Threads of
// several waves write the results, with no barrier after them: a block that
// goes on to read them needs one first.
// What bounds it is VALU issue (about 90 % of the issue slots at 5,000
// hypotheses of 160x120); so work common to the block is shared between lanes,
// the observed pixels without a point (44 % of the region there) and the slots
// the mesh did not draw are compacted away inside each wave, and terms are
// summed in double, which leaves the assignment of pixels to lanes free.  (5,000
// hypotheses of 2,000 voxels at 160x120 with the adjoint: 400 us against 429
// with every wave computing the block's bounds, block-wide lists and one lane
// per observed pixel.)
template <bool GRAD, bool COUNT = false, int RM = kRasterAny, int BS = kBlock, bool DEFER = false>
__device__ __forceinline__ void render_score_one(const SceneDev& s, const float* __restrict__ pose16,
                                                 float* __restrict__ logL_out, float* __restrict__ grad_out,
                                                 unsigned char* smem, unsigned* cnt = nullptr, int row_lo = -1,
                                                 int row_hi = -1) {
  static_assert(kPlaneViewBytes <= 64 * sizeof(float), "the plane view's share of LDS");
  constexpr int kScratch = (int)raster_lds_bytes(BS), NW = BS / 64, NV = GRAD ? 9 : 1;
  unsigned c_pair = 0, c_obs = 0, c_adj = 0;
  constexpr bool kOwnWeights = GRAD && BS > kBlock;
  unsigned long long* zbuf = reinterpret_cast<unsigned long long*>(smem + kScratch);

  const Cam& cam = s.cam;
  const ScoreConsts& sc = s.sc;
  const int H = cam.H, W = cam.W, h = sc.h;
  // ray tables indexed by column in [-2h, W + 2h) and row in [-2h, H + 2h)
  float* dxt = reinterpret_cast<float*>(zbuf + s.zcap) + 64 + 2 * h;
  float* dyt = dxt + W + 4 * h;
  const Pose P = load_pose(pose16);
  const Rect obj = object_rect(s.mesh, P, cam);
  if (DEFER && (obj.w() + 4 * h) * (obj.h() + 4 * h) > s.zcap) {
    if (threadIdx.x == 0) *logL_out = __uint_as_float(kDeferred);
    return;
  }
  for (int i = (int)threadIdx.x - 2 * h; i < W + 2 * h; i += BS) dxt[i] = ray_x(cam, i);
  for (int i = (int)threadIdx.x - 2 * h; i < H + 2 * h; i += BS) dyt[i] = ray_y(cam, i);
  if (threadIdx.x == BS - 1) *reinterpret_cast<PlaneView*>(zbuf + s.zcap) = plane_view(P, cam);
  // observed pixels whose window can see the object (none when nothing is drawn)
  Rect region = grow_clip(obj, h, W, H);
  if (obj.empty()) region.x1 = region.x0;
  // acc: l, d(dt) x3, d(dw) x3, d sigma, d p_out
  double acc[NV] = {};
  if (!obj.empty()) {
    // the depth buffer spans the object rectangle grown by 2h, past the image
    // edges if need be (those slots stay empty), so every window is inside it
    const Rect lds = grow(obj, 2 * h);
    const int lw = lds.w(), rw = region.w();
    const int ow = obj.w();
    int band = s.zcap / lw - 4 * h;
    // the queues of the waves, in the scratch after the window weights ((band +
    // 2h) x rw floats), or after everything for an image that leaves no room
    constexpr int kQueues = 2 * kWaveQueue * NW;
    const bool wide = GRAD && !kOwnWeights && weight_bytes(BS, W, h) > kScratch;
    float* wbuf = kOwnWeights ? dyt + H + 2 * h : reinterpret_cast<float*>(smem);  // once the band is drawn
    unsigned short* queue = reinterpret_cast<unsigned short*>(
                                wide ? reinterpret_cast<unsigned char*>(dyt + H + 2 * h) : smem + kScratch - kQueues) +
                            kWaveQueue * ((int)threadIdx.x >> 6);
    if (GRAD) band = min(band, (kOwnWeights ? s.zcap : (kScratch - (wide ? 0 : kQueues)) / 4) / rw - 2 * h);
    band = max(band, 1);
    // with a row range: only the region's rows in [row_lo, row_hi) (the
    // adjoint's weights still span the whole region's halo rows)
    const int ya = row_lo >= 0 ? max(region.y0, row_lo) : region.y0;
    const int yb = row_lo >= 0 ? min(region.y1, row_hi) : region.y1;
    for (int a = ya; a < yb; a += band) {
      const int b = min(a + band, yb);
      Rect L = lds;
      L.y0 = a - 2 * h;
      L.y1 = b + 2 * h;
      raster_band<COUNT, RM, BS>(s, P, L, zbuf, smem, cnt);
      // likelihood over observed rows [wa, wb); rows [a, b) are this band's own
      const int wa = GRAD ? max(a - h, region.y0) : a;
      const int wb = GRAD ? min(b + h, region.y1) : b;
      const int nw = (wb - wa) * rw;
      const float inv_rw = 1.0f / (float)rw;
      wave_compacted<NW>(
          nw, queue,
          [&](int k) {
            int r, c;
            row_col(k, rw, inv_rw, r, c);
            const bool valid = s.obs[3 * ((size_t)(wa + r) * W + (region.x0 + c)) + 2] > 0.0f;
            if (GRAD && !valid) wbuf[k] = 0.0f;
            return valid;
          },
          [&](int k, bool act) {
            if (!act) return;
            int r, c;
            row_col(k, rw, inv_rw, r, c);
            r += wa;
            c += region.x0;
            const float* q = s.obs + 3 * ((size_t)r * W + c);
            const float ox = q[0], oy = q[1], oz = q[2];
            float S, T;
            unsigned pairs = 0;
            switch (h) {
              case 1:
                window_sums<1, GRAD, COUNT>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, sc.c2, S, T, pairs);
                break;
              case 2:
                window_sums<2, GRAD, COUNT>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, sc.c2, S, T, pairs);
                break;
              case 3:
                window_sums<3, GRAD, COUNT>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, sc.c2, S, T, pairs);
                break;
              default:
                window_sums<0, GRAD, COUNT>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, sc.c2, S, T, pairs);
            }
            if (COUNT && r >= a && r < b) c_pair += pairs;
            const float Li = sc.a + sc.bn * S;
            const float iL = __builtin_amdgcn_rcpf(Li);  // 1 / L_i, hardware reciprocal (1 ulp)
            const float bL = sc.bn * iL;
            if (r >= a && r < b) {
              if (COUNT && S > 0.0f) ++c_obs;
              acc[0] += (double)f_ln(Li);
              if constexpr (GRAD) {
                acc[7] += (double)(bL * (T * sc.inv_s3 - 3.0f * S * sc.inv_s));
                acc[8] += (double)((sc.invV - sc.normM * S) * iL);
              }
            }
            if (GRAD) wbuf[k] = bL;
          });

      if constexpr (GRAD) {
        __syncthreads();
        // the drawn pixels of this band's own rows: d logL / d z_j over the
        // window, onto (dt, dw)
        const int ga = max(a, obj.y0), gb = min(b, obj.y1);
        const float inv_ow = 1.0f / (float)ow;
        wave_compacted<NW>(
            max(gb - ga, 0) * ow, queue,
            [&](int k) {
              int r, c;
              row_col(k, ow, inv_ow, r, c);
              return key_id(zbuf[(ga + r - L.y0) * lw + (obj.x0 + c - L.x0)]) < (uint32_t)s.mesh.T;
            },
            [&](int k, bool act) {
              if (!act) return;
              int r, c;
              row_col(k, ow, inv_ow, r, c);
              r += ga;
              c += obj.x0;
              const unsigned long long key = zbuf[(r - L.y0) * lw + (c - L.x0)];
              const uint32_t id = key_id(key);
              if (COUNT) ++c_adj;
              const float z = key_depth(key);
              const float dx = dxt[c], dy = dyt[r];
              const float qx = z * dx, qy = z * dy, qz = z;
              float g;
              switch (h) {
                case 1:
                  g = window_grad<1>(wbuf, wa, wb, region, s.obs, W, r, c, h, qx, qy, qz, dx, dy, sc.c2);
                  break;
                case 2:
                  g = window_grad<2>(wbuf, wa, wb, region, s.obs, W, r, c, h, qx, qy, qz, dx, dy, sc.c2);
                  break;
                case 3:
                  g = window_grad<3>(wbuf, wa, wb, region, s.obs, W, r, c, h, qx, qy, qz, dx, dy, sc.c2);
                  break;
                default:
                  g = window_grad<0>(wbuf, wa, wb, region, s.obs, W, r, c, h, qx, qy, qz, dx, dy, sc.c2);
              }
              g *= sc.inv_s2;
              const float4 no = s.mesh.normals[id];
              const float3 nn = rotate(P, no.x, no.y, no.z);
              const float sg = g * __builtin_amdgcn_rcpf(nn.x * dx + nn.y * dy + nn.z);
              const float tx = P.t[0] - qx, ty = P.t[1] - qy, tz = P.t[2] - qz;
              acc[1] += (double)(sg * nn.x);
              acc[2] += (double)(sg * nn.y);
              acc[3] += (double)(sg * nn.z);
              acc[4] += (double)(sg * (nn.y * tz - nn.z * ty));
              acc[5] += (double)(sg * (nn.z * tx - nn.x * tz));
              acc[6] += (double)(sg * (nn.x * ty - nn.y * tx));
            });
      }
      __syncthreads();
    }
  }
  if (COUNT) {
    atomicAdd(&cnt[kCntPair], c_pair);
    atomicAdd(&cnt[kCntObs], c_obs);
    atomicAdd(&cnt[kCntAdj], c_adj);
  }
  // thread 16 k writes value k; the background outside the region (not with a
  // row range) from summed-area tables: l of 0, d sigma of 2, d p_out of 1
  const int k = threadIdx.x >> 4;
  const bool writer = threadIdx.x < 16 * NV && (threadIdx.x & 15) == 0;
  double outside = 0.0;
  if (row_lo < 0 && writer && (k == 0 || k >= 7)) {
    const double* sat = s.sat + (k == 0 ? 0 : k == 7 ? 2 : 1) * ((size_t)(H + 1) * (W + 1));
    Rect all;
    all.x0 = 0;
    all.x1 = W;
    all.y0 = 0;
    all.y1 = H;
    outside = rect_sum(sat, W, all) - rect_sum(sat, W, region);
  }
  const double total = block_total<NV, BS>(acc, reinterpret_cast<double*>(smem)) + outside;
  if (writer) *(k == 0 ? logL_out : grad_out + (k - 1)) = (float)total;
}

// RM: the rasteriser compiled in (the launcher picks it from the mesh, so
// that meshes without large primitives run the plain one alone).
template <bool GRAD, int RM, int BS, int PART>
__global__ __launch_bounds__(BS, 4) void k_render_score(SceneDev s, const float* __restrict__ poses, int N, float* logL,
                                                        float* __restrict__ grad) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = blockIdx.x;
  if (n >= N) return;
  if (PART == kRest && __float_as_uint(logL[n]) != kDeferred) return;
  render_score_one<GRAD, false, RM, BS, PART == kFirst>(s, poses + 16 * (size_t)n, logL + n,
                                                        GRAD ? grad + 8 * (size_t)n : nullptr, smem);
}

static bool defers(const SceneDev& s, long long N) {
  const long long whole = (long long)(s.cam.W + 4 * s.sc.h) * (s.cam.H + 4 * s.sc.h);
  return whole > s.zcap && (s.cam.W * s.cam.H > kBandedPixels || N >= kBandedCount);
}
static int rest_block(const SceneDev& s) { return s.cam.W * s.cam.H > kWholeCuPixels ? 1024 : 512; }

// The scene with the depth buffer that a block of bs > kBlock threads has room
// for, whatever the scene's tile: its share of a CU's LDS, no more than the image
// needs.  False when not even one band fits (the widest images).
static bool roomy_scene(const SceneDev& s, int bs, bool grad, SceneDev* t) {
  *t = s;
  const size_t share = kLdsPerCU / (1024 / bs), rest = fused_lds_bytes(s, bs, 0);
  const int fit = share > rest ? (int)((share - rest) / (kFusedBytesPerKey + (grad ? 4 : 0))) : 0;
  const int whole = (s.cam.W + 4 * s.sc.h) * (s.cam.H + 4 * s.sc.h);
  t->zcap = std::max(min_zcap(s), std::min(fit, whole));
  return launch_lds_bytes(*t, bs, t->zcap, grad) <= kLdsPerCU;
}

// A group of scenes in one launch, one workgroup per (scene, hypothesis)
// item.  Items are numbered scene by scene in the order the host chose
// (costliest hypotheses first), so the expensive scenes start early and the
// cheap ones fill the tail; the hardware dispatcher hands them out in order.
// The item's scene is copied from the argument member by member at constant
// positions: indexing the argument with the scene number would move it to
// scratch memory.  No static LDS either, which would cost a resident block
// per CU at the default tile.
template <bool GRAD, int RM, int BS, int PART>
__global__ __launch_bounds__(BS, 4) void k_batch(const BatchGroupDev G) {
  extern __shared__ __align__(16) unsigned char smem[];
  const long long w = blockIdx.x;
  if (w >= G.first[G.S]) return;
  int k = 0;
  for (int j = 1; j < G.S; ++j) k = G.first[j] <= w ? j : k;
  SceneDev s;
  const float* poses = nullptr;
  float *logL = nullptr, *grad = nullptr;
  long long first = 0;
#pragma unroll
  for (int j = 0; j < kBatchGroup; ++j)
    if (k == j) {
      s = G.s[j];
      poses = G.poses[j];
      logL = G.logL[j];
      grad = G.grad[j];
      first = G.first[j];
    }
  const long long n = w - first;
  if (PART == kRest && __float_as_uint(logL[n]) != kDeferred) return;
  render_score_one<GRAD, false, RM, BS, PART == kFirst>(s, poses + 16 * n, logL + n, GRAD ? grad + 8 * n : nullptr,
                                                        smem);
}

template <int BS, int PART>
static void launch_batch_part(const BatchGroupDev& g, bool grad, bool big, size_t lds, hipStream_t st) {
  auto k = grad ? (big ? k_batch<true, kRasterAny, BS, PART> : k_batch<true, kRasterSmall, BS, PART>)
                : (big ? k_batch<false, kRasterAny, BS, PART> : k_batch<false, kRasterSmall, BS, PART>);
  hipLaunchKernelGGL(k, dim3((unsigned)g.first[g.S]), dim3(BS), lds, st, g);
}

// The group's launch and, when one of its images is large enough for objects
// beyond the tiles (see launch_render_score), a second one for what it leaves.
hipError_t launch_batch(const BatchGroupDev& g, bool grad, size_t lds, hipStream_t st) {
  bool big = false, defer = false, fits = true;
  int bs = 512;
  for (int k = 0; k < g.S; ++k) {
    big = big || g.s[k].mesh.has_big != 0;
    lds = std::max(lds, launch_lds_bytes(g.s[k], kBlock, g.s[k].zcap, grad));
    if (defers(g.s[k], g.first[k + 1] - g.first[k])) {
      defer = true;
      bs = std::max(bs, rest_block(g.s[k]));
    }
  }
  BatchGroupDev rest = g;
  size_t rest_lds = 0;
  for (int k = 0; k < g.S && defer; ++k) {
    fits = fits && roomy_scene(g.s[k], bs, grad, &rest.s[k]);
    rest_lds = std::max(rest_lds, launch_lds_bytes(rest.s[k], bs, rest.s[k].zcap, grad));
  }
  if (defer && fits) {
    launch_batch_part<kBlock, kFirst>(g, grad, big, lds, st);
    if (bs == 1024)
      launch_batch_part<1024, kRest>(rest, grad, big, rest_lds, st);
    else
      launch_batch_part<512, kRest>(rest, grad, big, rest_lds, st);
  } else {
    launch_batch_part<kBlock, kAlone>(g, grad, big, lds, st);
  }
  return hipGetLastError();
}

// n_refine Adam steps on each of N poses of a scene, one workgroup per pose:
// the fused render + score + adjoint, then the update, with the pose kept in
// LDS between steps (the same arithmetic as render_score + adam_pose launched
// in turn, starting from zero moments).
__global__ __launch_bounds__(kBlock) void k_refine_pose(SceneDev s, float* __restrict__ poses, int N, int n_refine,
                                                        float lr_t, float lr_r, float b1, float b2, float eps) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float P[16];
  __shared__ float g[8];
  __shared__ float L;
  const int n = blockIdx.x;
  if (n >= N) return;
  float* pose = poses + 16 * (size_t)n;
  float m[6] = {0, 0, 0, 0, 0, 0}, v[6] = {0, 0, 0, 0, 0, 0};  // used by thread 0
  if (threadIdx.x < 16) P[threadIdx.x] = pose[threadIdx.x];
  __syncthreads();
  for (int it = 1; it <= n_refine; ++it) {
    render_score_one<true>(s, P, &L, g, smem);
    __syncthreads();  // g[3..5] come from the second wave
    if (threadIdx.x == 0) adam_update(P, g, m, v, it, lr_t, lr_r, b1, b2, eps);
    __syncthreads();
  }
  if (threadIdx.x < 16) pose[threadIdx.x] = P[threadIdx.x];
}

hipError_t launch_refine_pose(const SceneDev& s, float* poses, int N, int n_refine, float lr_t, float lr_r, float b1,
                              float b2, float eps, hipStream_t st) {
  hipLaunchKernelGGL(k_refine_pose, dim3(N), dim3(kBlock), launch_lds_bytes(s, kBlock, s.zcap, true), st, s, poses, N, n_refine, lr_t,
                     lr_r, b1, b2, eps);
  return hipGetLastError();
}

// One Adam step of one pose spread over row bands: block b scores the image
// rows [b R, (b + 1) R) of the pose's region (render, windows, adjoint) and
// writes its terms to partial[9 b .. 9 b + 9) (logL, d(dt, dw), d sigma,
// d p_out, without the background outside the region, which the pose
// gradient does not involve).  The block that finishes last (the count of
// finished blocks follows the partial sums and is left at zero) adds the bands
// in band order, in double, and updates the pose; the moments live in
// state[0..12) (zero at iter 1).
// A step is a few dozen blocks on 256 CUs, so it lasts as long as one block:
// 1,024 threads and a depth buffer that holds the band.  (A 160x120 frame's
// step: 36 us; with 256 threads and the update in a launch of its own, 53 + 8.)
constexpr int kBandBlock = 1024;
template <int RM>
__global__ __launch_bounds__(kBandBlock, 4) void k_refine_bands(SceneDev s, float* pose, int R, float* partial,
                                                                float* __restrict__ state, int iter, float lr_t,
                                                                float lr_r, float b1, float b2, float eps) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.x, nb = gridDim.x;
  render_score_one<true, false, RM, kBandBlock>(s, pose, partial + 9 * b, partial + 9 * b + 1, smem, nullptr, b * R,
                                                (b + 1) * R);
  __threadfence();  // each writer's terms, before the count
  __syncthreads();
  unsigned* count = reinterpret_cast<unsigned*>(partial + 9 * nb);
  if (threadIdx.x >= 64) return;
  unsigned done = 0;
  if (threadIdx.x == 0) done = atomicAdd(count, 1u);
  if (__builtin_amdgcn_readfirstlane(done) != (unsigned)nb - 1u) return;
  __threadfence();
  // lane k < 6: the bands of component k in order
  float g = 0.0f;
  if (threadIdx.x < 6) {
    double t = 0.0;
    for (int i = 0; i < nb; ++i)
      t += (double)__hip_atomic_load(partial + 9 * i + 1 + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    g = (float)t;
  }
  float gk[6], m[6], v[6], P[16];
  for (int k = 0; k < 6; ++k) gk[k] = __shfl(g, k, 64);
  if (threadIdx.x != 0) return;
  for (int k = 0; k < 6; ++k) {
    m[k] = iter == 1 ? 0.0f : state[k];
    v[k] = iter == 1 ? 0.0f : state[6 + k];
  }
  for (int k = 0; k < 16; ++k) P[k] = pose[k];
  adam_update(P, gk, m, v, iter, lr_t, lr_r, b1, b2, eps);
  for (int k = 0; k < 16; ++k) pose[k] = P[k];
  for (int k = 0; k < 6; ++k) {
    state[k] = m[k];
    state[6 + k] = v[k];
  }
  *count = 0u;
}

hipError_t launch_refine_banded(const SceneDev& s, float* pose, int n_refine, float lr_t, float lr_r, float b1,
                                float b2, float eps, int R, float* partial, float* state, hipStream_t st) {
  const int nb = (s.cam.H + R - 1) / R, h = s.sc.h;
  // the depth buffer and the weights of R rows at the image's width; the
  // widest images fall back to bands within the block
  SceneDev t = s;
  t.zcap = std::max(min_zcap(s), (R + 4 * h) * (s.cam.W + 4 * h));
  const size_t fixed = launch_lds_bytes(s, kBandBlock, 0, true);
  t.zcap = std::min(t.zcap, (int)((kLdsPerCU - fixed) / (kFusedBytesPerKey + 4)));
  const size_t lds = launch_lds_bytes(t, kBandBlock, t.zcap, true);
  for (int it = 1; it <= n_refine; ++it)
    hipLaunchKernelGGL((s.mesh.has_big ? k_refine_bands<kRasterBig> : k_refine_bands<kRasterSmall>), dim3(nb),
                       dim3(kBandBlock), lds, st, t, pose, R, partial, state, it, lr_t, lr_r, b1, b2, eps);
  return hipGetLastError();
}

// Window sums under each deviation of a noise grid: S[a] = sum_j
// exp(-D_ij c2[a]) over the rendered points of the window of observed point
// (ox, oy, oz) at pixel (r, c) (as window_sums, with each distance computed
// once).  NA > 0: the grid's number of deviations known at compile time (no
// exponential for the unused ones); NA = 0: any number up to kMaxSigma.
template <int HH, int NA>
__device__ __forceinline__ void window_sums_grid(const unsigned long long* __restrict__ zbuf, const Rect& L, int lw,
                                                 const float* __restrict__ dxt, const float* __restrict__ dyt, int r,
                                                 int c, int h, float ox, float oy, float oz, const NoiseGridDev& g,
                                                 float (&S)[kMaxSigma]) {
#pragma unroll
  for (int a = 0; a < kMaxSigma; ++a) S[a] = 0.0f;
  auto add = [&](float D, bool drawn) {
#pragma unroll
    for (int a = 0; a < (NA > 0 ? NA : kMaxSigma); ++a)
      if (NA > 0 || a < g.A) {
        const float e = f_exp2(-D * g.c2[a]);
        S[a] += drawn ? e : 0.0f;
      }
  };
  if (HH > 0) {
    constexpr int n = 2 * HH + 1;
    float dxs[n];
#pragma unroll
    for (int k = 0; k < n; ++k) dxs[k] = dxt[c - HH + k];
    const unsigned long long* zr = zbuf + (r - HH - L.y0) * lw + (c - HH - L.x0);
#pragma unroll 1
    for (int j = 0; j < n; ++j, zr += lw) {
      const float dy = dyt[r - HH + j];
#pragma unroll
      for (int k = 0; k < n; ++k) {
        const float z = key_depth(zr[k]);
        const float ex = ox - z * dxs[k], ey = oy - z * dy, ez = oz - z;
        add(ex * ex + ey * ey + ez * ez, HH < 3 || z != key_depth(kEmptyKey));
      }
    }
  } else {
    const int n = 2 * h + 1;
    const float* dxw = dxt + c - h;
    const float* dyw = dyt + r - h;
    const unsigned long long* zr = zbuf + (r - h - L.y0) * lw + (c - h - L.x0);
#pragma unroll 1
    for (int j = 0; j < n; ++j, zr += lw) {
      const float dy = dyw[j];
#pragma unroll (NA > 0 ? 4 : 1)
      for (int k = 0; k < n; ++k) {
        const float z = key_depth(zr[k]);
        const float ex = ox - z * dxw[k], ey = oy - z * dy, ez = oz - z;
        add(ex * ex + ey * ey + ez * ez, z != key_depth(kEmptyKey));
      }
    }
  }
}

// logL of one hypothesis under every point of the noise grid (grid_out[k],
// k = a * B + b, unless null) and their weighted log-sum-exp (*marg_out).  The
// same render and windows as render_score_one; each observed pixel's window
// distances are computed once and exponentiated per deviation.  With
// row0 >= 0 the block instead scores the full-width image rows [row0, row1)
// (their pixels only, no background table) and grid_out[k] receives the
// block's sum for grid point k; marg_out is not written.  DEFER as for
// render_score_one, the mark in *marg_out.  Whole block of BS threads.
// What bounds it is VALU issue, most of it the windows' exponentials (A per
// pair): so observed pixels without a point are compacted away, and the grid
// points of a deviation are unrolled over registers for up to four deviations
// (NB of them each; more deviations go through LDS, blocks of kBlock only).
// 5,000 hypotheses of 2,000 voxels at 160x120, 4 x 4 points: 491 us against 697
// with one lane per observed pixel and the sums indexed through LDS.
template <int RM, int BS, bool DEFER>
__device__ __forceinline__ void render_score_grid_one(const SceneDev& s, const NoiseGridDev& g,
                                                      const float* __restrict__ pose16, float* __restrict__ grid_out,
                                                      float* __restrict__ marg_out, unsigned char* smem, int row0,
                                                      int row1) {
  constexpr int kScratch = (int)raster_lds_bytes(BS), NW = BS / 64;
  unsigned long long* zbuf = reinterpret_cast<unsigned long long*>(smem + kScratch);
  float* sbuf = reinterpret_cast<float*>(smem);  // NA = 0, per thread: S[a] normM[a] (raster scratch, free by then)
  unsigned short* queue = reinterpret_cast<unsigned short*>(smem + kScratch) - kWaveQueue * (NW - ((int)threadIdx.x >> 6));
  const Cam& cam = s.cam;
  const int H = cam.H, W = cam.W, h = s.sc.h;
  float* dxt = reinterpret_cast<float*>(zbuf + s.zcap) + 64 + 2 * h;
  float* dyt = dxt + W + 4 * h;
  const Pose P = load_pose(pose16);
  const bool rows = row0 >= 0;
  Rect all;
  all.x0 = 0;
  all.x1 = W;
  all.y0 = 0;
  all.y1 = H;
  Rect obj = all;
  if (rows) {
    obj.y0 = row0;
    obj.y1 = row1;
  } else {
    obj = object_rect(s.mesh, P, cam);
  }
  if (DEFER && (obj.w() + 4 * h) * (obj.h() + 4 * h) > s.zcap) {
    if (threadIdx.x == 0) *marg_out = __uint_as_float(kDeferred);
    return;
  }
  for (int i = (int)threadIdx.x - 2 * h; i < W + 2 * h; i += BS) dxt[i] = ray_x(cam, i);
  for (int i = (int)threadIdx.x - 2 * h; i < H + 2 * h; i += BS) dyt[i] = ray_y(cam, i);
  if (threadIdx.x == BS - 1) *reinterpret_cast<PlaneView*>(zbuf + s.zcap) = plane_view(P, cam);
  Rect region = rows ? obj : grow_clip(obj, h, W, H);
  if (obj.empty()) region.x1 = region.x0;
  const int nk_grid = g.A * g.B;
  // the sum of grid point (a, b) in slot a NB + b (NA > 0) or a B + b
  double acc[kMaxNoise] = {};
  int NBs = g.B;
  if (!obj.empty()) {
    const Rect lds = grow(obj, 2 * h);
    const int lw = lds.w(), rw = region.w();
    const int band = max(s.zcap / lw - 4 * h, 1);
    for (int a = region.y0; a < region.y1; a += band) {
      const int b = min(a + band, region.y1);
      Rect L = lds;
      L.y0 = a - 2 * h;
      L.y1 = b + 2 * h;
      raster_band<false, RM, BS>(s, P, L, zbuf, smem, nullptr);
      const float inv_rw = 1.0f / (float)rw;
      // na: the grid's number of deviations as a compile-time constant (0: any)
      auto pixels = [&](auto na) {
        constexpr int NA = decltype(na)::value, NB = NA > 0 ? kMaxNoise / (NA > 0 ? NA : 1) : 1;
        if (NA > 0) NBs = NB;
        wave_compacted<NW>(
            (b - a) * rw, queue,
            [&](int k) {
              int r, c;
              row_col(k, rw, inv_rw, r, c);
              return s.obs[3 * ((size_t)(a + r) * W + (region.x0 + c)) + 2] > 0.0f;
            },
            [&](int k, bool act) {
              if (!act) return;
              int r, c;
              row_col(k, rw, inv_rw, r, c);
              r += a;
              c += region.x0;
              const float* q = s.obs + 3 * ((size_t)r * W + c);
              const float ox = q[0], oy = q[1], oz = q[2];
              float S[kMaxSigma];
              switch (h) {
                case 1:
                  window_sums_grid<1, NA>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, g, S);
                  break;
                case 2:
                  window_sums_grid<2, NA>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, g, S);
                  break;
                case 3:
                  window_sums_grid<3, NA>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, g, S);
                  break;
                default:
                  window_sums_grid<0, NA>(zbuf, L, lw, dxt, dyt, r, c, h, ox, oy, oz, g, S);
              }
              if constexpr (NA > 0) {
#pragma unroll
                for (int ai = 0; ai < NA; ++ai) {
                  const float Sn = S[ai] * g.normM[ai];
#pragma unroll
                  for (int bi = 0; bi < NB; ++bi)
                    if (bi < g.B)
                      acc[ai * NB + bi] += (double)f_ln(g.pa[ai * g.B + bi] + g.pomp[ai * g.B + bi] * Sn);
                }
              } else {
#pragma unroll
                for (int ai = 0; ai < kMaxSigma; ++ai)
                  if (ai < g.A) sbuf[ai * BS + threadIdx.x] = S[ai] * g.normM[ai];
#pragma unroll
                for (int kk = 0; kk < kMaxNoise; ++kk)
                  if (kk < nk_grid)
                    acc[kk] += (double)f_ln(g.pa[kk] + g.pomp[kk] * sbuf[g.ka[kk] * BS + threadIdx.x]);
              }
            });
      };
      switch (g.A) {
        case 1:
          pixels(std::integral_constant<int, 1>{});
          break;
        case 2:
          pixels(std::integral_constant<int, 2>{});
          break;
        case 3:
          pixels(std::integral_constant<int, 3>{});
          break;
        case 4:
          pixels(std::integral_constant<int, 4>{});
          break;
        default:
          if constexpr (BS == kBlock) pixels(std::integral_constant<int, 0>{});
      }
      __syncthreads();
    }
  }
  // thread 16 slot holds a grid point's sum: k and, when it is one, the
  // background outside the region
  const int slot = threadIdx.x >> 4, ka = slot / NBs, kb = slot - ka * NBs;
  const int k = ka * g.B + kb;
  const bool writer = threadIdx.x < 16 * kMaxNoise && (threadIdx.x & 15) == 0 && ka < g.A && kb < g.B;
  double outside = 0.0;
  if (writer && !rows) {
    const double* sat = g.sat + g.sat_stride * k;
    outside = rect_sum(sat, W, all) - rect_sum(sat, W, region);
  }
  double* red = reinterpret_cast<double*>(smem);
  const double v = block_total<kMaxNoise, BS>(acc, red) + outside;
  if (writer && grid_out) grid_out[k] = (float)v;
  if (rows) return;
  double* lse = red + kMaxNoise * (BS / 4);
  if (writer) lse[k] = v + (double)g.logw[k];
  __syncthreads();
  if (threadIdx.x < 64) {  // lanes 0 .. 15 hold the grid points
    const bool has = (int)threadIdx.x < nk_grid;
    const double x = has ? lse[threadIdx.x] : -1e300;
    double m = x;
    for (int o = 8; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    double e = has ? exp(x - m) : 0.0;
    for (int o = 8; o >= 1; o >>= 1) e += __shfl_xor(e, o, 64);
    if (threadIdx.x == 0) *marg_out = (float)(m + log(e));
  }
}

template <int RM, int BS, int PART>
__global__ __launch_bounds__(BS, 4) void k_render_score_grid(SceneDev s, NoiseGridDev g,
                                                             const float* __restrict__ poses, int N,
                                                             float* __restrict__ logL_grid, float* logL_marg) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = blockIdx.x;
  if (n >= N) return;
  if (PART == kRest && __float_as_uint(logL_marg[n]) != kDeferred) return;
  float* gout = logL_grid ? logL_grid + (size_t)g.A * g.B * n : nullptr;
  render_score_grid_one<RM, BS, PART == kFirst>(s, g, poses + 16 * (size_t)n, gout, logL_marg + n, smem, -1, -1);
}

template <int BS, int PART = kAlone>
static void launch_grid_bs(const SceneDev& s, const NoiseGridDev& g, const float* poses, int N, float* logL_grid,
                           float* logL_marg, hipStream_t st) {
  hipLaunchKernelGGL((s.mesh.has_big ? k_render_score_grid<kRasterBig, BS, PART>
                                     : k_render_score_grid<kRasterSmall, BS, PART>),
                     dim3(N), dim3(BS),
                     std::max(fused_lds_bytes(s, BS, s.zcap), total_lds_bytes(kMaxNoise, BS) + kMaxNoise * sizeof(double)),
                     st, s, g, poses, N, logL_grid, logL_marg);
}

// Block sizes as for launch_render_score; more than four deviations need the
// 256-thread block.
hipError_t launch_render_score_grid(const SceneDev& s, const NoiseGridDev& g, const float* poses, int N,
                                    float* logL_grid, float* logL_marg, hipStream_t st) {
  SceneDev t;
  if (g.A > 4) {
    launch_grid_bs<kBlock>(s, g, poses, N, logL_grid, logL_marg, st);
  } else if (N <= kCUs && roomy_scene(s, 1024, false, &t)) {
    launch_grid_bs<1024>(t, g, poses, N, logL_grid, logL_marg, st);
  } else if (N <= 2 * kCUs && roomy_scene(s, 512, false, &t)) {
    launch_grid_bs<512>(t, g, poses, N, logL_grid, logL_marg, st);
  } else if (defers(s, N) && roomy_scene(s, 512, false, &t)) {
    launch_grid_bs<kBlock, kFirst>(s, g, poses, N, logL_grid, logL_marg, st);
    launch_grid_bs<512, kRest>(t, g, poses, N, logL_grid, logL_marg, st);
  } else {
    launch_grid_bs<kBlock>(s, g, poses, N, logL_grid, logL_marg, st);
  }
  return hipGetLastError();
}

// The noise grid of one observation point (sigma, p_out): the constants of
// eq. (1) as the host computes them, in double then rounded.
__device__ NoiseGridDev grid_point(float sigma, float p_out, double inv_V, double M) {
  NoiseGridDev g{};
  const double s = sigma;
  g.A = 1;
  g.B = 1;
  g.c2[0] = (float)(1.0 / (2.0 * s * s) / 0.69314718055994530942);
  g.normM[0] = (float)(pow(2.0 * 3.14159265358979323846 * s * s, -1.5) / M);
  g.ka[0] = 0;
  g.pa[0] = (float)((double)p_out * inv_V);
  g.pomp[0] = (float)(1.0 - (double)p_out);
  g.logw[0] = 0.0f;
  return g;
}

// Block (band b, scene j of the group): full-width rows [b R, (b + 1) R) of
// scene j's image under the group's noise grid, or under the scene's own
// (sigma, p_out) when G.noise[j] is set; per-point sums to
// partial[((G.first + j) n_bands + b) kMaxNoise + k].
__global__ __launch_bounds__(kBlock) void k_score_rows_grid(RowsGroupDev G, int R, int n_bands,
                                                            float* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.x, j = blockIdx.y;
  if (j >= G.S) return;
  const SceneDev& s = G.s[j];
  const int row0 = b * R;
  const int row1 = min(s.cam.H, row0 + R);
  float* out = partial + ((size_t)(G.first + j) * n_bands + b) * kMaxNoise;
  if (row0 >= row1) {
    if (threadIdx.x < kMaxNoise) out[threadIdx.x] = 0.0f;
    return;
  }
  if (G.noise[j]) {
    const NoiseGridDev g = grid_point(G.noise[j][0], G.noise[j][1], G.inv_V, G.M_norm);
    render_score_grid_one<kRasterAny, kBlock, false>(s, g, G.pose[j], out, nullptr, smem, row0, row1);
  } else {
    render_score_grid_one<kRasterAny, kBlock, false>(s, G.grid, G.pose[j], out, nullptr, smem, row0, row1);
  }
}

// One thread per (scene, grid point): the band sums in band order, in
// double; then per scene the log-sum-exp with the grid's log weights.
__global__ void k_reduce_rows_grid(const float* __restrict__ partial, int P, int n_bands, int nk,
                                   NoiseGridDev g, float* __restrict__ grid_out, float* __restrict__ marg_out) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  double v[kMaxNoise], m = -1e300;
  for (int k = 0; k < nk; ++k) {
    double t = 0.0;
    for (int b = 0; b < n_bands; ++b) t += (double)partial[((size_t)p * n_bands + b) * kMaxNoise + k];
    v[k] = t;
    grid_out[(size_t)p * nk + k] = (float)t;
    m = fmax(m, t + (double)g.logw[k]);
  }
  if (marg_out) {
    double t = 0.0;
    for (int k = 0; k < nk; ++k) t += exp(v[k] + (double)g.logw[k] - m);
    marg_out[p] = (float)(m + log(t));
  }
}

hipError_t launch_score_rows_grid(const RowsGroupDev& G, int R, int n_bands, float* partial, hipStream_t st) {
  hipLaunchKernelGGL(k_score_rows_grid, dim3(n_bands, G.S), dim3(kBlock),
                     std::max(fused_lds_bytes(G.s[0]), total_lds_bytes(kMaxNoise, kBlock)), st, G, R, n_bands, partial);
  return hipGetLastError();
}

hipError_t launch_reduce_rows_grid(const float* partial, int P, int n_bands, int nk, const NoiseGridDev& g,
                                   float* grid_out, float* marg_out, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce_rows_grid, dim3((P + 63) / 64), dim3(64), 0, st, partial, P, n_bands, nk, g, grid_out,
                     marg_out);
  return hipGetLastError();
}

// The counting instantiation: same work, plus per-launch totals of the work
// items in work[kCntN] (64-bit, accumulated).
__global__ __launch_bounds__(kBlock) void k_render_score_count(SceneDev s, const float* __restrict__ poses, int N,
                                                               float* __restrict__ logL, float* __restrict__ grad,
                                                               unsigned long long* __restrict__ work) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ unsigned cnt[kCntN];
  const int n = blockIdx.x;
  if (n >= N) return;
  if (threadIdx.x < kCntN) cnt[threadIdx.x] = 0u;
  __syncthreads();
  render_score_one<true, true>(s, poses + 16 * (size_t)n, logL + n, grad + 8 * (size_t)n, smem, cnt);
  __syncthreads();
  if (threadIdx.x < kCntN) atomicAdd(&work[threadIdx.x], (unsigned long long)cnt[threadIdx.x]);
}

hipError_t launch_render_score_count(const SceneDev& s, const float* poses, int N, float* logL, float* grad,
                                     unsigned long long* work, hipStream_t st) {
  hipLaunchKernelGGL(k_render_score_count, dim3(N), dim3(kBlock), launch_lds_bytes(s, kBlock, s.zcap, true), st, s,
                     poses, N, logL, grad, work);
  return hipGetLastError();
}

template <int BS, int PART = kAlone>
static void launch_render_score_bs(const SceneDev& s, const float* poses, int N, float* logL, float* grad,
                                   hipStream_t st) {
  const size_t lds = launch_lds_bytes(s, BS, s.zcap, grad != nullptr);
  const bool big = s.mesh.has_big != 0;
  auto k = grad ? (big ? k_render_score<true, kRasterBig, BS, PART> : k_render_score<true, kRasterSmall, BS, PART>)
                : (big ? k_render_score<false, kRasterBig, BS, PART> : k_render_score<false, kRasterSmall, BS, PART>);
  hipLaunchKernelGGL(k, dim3(N), dim3(BS), lds, st, s, poses, N, logL, grad);
}

bool launch_uses_tile(const SceneDev& s, int N, bool grad) {
  SceneDev t;
  return !(N <= kCUs && roomy_scene(s, 1024, grad, &t)) && !(N <= 2 * kCUs && roomy_scene(s, 512, grad, &t));
}

// One workgroup scores one hypothesis; how large a one is chosen for two
// reasons, and no result depends on it.
// * A launch of fewer hypotheses than the chip has slots lasts as long as one
//   workgroup: up to one hypothesis per CU, each gets all of a CU's sixteen
//   waves and its LDS (256 hypotheses at 64x48: 13.7 against 17.5 us), up to two,
//   half of them.
// * An object beyond the 256-thread block's depth buffer is drawn in bands of
//   rows, each setting the mesh up again.  Such hypotheses are left to a second
//   launch of 512 threads with half a CU's LDS, or all of it where images are
//   large enough for objects beyond that too.  The second launch costs about
//   4 us where nothing is left to it, so small images go without unless there
//   are hypotheses enough to hide that.  (10,000 hypotheses of 1,500 voxels at
//   320x240: 1,835 against 3,091 us.)
//   512 threads for everything cost small objects 11 % (partly filled waves,
//   work that every wave repeats).
hipError_t launch_render_score(const SceneDev& s, const float* poses, int N, float* logL, float* grad,
                               hipStream_t st) {
  const bool g = grad != nullptr;
  SceneDev t;
  if (N <= kCUs && roomy_scene(s, 1024, g, &t)) {
    launch_render_score_bs<1024>(t, poses, N, logL, grad, st);
  } else if (N <= 2 * kCUs && roomy_scene(s, 512, g, &t)) {
    launch_render_score_bs<512>(t, poses, N, logL, grad, st);
  } else if (defers(s, N) && roomy_scene(s, rest_block(s), g, &t)) {
    launch_render_score_bs<kBlock, kFirst>(s, poses, N, logL, grad, st);
    if (rest_block(s) == 1024)
      launch_render_score_bs<1024, kRest>(t, poses, N, logL, grad, st);
    else
      launch_render_score_bs<512, kRest>(t, poses, N, logL, grad, st);
  } else {
    launch_render_score_bs<kBlock>(s, poses, N, logL, grad, st);
  }
  return hipGetLastError();
}

}  // namespace b3d
