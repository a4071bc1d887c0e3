// Split-path likelihood kernels over point images in device memory: the
// windowed robust likelihood of eq. (1) (one workgroup per hypothesis,
// rendered rows staged through LDS with a halo of the window half-width),
// its adjoint, and the per-pixel background terms with their summed-area
// tables used by the fused path.
#include "b3d_launch.hpp"

namespace b3d {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_ln(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }

// Stage rows [y0, y1) of a point image into LDS as three planes, with 16-byte
// loads for the aligned middle of the span.
__device__ __forceinline__ void put_plane(float* sx, float* sy, float* sz, int f, float v) {
  const int p = f / 3, comp = f - 3 * p;
  (comp == 0 ? sx : (comp == 1 ? sy : sz))[p] = v;
}

__device__ __forceinline__ void stage_rows(const float* __restrict__ img, int W, int y0, int y1, float* sx, float* sy,
                                           float* sz) {
  const int nf = (y1 - y0) * W * 3;
  const float* src = img + (size_t)y0 * W * 3;
  const int head = (int)(((16 - ((uintptr_t)src & 15)) & 15) / 4);
  const int h0 = min(head, nf);
  for (int f = threadIdx.x; f < h0; f += kBlock) put_plane(sx, sy, sz, f, src[f]);
  const int nv = (nf - h0) / 4;
  const float4* v4 = reinterpret_cast<const float4*>(src + h0);
  for (int i = threadIdx.x; i < nv; i += kBlock) {
    const float4 v = v4[i];
    const int f = h0 + 4 * i;
    put_plane(sx, sy, sz, f, v.x);
    put_plane(sx, sy, sz, f + 1, v.y);
    put_plane(sx, sy, sz, f + 2, v.z);
    put_plane(sx, sy, sz, f + 3, v.w);
  }
  for (int f = h0 + 4 * nv + threadIdx.x; f < nf; f += kBlock) put_plane(sx, sy, sz, f, src[f]);
}

// Window sums S = sum_j exp2(-D c2) and T = sum_j exp2(-D c2) D of the
// observed point (ox, oy, oz) at pixel (r, c) over staged rows starting at y0
// (rows outside [0, H) and columns outside [0, W) do not exist).  HH > 0:
// half-width known at compile time (rows rolled, columns unrolled,
// predicated); HH = 0: any h.
template <int HH, bool WANT_T>
__device__ __forceinline__ void window_sums(const ScoreConsts& sc, int H, int W, int r, int c, float ox, float oy,
                                            float oz, const float* sx, const float* sy, const float* sz, int y0,
                                            float& S, float& T) {
  S = 0.0f;
  T = 0.0f;
  if (HH > 0) {
    constexpr int n = 2 * HH + 1;
    int cc[n];
    bool cv[n];
#pragma unroll
    for (int k = 0; k < n; ++k) {
      const int cj = c - HH + k;
      cv[k] = cj >= 0 && cj < W;
      cc[k] = min(max(cj, 0), W - 1);
    }
#pragma unroll 1
    for (int j = 0; j < n; ++j) {
      const int rj = r - HH + j;
      if (rj < 0 || rj >= H) continue;
      const int base = (rj - y0) * W;
#pragma unroll
      for (int k = 0; k < n; ++k) {
        const float qz = sz[base + cc[k]];
        const bool ok = cv[k] && qz > 0.0f;
        const float ex = ox - sx[base + cc[k]], ey = oy - sy[base + cc[k]], ez = oz - qz;
        const float D = ok ? ex * ex + ey * ey + ez * ez : 0.0f;
        const float e = ok ? fast_exp2(-D * sc.c2) : 0.0f;
        S += e;
        if (WANT_T) T += e * D;
      }
    }
  } else {
    const int r0 = max(r - sc.h, 0), r1 = min(r + sc.h, H - 1);
    const int c0 = max(c - sc.h, 0), c1 = min(c + sc.h, W - 1);
    for (int rj = r0; rj <= r1; ++rj) {
      const int base = (rj - y0) * W;
      for (int cj = c0; cj <= c1; ++cj) {
        const float qz = sz[base + cj];
        if (!(qz > 0.0f)) continue;
        const float ex = ox - sx[base + cj], ey = oy - sy[base + cj], ez = oz - qz;
        const float D = ex * ex + ey * ey + ez * ez;
        const float e = fast_exp2(-D * sc.c2);
        S += e;
        if (WANT_T) T += e * D;
      }
    }
  }
}

template <bool WANT_T>
__device__ __forceinline__ void window_sums_h(const ScoreConsts& sc, int H, int W, int r, int c, float ox, float oy,
                                              float oz, const float* sx, const float* sy, const float* sz, int y0,
                                              float& S, float& T) {
  switch (sc.h) {
    case 1:
      window_sums<1, WANT_T>(sc, H, W, r, c, ox, oy, oz, sx, sy, sz, y0, S, T);
      break;
    case 2:
      window_sums<2, WANT_T>(sc, H, W, r, c, ox, oy, oz, sx, sy, sz, y0, S, T);
      break;
    default:
      window_sums<0, WANT_T>(sc, H, W, r, c, ox, oy, oz, sx, sy, sz, y0, S, T);
  }
}

__global__ __launch_bounds__(kBlock) void k_score(const float* __restrict__ obs, const float* __restrict__ rend, int N,
                                                  int H, int W, ScoreConsts sc, float* __restrict__ logL, int cap) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* red = reinterpret_cast<float*>(smem);
  float* sx = red + 64;
  const int n = blockIdx.x;
  if (n >= N) return;
  const float* rn = rend + (size_t)n * H * W * 3;
  const int h = sc.h;
  const int band = max(cap / (3 * W) - 2 * h, 1);
  float acc[1] = {0.0f};
  for (int a = 0; a < H; a += band) {
    const int b = min(a + band, H);
    const int y0 = max(a - h, 0), y1 = min(b + h, H);
    const int np = (y1 - y0) * W;
    float* sy = sx + np;
    float* sz = sy + np;
    stage_rows(rn, W, y0, y1, sx, sy, sz);
    __syncthreads();
    for (int k = threadIdx.x; k < (b - a) * W; k += kBlock) {
      const int r = a + k / W, c = k - (k / W) * W;
      const float* q = obs + 3 * ((size_t)r * W + c);
      const float oz = q[2];
      if (!(oz > 0.0f)) continue;
      float S, T;
      window_sums_h<false>(sc, H, W, r, c, q[0], q[1], oz, sx, sy, sz, y0, S, T);
      acc[0] += fast_ln(sc.a + sc.bn * S);
    }
    __syncthreads();
  }
  block_sum<1>(acc, red);
  if (threadIdx.x == 0) logL[n] = acc[0];
}

hipError_t launch_score(const float* obs, const float* rend, int N, int H, int W, const ScoreConsts& sc, float* logL,
                        int cap, hipStream_t st) {
  const size_t lds = sizeof(float) * (64 + (size_t)cap);
  hipLaunchKernelGGL(k_score, dim3(N), dim3(kBlock), lds, st, obs, rend, N, H, W, sc, logL, cap);
  return hipGetLastError();
}

// Adjoint of k_score.  Per band of output rows [a, b): rendered rows
// [a - 2h, b + 2h) and the weights w_i = (b/L_i) of observed rows
// [a - h, b + h) go to LDS; then every rendered pixel gathers
// sum_i w_i K_ij (q~_i - q_j) / sigma^2 over its window (the window is
// symmetric, so no atomics are needed).
__global__ __launch_bounds__(kBlock) void k_score_backward(const float* __restrict__ obs, const float* __restrict__ rend,
                                                           int N, int H, int W, ScoreConsts sc,
                                                           const float* __restrict__ dlogL, float* __restrict__ d_rend,
                                                           float* __restrict__ d_sigma, float* __restrict__ d_pout,
                                                           int cap) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* red = reinterpret_cast<float*>(smem);
  float* sx = red + 64;
  const int n = blockIdx.x;
  if (n >= N) return;
  const float g = dlogL ? dlogL[n] : 1.0f;
  const float* rn = rend + (size_t)n * H * W * 3;
  float* dn = d_rend ? d_rend + (size_t)n * H * W * 3 : nullptr;
  const int h = sc.h;
  // LDS: 3 planes of (band + 4h) rows and 1 plane of (band + 2h) rows
  const int band = max(cap / (4 * W) - 4 * h, 1);
  float acc[2] = {0.0f, 0.0f};  // d/dsigma, d/dp_out
  for (int a = 0; a < H; a += band) {
    const int b = min(a + band, H);
    const int y0 = max(a - 2 * h, 0), y1 = min(b + 2 * h, H);
    const int wa = max(a - h, 0), wb = min(b + h, H);
    const int np = (y1 - y0) * W;
    float* sy = sx + np;
    float* sz = sy + np;
    float* sw = sz + np;
    stage_rows(rn, W, y0, y1, sx, sy, sz);
    __syncthreads();
    for (int k = threadIdx.x; k < (wb - wa) * W; k += kBlock) {
      const int r = wa + k / W, c = k - (k / W) * W;
      const float* q = obs + 3 * ((size_t)r * W + c);
      const float oz = q[2];
      float w = 0.0f;
      if (oz > 0.0f) {
        float S, T;
        window_sums_h<true>(sc, H, W, r, c, q[0], q[1], oz, sx, sy, sz, y0, S, T);
        const float L = sc.a + sc.bn * S;
        w = sc.bn / L;
        if (r >= a && r < b) {
          acc[0] += w * (T * sc.inv_s3 - 3.0f * S * sc.inv_s);
          acc[1] += (sc.invV - sc.normM * S) / L;
        }
      }
      sw[k] = w;
    }
    __syncthreads();
    if (dn) {
      const float scale = g * sc.inv_s2;
      for (int k = threadIdx.x; k < (b - a) * W; k += kBlock) {
        const int r = a + k / W, c = k - (k / W) * W;
        const int pj = (r - y0) * W + c;
        const float qz = sz[pj];
        float gx = 0.0f, gy = 0.0f, gz = 0.0f;
        if (qz > 0.0f) {
          const float qx = sx[pj], qy = sy[pj];
          const int r0 = max(r - h, 0), r1 = min(r + h, H - 1);
          const int c0 = max(c - h, 0), c1 = min(c + h, W - 1);
          for (int ri = r0; ri <= r1; ++ri) {
            for (int ci = c0; ci <= c1; ++ci) {
              const float w = sw[(ri - wa) * W + ci];
              if (w == 0.0f) continue;
              const float* q = obs + 3 * ((size_t)ri * W + ci);
              const float ex = q[0] - qx, ey = q[1] - qy, ez = q[2] - qz;
              const float e = w * fast_exp2(-(ex * ex + ey * ey + ez * ez) * sc.c2);
              gx += e * ex;
              gy += e * ey;
              gz += e * ez;
            }
          }
        }
        float* o = dn + 3 * ((size_t)r * W + c);
        o[0] = gx * scale;
        o[1] = gy * scale;
        o[2] = gz * scale;
      }
    }
    __syncthreads();
  }
  block_sum<2>(acc, red);
  if (threadIdx.x == 0) {
    if (d_sigma) d_sigma[n] = g * acc[0];
    if (d_pout) d_pout[n] = g * acc[1];
  }
}

hipError_t launch_score_backward(const float* obs, const float* rend, int N, int H, int W, const ScoreConsts& sc,
                                 const float* dlogL, float* d_rend, float* d_sigma, float* d_pout, int cap,
                                 hipStream_t st) {
  const size_t lds = sizeof(float) * (64 + (size_t)cap);
  hipLaunchKernelGGL(k_score_backward, dim3(N), dim3(kBlock), lds, st, obs, rend, N, H, W, sc, dlogL, d_rend, d_sigma,
                     d_pout, cap);
  return hipGetLastError();
}

// ---- split path over a ring of rows --------------------------------------
//
// The rendered point image of a hypothesis is streamed from top to bottom
// exactly once: an LDS ring holds, in their stored x, y, z order, the rows a
// window can still reach, and the next R rows are loaded into registers
// (kRingPF 16-byte words per thread) while the current R rows are scored, so
// that the loads stay in flight across the arithmetic and the barriers.  A
// row y sits in slot y mod nrows.  Needs W a multiple of 4 and 16-byte
// aligned images (rows are then whole 16-byte words); the host checks both.

constexpr int kRingPF = 8;  // float4 words per thread per step, score
constexpr int kRingPP = 8;  // output pixels per thread per step, score

typedef float f4v __attribute__((ext_vector_type(4)));

template <int PF>
__device__ __forceinline__ void rows_load(const float* __restrict__ img, int wpr, int y0, int y1, f4v (&v)[PF]) {
  // every lane loads PF words (beyond the span: its last word again), so the
  // registers are written unconditionally; rows_store drops the extra ones
  const int nw = y1 > y0 ? (y1 - y0) * wpr : 0;
  if (nw == 0) return;
  const f4v* src = reinterpret_cast<const f4v*>(img) + (size_t)y0 * wpr;
  const int rounds = (nw + kBlock - 1) / kBlock;  // uniform: whole rounds past the span are skipped
#pragma unroll
  for (int i = 0; i < PF; ++i)
    if (i < rounds) v[i] = src[min((int)threadIdx.x + i * kBlock, nw - 1)];
}

template <int PF>
__device__ __forceinline__ void rows_store(float* ring, int nrows, int wpr, int y0, int y1, const f4v (&v)[PF]) {
  const int nw = y1 > y0 ? (y1 - y0) * wpr : 0;
  if (nw == 0) return;
  f4v* dst = reinterpret_cast<f4v*>(ring);
  // word k = tid + i kBlock of the span sits in row (k / wpr), column (k mod
  // wpr); both advance by fixed amounts from one i to the next
  const int dq = kBlock / wpr, dm = kBlock - dq * wpr;
  int ro = (int)threadIdx.x / wpr;
  int col = (int)threadIdx.x - ro * wpr;
  int slot = (y0 + ro) % nrows;
  const int rounds = (nw + kBlock - 1) / kBlock;
#pragma unroll
  for (int i = 0; i < PF; ++i) {
    if (i >= rounds) break;
    if ((int)threadIdx.x + i * kBlock < nw) dst[slot * wpr + col] = v[i];
    col += dm;
    int carry = dq;
    if (col >= wpr) {
      col -= wpr;
      ++carry;
    }
    slot += carry;
    while (slot >= nrows) slot -= nrows;
  }
}

// Window sums S = sum_j exp2(-D c2) (and T = sum_j exp2(-D c2) D) of the
// observed point o at pixel (r, c) over the rendered rows held in the ring.
template <int HH, bool WANT_T>
__device__ __forceinline__ void window_ring(const ScoreConsts& sc, int H, int W, int nrows, int r, int c, float ox,
                                            float oy, float oz, const float* ring, float& S, float& T) {
  const int h = HH > 0 ? HH : sc.h;
  S = 0.0f;
  T = 0.0f;
  int slot = (r - h + nrows) % nrows;
  if (HH > 0) {
    constexpr int n = 2 * HH + 1;
    int cc[n];
    bool cv[n];
#pragma unroll
    for (int k = 0; k < n; ++k) {
      const int cj = c - HH + k;
      cv[k] = cj >= 0 && cj < W;
      cc[k] = 3 * min(max(cj, 0), W - 1);
    }
#pragma unroll 1
    for (int j = 0; j < n; ++j) {
      const int rj = r - HH + j;
      if (rj >= 0 && rj < H) {
        const float* row = ring + slot * 3 * W;
#pragma unroll
        for (int k = 0; k < n; ++k) {
          const float qz = row[cc[k] + 2];
          const bool ok = cv[k] && qz > 0.0f;
          const float ex = ox - row[cc[k]], ey = oy - row[cc[k] + 1], ez = oz - qz;
          const float D = ok ? ex * ex + ey * ey + ez * ez : 0.0f;
          const float e = ok ? fast_exp2(-D * sc.c2) : 0.0f;
          S += e;
          if (WANT_T) T += e * D;
        }
      }
      slot = slot + 1 == nrows ? 0 : slot + 1;
    }
  } else {
    const int c0 = max(c - h, 0), c1 = min(c + h, W - 1);
    for (int rj = r - h; rj <= r + h; ++rj) {
      if (rj >= 0 && rj < H) {
        const float* row = ring + slot * 3 * W;
        for (int cj = c0; cj <= c1; ++cj) {
          const float qz = row[3 * cj + 2];
          if (!(qz > 0.0f)) continue;
          const float ex = ox - row[3 * cj], ey = oy - row[3 * cj + 1], ez = oz - qz;
          const float D = ex * ex + ey * ey + ez * ez;
          const float e = fast_exp2(-D * sc.c2);
          S += e;
          if (WANT_T) T += e * D;
        }
      }
      slot = slot + 1 == nrows ? 0 : slot + 1;
    }
  }
}

// ---- the observed image's valid pixels, listed once per call -------------
//
// Every hypothesis is scored against the same observed image, so its valid
// pixels (z > 0) are listed once, row-major, in the caller's workspace:
// rows[r] = index of row r's first entry (rows[H] = number of entries),
// list[e] = (x, y, z, pixel index as int bits).  The scoring kernels then
// take only those pixels, densely, instead of every pixel of a row.

__device__ __forceinline__ int block_excl_scan(int v, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;  // inclusive scan within the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  int off = 0, tot = 0;
  for (int w = 0; w < kWaves; ++w) {
    off += w < wave ? wsum[w] : 0;
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return off + x - v;
}

// Block r counts the valid pixels of row r into rows[r + 1].
__global__ __launch_bounds__(kBlock) void k_obs_count(const float* __restrict__ obs, int H, int W, int* rows) {
  __shared__ int wsum[kWaves];
  const int r = blockIdx.x;
  int n = 0;
  for (int c = threadIdx.x; c < W; c += kBlock) n += obs[3 * ((size_t)r * W + c) + 2] > 0.0f ? 1 : 0;
  int total;
  (void)block_excl_scan(n, wsum, &total);
  if (threadIdx.x == 0) rows[r + 1] = total;
  if (r == 0 && threadIdx.x == 0) rows[0] = 0;
}

// One block: rows[1..H] from counts to running totals.
__global__ __launch_bounds__(kBlock) void k_obs_scan(int H, int* rows) {
  __shared__ int wsum[kWaves];
  int carry = 0;
  for (int base = 1; base <= H; base += kBlock) {
    const int r = base + (int)threadIdx.x;
    const int v = r <= H ? rows[r] : 0;
    int total;
    const int ex = block_excl_scan(v, wsum, &total);
    if (r <= H) rows[r] = carry + ex + v;
    carry += total;
  }
}

// Block r writes row r's valid pixels, in column order, from rows[r].
__global__ __launch_bounds__(kBlock) void k_obs_fill(const float* __restrict__ obs, int H, int W,
                                                     const int* __restrict__ rows, float4* __restrict__ list) {
  __shared__ int wsum[kWaves];
  const int r = blockIdx.x;
  int at = rows[r];
  for (int base = 0; base < W; base += kBlock) {
    const int c = base + (int)threadIdx.x;
    const float* q = obs + 3 * ((size_t)r * W + min(c, W - 1));
    const bool v = c < W && q[2] > 0.0f;
    int total;
    const int ex = block_excl_scan(v ? 1 : 0, wsum, &total);
    if (v) list[at + ex] = make_float4(q[0], q[1], q[2], __int_as_float(r * W + c));
    at += total;
  }
}

size_t score_workspace_bytes(int H, int W) {
  return (((size_t)(H + 1) * sizeof(int) + 15) & ~(size_t)15) + sizeof(float4) * (size_t)H * W;
}

hipError_t launch_obs_list(const float* obs, int H, int W, void* workspace, hipStream_t st) {
  int* rows = reinterpret_cast<int*>(workspace);
  float4* list = reinterpret_cast<float4*>(reinterpret_cast<char*>(workspace) +
                                           (((size_t)(H + 1) * sizeof(int) + 15) & ~(size_t)15));
  hipLaunchKernelGGL(k_obs_count, dim3(H), dim3(kBlock), 0, st, obs, H, W, rows);
  hipLaunchKernelGGL(k_obs_scan, dim3(1), dim3(kBlock), 0, st, H, rows);
  hipLaunchKernelGGL(k_obs_fill, dim3(H), dim3(kBlock), 0, st, obs, H, W, rows, list);
  return hipGetLastError();
}

// Entries [e0, e1) of the list into registers, kRingPP per thread at most
// (beyond e1: z = 0, which no step scores).
template <int PP>
__device__ __forceinline__ void entries_load(const float4* __restrict__ list, int e0, int e1, f4v (&v)[PP]) {
  const f4v* src = reinterpret_cast<const f4v*>(list);
  const int rounds = (e1 - e0 + kBlock - 1) / kBlock;  // uniform
#pragma unroll
  for (int i = 0; i < PP; ++i) {
    if (i < rounds) {
      const int e = e0 + (int)threadIdx.x + i * kBlock;
      f4v x = src[min(e, max(e1 - 1, 0))];
      if (e >= e1) x.z = 0.0f;
      v[i] = x;
    }
  }
}

// logL of one hypothesis per workgroup; rows [a, a + R) per step, the ring
// holding rendered rows [a - h, a + R + h), the step's valid observed pixels
// taken from the list, one per lane.
template <int HH>
__global__ __launch_bounds__(kBlock) void k_score_ring(const int* __restrict__ rows, const float4* __restrict__ list,
                                                       const float* __restrict__ rend, int N, int H, int W,
                                                       ScoreConsts sc, int R, float* __restrict__ logL) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* red = reinterpret_cast<float*>(smem);
  float* ring = red + 64;
  const int n = blockIdx.x;
  if (n >= N) return;
  const int h = HH > 0 ? HH : sc.h;
  const int nrows = R + 2 * h, wpr = 3 * W / 4;
  const float* rn = rend + (size_t)n * H * W * 3;
  f4v v[kRingPF], cur[kRingPP];
  rows_load<kRingPF>(rn, wpr, 0, min(h, H), v);
  rows_store<kRingPF>(ring, nrows, wpr, 0, min(h, H), v);
  rows_load<kRingPF>(rn, wpr, min(h, H), min(h + R, H), v);
  float acc[1] = {0.0f};
  for (int a = 0; a < H; a += R) {
    const int ya = min(a + h, H), yb = min(a + R + h, H);
    const int e0 = rows[a], e1 = rows[min(a + R, H)];
    lds_barrier();
    rows_store<kRingPF>(ring, nrows, wpr, ya, yb, v);
    // this step's entries (issued before the next rows, so that waiting for
    // them does not wait for those)
    entries_load<kRingPP>(list, e0, e1, cur);
    lds_barrier();
    rows_load<kRingPF>(rn, wpr, yb, min(yb + R, H), v);  // the next step's rows, in flight while these are scored
    const int rounds = (e1 - e0 + kBlock - 1) / kBlock;
#pragma unroll 1
    for (int i = 0; i < rounds; ++i) {
      const f4v it = cur[0];
#pragma unroll
      for (int t = 0; t + 1 < kRingPP; ++t) cur[t] = cur[t + 1];
      if (it.z > 0.0f) {
        const int p = __float_as_int(it.w);
        const int r = p / W;
        float S, T;
        window_ring<HH, false>(sc, H, W, nrows, r, p - r * W, it.x, it.y, it.z, ring, S, T);
        acc[0] += fast_ln(sc.a + sc.bn * S);
      }
    }
  }
  block_sum<1>(acc, red);
  if (threadIdx.x == 0) logL[n] = acc[0];
}

int score_ring_rows(int H, int W, int h) {
  if (W % 4 != 0) return 0;
  const int wpr = 3 * W / 4;
  int R = std::min(kRingPF * kBlock / wpr, kRingPP * kBlock / W);
  // five workgroups per CU
  while (R > 0 && sizeof(float) * (64 + (size_t)(R + 2 * h) * 3 * W) > 32768) --R;
  if (R < std::max(h, 1)) return 0;  // the prologue loads h rows in one step
  return std::min(R, H);
}

hipError_t launch_score_ring(const float* obs, const float* rend, int N, int H, int W, const ScoreConsts& sc, int R,
                             void* workspace, float* logL, hipStream_t st) {
  if (hipError_t e = launch_obs_list(obs, H, W, workspace, st)) return e;
  const int* rows = reinterpret_cast<const int*>(workspace);
  const float4* list = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(workspace) +
                                                       (((size_t)(H + 1) * sizeof(int) + 15) & ~(size_t)15));
  const size_t lds = sizeof(float) * (64 + (size_t)(R + 2 * sc.h) * 3 * W);
  switch (sc.h) {
    case 1:
      hipLaunchKernelGGL(k_score_ring<1>, dim3(N), dim3(kBlock), lds, st, rows, list, rend, N, H, W, sc, R, logL);
      break;
    case 2:
      hipLaunchKernelGGL(k_score_ring<2>, dim3(N), dim3(kBlock), lds, st, rows, list, rend, N, H, W, sc, R, logL);
      break;
    case 3:
      hipLaunchKernelGGL(k_score_ring<3>, dim3(N), dim3(kBlock), lds, st, rows, list, rend, N, H, W, sc, R, logL);
      break;
    default:
      hipLaunchKernelGGL(k_score_ring<0>, dim3(N), dim3(kBlock), lds, st, rows, list, rend, N, H, W, sc, R, logL);
  }
  return hipGetLastError();
}

// Adjoint of k_score_ring: a workgroup per hypothesis streams its point image
// once (as 16-byte words where it is made of them: VEC), writing the gradient's
// zeros and finding the rectangle of drawn pixels; then the likelihood and its adjoint run over that rectangle
// alone, in LDS, in bands of rows where it does not fit.  Observed pixels whose
// window sees no drawn pixel have no gradient but d/dp_out = 1/p_out each, so
// they are only counted.  What bounds it is the image's traffic (read once,
// written once: 24 bytes a pixel); the rectangle's arithmetic overlaps other
// workgroups' streaming.  (2,000 images of 160x120: 250 us, against 522 for a ring
// of all rows; 300 of 320x240 with a table in most of the image: 1,152 against
// 3,003 with the pose adjoint.  Small images that are full of drawn pixels, in
// great number and with windows up to 3 x 3, are where the ring was faster: 3,000 of
// 64x48, 186 us against 247; mostly empty they take 83 against 142.)
//   LDS: points x | y | z of the band's rendered rows [a - 2h, b + 2h) and of
//   columns [x0 - 2h, x1 + 2h) (an empty or outside slot holds a far point,
//   whose terms are exactly 0), the weights w_i = g b / L_i of observed rows
//   [a - h, b + h), the waves' queues: area_bytes of points and weights, at
//   least what one row and its halo take at the image's width.
constexpr size_t kCropLds = 80 * 1024;  // the most: two workgroups per CU
constexpr size_t crop_fixed_bytes(int bs) {
  return 64 * sizeof(int) + (sizeof(double) * 3 + 2 * kWaveQueue) * (bs / 64);
}
constexpr float kFarPoint = 1.0e15f;

struct CropLds {
  float *px, *py, *pz, *w;
};

// Bytes of one row of a band of lw points and rw weights.
__host__ __device__ __forceinline__ int crop_row_bytes(int lw, int rw) { return 12 * lw + 4 * rw; }

// Sums over the window of the observed point o at band slot (r, c) (row and
// column of the crop).  A point at infinity makes infinity times 0 of an empty
// slot's term: such a pixel's window is gone through again, empty slots skipped.
template <int HH, bool WANT_T>
__device__ __forceinline__ void window_crop(const CropLds& L, int lw, int h, int slot0, float ox, float oy, float oz,
                                            float c2, float& S, float& T) {
  S = 0.0f;
  T = 0.0f;
  const int n = HH > 0 ? 2 * HH + 1 : 2 * h + 1;
  int at = slot0;
#pragma unroll 1
  for (int j = 0; j < n; ++j, at += lw) {
    auto pair = [&](int i) {
      const float ex = ox - L.px[i], ey = oy - L.py[i], ez = oz - L.pz[i];
      const float D = ex * ex + ey * ey + ez * ez;
      const float e = fast_exp2(-D * c2);
      S += e;
      if (WANT_T) T += e * D;
    };
    if constexpr (HH > 0) {
#pragma unroll
      for (int k = 0; k < 2 * HH + 1; ++k) pair(at + k);
    } else {
      for (int k = 0; k < n; ++k) pair(at + k);
    }
  }
  if (WANT_T && T != T) {
    S = T = 0.0f;
    at = slot0;
    for (int j = 0; j < n; ++j, at += lw)
      for (int i = at; i < at + n; ++i)
        if (L.pz[i] != kFarPoint) {
          const float ex = ox - L.px[i], ey = oy - L.py[i], ez = oz - L.pz[i];
          const float D = ex * ex + ey * ey + ez * ez;
          const float e = fast_exp2(-D * c2);
          S += e;
          T += e * D;
        }
  }
}

template <int HH, bool VEC, int BS>
__global__ __launch_bounds__(BS, 4) void k_score_backward_crop(const float* __restrict__ obs,
                                                               const float* __restrict__ rend, int N, int H, int W,
                                                               ScoreConsts sc, const int* __restrict__ rows,
                                                               const float* __restrict__ dlogL,
                                                               float* __restrict__ d_rend, float* __restrict__ d_sigma,
                                                               float* __restrict__ d_pout, int area_bytes) {
  constexpr int kCropWaves = BS / 64;
  constexpr size_t kCropFixed = crop_fixed_bytes(BS);
  extern __shared__ __align__(16) unsigned char smem[];
  int* rect = reinterpret_cast<int*>(smem);  // row and column bounds of the drawn pixels
  double* sums = reinterpret_cast<double*>(rect + 64);
  unsigned short* queue = reinterpret_cast<unsigned short*>(sums + 3 * kCropWaves) + kWaveQueue * (threadIdx.x >> 6);
  float* area = reinterpret_cast<float*>(smem + kCropFixed);
  const int n = blockIdx.x;
  if (n >= N) return;
  const int h = HH > 0 ? HH : sc.h;
  const float g = dlogL ? dlogL[n] : 1.0f;
  const float* rn = rend + (size_t)n * H * W * 3;
  float* dn = d_rend ? d_rend + (size_t)n * H * W * 3 : nullptr;
  if (threadIdx.x < 4) rect[threadIdx.x] = (threadIdx.x & 1) ? -1 : 0x7fffffff;
  __syncthreads();
  // 1. the image once
  int r_lo = 0x7fffffff, r_hi = -1, c_lo = 0x7fffffff, c_hi = -1;
  if constexpr (VEC) {  // quads of pixels as three 16-byte words, four quads a turn
    const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const int qpr = W / 4, nq = H * qpr;
    const f4v* src = reinterpret_cast<const f4v*>(rn);
    f4v* dst = reinterpret_cast<f4v*>(dn);
    constexpr int kTurn = 4;
    for (int base = threadIdx.x; base < nq; base += kTurn * BS) {
      f4v v[kTurn][3];
#pragma unroll
      for (int u = 0; u < kTurn; ++u) {
        const int q = min(base + u * BS, nq - 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) v[u][k] = src[3 * (size_t)q + k];
      }
      if (dn) {
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
          const int q = base + u * BS;
          if (q < nq)
#pragma unroll
            for (int k = 0; k < 3; ++k) dst[3 * (size_t)q + k] = zero;
        }
      }
#pragma unroll
      for (int u = 0; u < kTurn; ++u) {
        const bool d0 = v[u][0].z > 0.0f, d1 = v[u][1].y > 0.0f, d2 = v[u][2].x > 0.0f, d3 = v[u][2].w > 0.0f;
        if (d0 || d1 || d2 || d3) {  // (a quad read twice at the end changes nothing)
          const int q = min(base + u * BS, nq - 1);
          const int r = q / qpr, c = 4 * (q - r * qpr);
          r_lo = min(r_lo, r);
          r_hi = max(r_hi, r);
          c_lo = min(c_lo, c + (d0 ? 0 : d1 ? 1 : d2 ? 2 : 3));
          c_hi = max(c_hi, c + (d3 ? 3 : d2 ? 2 : d1 ? 1 : 0));
        }
      }
    }
  } else {
    const int np = H * W;
    if (dn)
      for (size_t k = threadIdx.x; k < 3 * (size_t)np; k += BS) dn[k] = 0.0f;
#pragma unroll 8
    for (int p = threadIdx.x; p < np; p += BS) {
      if (rn[3 * (size_t)p + 2] > 0.0f) {
        const int r = p / W, c = p - r * W;
        r_lo = min(r_lo, r);
        r_hi = max(r_hi, r);
        c_lo = min(c_lo, c);
        c_hi = max(c_hi, c);
      }
    }
  }
  if (r_hi >= 0) {
    atomicMin(&rect[0], r_lo);
    atomicMax(&rect[1], r_hi);
    atomicMin(&rect[2], c_lo);
    atomicMax(&rect[3], c_hi);
  }
  __syncthreads();  // the zeros are in memory before any gradient
  const int y0 = rect[0], y1 = rect[1] + 1, x0 = rect[2], x1 = rect[3] + 1;
  // d/dsigma, d/dp_out, observed pixels counted there
  double acc[3] = {0.0, 0.0, 0.0};
  if (y1 > 0) {
    const int ry0 = max(y0 - h, 0), ry1 = min(y1 + h, H), rx0 = max(x0 - h, 0), rx1 = min(x1 + h, W);
    const int lx0 = x0 - 2 * h, lw = x1 - x0 + 4 * h, rw = rx1 - rx0;
    const int room = area_bytes / crop_row_bytes(lw, rw);
    const int band = max(room - 4 * h, 1);
    const float inv_lw = 1.0f / (float)lw, inv_rw = 1.0f / (float)rw, inv_ow = 1.0f / (float)(x1 - x0);
    const float gb = g * sc.bn;
    for (int a = ry0; a < ry1; a += band) {
      const int b = min(a + band, ry1);
      const int wa = max(a - h, ry0), wb = min(b + h, ry1);
      const int ly0 = a - 2 * h, nl = (b - a + 4 * h) * lw;
      CropLds L;
      L.px = area;
      L.py = L.px + nl;
      L.pz = L.py + nl;
      L.w = L.pz + nl;
      // 2. the band's points
      for (int k = threadIdx.x; k < nl; k += BS) {
        int r, c;
        row_col(k, lw, inv_lw, r, c);
        r += ly0;
        c += lx0;
        float x = 0.0f, y = 0.0f, z = kFarPoint;
        if (r >= y0 && r < y1 && c >= x0 && c < x1) {
          const float* q = rn + 3 * ((size_t)r * W + c);
          if (q[2] > 0.0f) {
            x = q[0];
            y = q[1];
            z = q[2];
          }
        }
        L.px[k] = x;
        L.py[k] = y;
        L.pz[k] = z;
      }
      __syncthreads();
      // 3. window sums and weights of the valid observed pixels
      wave_compacted<kCropWaves>(
          (wb - wa) * rw, queue,
          [&](int k) {
            int r, c;
            row_col(k, rw, inv_rw, r, c);
            const bool valid = obs[3 * ((size_t)(wa + r) * W + (rx0 + c)) + 2] > 0.0f;
            if (!valid) L.w[k] = 0.0f;
            return valid;
          },
          [&](int k, bool act) {
            if (!act) return;
            int r, c;
            row_col(k, rw, inv_rw, r, c);
            r += wa;
            c += rx0;
            const float* q = obs + 3 * ((size_t)r * W + c);
            float S, T;
            window_crop<HH, true>(L, lw, h, (r - h - ly0) * lw + (c - h - lx0), q[0], q[1], q[2], sc.c2, S, T);
            const float Li = sc.a + sc.bn * S;
            if (r >= a && r < b) {
              acc[0] += (double)((sc.bn / Li) * (T * sc.inv_s3 - 3.0f * S * sc.inv_s));
              acc[1] += (double)((sc.invV - sc.normM * S) / Li);
              acc[2] += 1.0;
            }
            L.w[k] = gb / Li;
          });
      __syncthreads();
      // 4. every drawn pixel of the rows [a, b) gathers over its window (the
      //    window is symmetric: no atomics)
      if (dn) {
        const int ga = max(a, y0), gc = min(b, y1);
        wave_compacted<kCropWaves>(
            max(gc - ga, 0) * (x1 - x0), queue,
            [&](int k) {
              int r, c;
              row_col(k, x1 - x0, inv_ow, r, c);
              return L.pz[(ga + r - ly0) * lw + (c + 2 * h)] < kFarPoint;
            },
            [&](int k, bool act) {
              if (!act) return;
              int r, c;
              row_col(k, x1 - x0, inv_ow, r, c);
              r += ga;
              const int slot = (r - ly0) * lw + (c + 2 * h);
              c += x0;
              const float qx = L.px[slot], qy = L.py[slot], qz = L.pz[slot];
              float gx = 0.0f, gy = 0.0f, gz = 0.0f;
              auto term = [&](float w, const float* q) {
                const float ex = q[0] - qx, ey = q[1] - qy, ez = q[2] - qz;
                const float e = w * fast_exp2(-(ex * ex + ey * ey + ez * ez) * sc.c2);
                gx += e * ex;
                gy += e * ey;
                gz += e * ez;
              };
              bool done = false;
              if (HH > 0 && r - HH >= wa && r + HH < wb && c - HH >= rx0 && c + HH < rx1) {
                const float* w = L.w + (r - HH - wa) * rw + (c - HH - rx0);
                const float* o = obs + 3 * ((size_t)(r - HH) * W + (c - HH));
#pragma unroll 1
                for (int j = 0; j < 2 * HH + 1; ++j, w += rw, o += 3 * (size_t)W)
#pragma unroll
                  for (int i = 0; i < 2 * HH + 1; ++i) term(w[i], o + 3 * i);
                // (a pixel without a measurement may hold anything: 0 times that is not 0)
                const float any = gx + gy + gz;
                done = any == any;
              }
              if (!done) {
                gx = gy = gz = 0.0f;
                for (int ri = max(r - h, wa); ri <= min(r + h, wb - 1); ++ri)
                  for (int ci = max(c - h, rx0); ci <= min(c + h, rx1 - 1); ++ci) {
                    const float w = L.w[(ri - wa) * rw + (ci - rx0)];
                    if (w != 0.0f) term(w, obs + 3 * ((size_t)ri * W + ci));
                  }
              }
              float* o = dn + 3 * ((size_t)r * W + c);
              o[0] = gx * sc.inv_s2;
              o[1] = gy * sc.inv_s2;
              o[2] = gz * sc.inv_s2;
            });
      }
      __syncthreads();
    }
  }
  // less all observed pixels: whole numbers, exact
  for (int r = threadIdx.x; r < H; r += BS) acc[2] -= (double)rows[r + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double v = wave_sum(acc[k]);
    if (lane == 0) sums[3 * wave + k] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t[3] = {0.0, 0.0, 0.0};
    for (int w = 0; w < kCropWaves; ++w)
      for (int k = 0; k < 3; ++k) t[k] += sums[3 * w + k];
    // the observed pixels that see nothing
    t[1] -= t[2] * (double)(sc.invV / sc.a);
    if (d_sigma) d_sigma[n] = (float)((double)g * t[0]);
    if (d_pout) d_pout[n] = (float)((double)g * t[1]);
  }
}

// Whether the kernel takes images of width W: one row and its halo in LDS.
bool score_backward_crop_fits(int W, int h) {
  return (size_t)(4 * h + 1) * crop_row_bytes(W + 4 * h, W) <= kCropLds - crop_fixed_bytes(512);
}

template <bool VEC, int BS>
static auto crop_kernel(int h) {
  return h == 1   ? k_score_backward_crop<1, VEC, BS>
         : h == 2 ? k_score_backward_crop<2, VEC, BS>
         : h == 3 ? k_score_backward_crop<3, VEC, BS>
                  : k_score_backward_crop<0, VEC, BS>;
}

// Threads and LDS by how many workgroups a CU then holds, which is what bounds
// small images: never more LDS than the whole image needs; 256 threads up to
// 1,024 pixels (3,000 images of 24x32, 3x3 windows, mostly empty or full: 40 and
// 87 us against 57 and 108 with 512); and half of the LDS, four workgroups per
// CU instead of two, where there are hypotheses for them and a band still has
// more rows of its own than 5/4 of its halo's (3,000 of 48x64, 3x3: 83 and 246 us
// against 101 and 277; 500 of 120x160, 7x7, a halo of most of the band: 135 and
// 1,409 against 122 and 713).
hipError_t launch_score_backward_crop(const float* obs, const float* rend, int N, int H, int W, const ScoreConsts& sc,
                                      void* workspace, const float* dlogL, float* d_rend, float* d_sigma,
                                      float* d_pout, hipStream_t st) {
  // the rows' counts of observed pixels alone: the list is not read
  int* rows = reinterpret_cast<int*>(workspace);
  hipLaunchKernelGGL(k_obs_count, dim3(H), dim3(kBlock), 0, st, obs, H, W, rows);
  const bool vec = W % 4 == 0 && (((uintptr_t)rend | (uintptr_t)d_rend) & 15) == 0;
  const int h = sc.h, bs = H * W <= 1024 ? 256 : 512, fixed = (int)crop_fixed_bytes(bs);
  const int row = crop_row_bytes(W + 4 * h, W);
  int area = (int)kCropLds - fixed;
  const int half = (int)kCropLds / 2 - fixed;
  if (N > 2 * kCUs && half / row - 4 * h > 5 * h) area = half;
  area = (int)std::min<size_t>(area, (size_t)(H + 4 * h) * row);
  auto k = bs == 256 ? (vec ? crop_kernel<true, 256>(h) : crop_kernel<false, 256>(h))
                     : (vec ? crop_kernel<true, 512>(h) : crop_kernel<false, 512>(h));
  hipLaunchKernelGGL(k, dim3(N), dim3(bs), (size_t)(fixed + area), st, obs, rend, N, H, W, sc, rows, dlogL, d_rend,
                     d_sigma, d_pout, area);
  return hipGetLastError();
}

// Inclusive sum over the lanes of a wave up to this one.
__device__ __forceinline__ double wave_scan(double v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}

// Per-pixel likelihood terms of the background alone (double precision: l_p,
// dl_p/dp_out, dl_p/dsigma, zero for invalid observed pixels), summed along
// the rows: block (r, y) writes row r of the three tables of parameters y,
// sat[k][r (W + 1) + c] = sum of term k over row r - 1, columns < c (row 0:
// zeros).  k_sat_cols then sums down the columns.  A row's terms and their
// running sums stay in the block: one launch instead of two and a pass over
// three images less, and the sums are scans across lanes (one thread per row
// took 71 us at 320x240, one per column 70, the terms 17; these two kernels take 30).
__global__ __launch_bounds__(kBlock) void k_bg_rows(SceneDev s, BgTablesDev B) {
  __shared__ double part[3][kWaves];
  const int H = s.cam.H, W = s.cam.W, r = (int)blockIdx.x - 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const ScoreConsts& sc = B.sc[blockIdx.y];
  const size_t table = (size_t)(H + 1) * (W + 1);
  double* out = B.sat + B.stride * blockIdx.y + (size_t)blockIdx.x * (W + 1);
  if (threadIdx.x < 3) out[threadIdx.x * table] = 0.0;
  double carry[3] = {0.0, 0.0, 0.0};
  for (int base = 0; base < W; base += kBlock) {
    const int c = base + (int)threadIdx.x;
    double v[3] = {0.0, 0.0, 0.0};
    const float* q = s.obs + 3 * ((size_t)max(r, 0) * W + min(c, W - 1));
    if (r >= 0 && c < W && q[2] > 0.0f) {
      double S = 0.0, T = 0.0;
      if (s.bg) {
        const int h = sc.h;
        for (int rj = max(r - h, 0); rj <= min(r + h, H - 1); ++rj)
          for (int cj = max(c - h, 0); cj <= min(c + h, W - 1); ++cj) {
            const unsigned long long k = s.bg[(size_t)rj * W + cj];
            if (k == kEmptyKey) continue;
            const double z = (double)key_depth(k);
            const double ex = (double)q[0] - z * (double)ray_x(s.cam, cj);
            const double ey = (double)q[1] - z * (double)ray_y(s.cam, rj);
            const double ez = (double)q[2] - z;
            const double D = ex * ex + ey * ey + ez * ez;
            const double e = exp(-D * sc.dc);
            S += e;
            T += e * D;
          }
      }
      const double L = sc.da + sc.dbn * S;
      v[0] = log(L);
      v[1] = (sc.dinvV - sc.dnormM * S) / L;
      v[2] = (sc.dbn / L) * (T * sc.dinv_s3 - 3.0 * S * sc.dinv_s);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      v[k] = wave_scan(v[k]);
      if (lane == 63) part[k][wave] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double before = carry[k];
      for (int w = 0; w < kWaves; ++w) {
        before += w < wave ? part[k][w] : 0.0;
        carry[k] += part[k][w];
      }
      if (c < W) out[k * table + c + 1] = before + v[k];
    }
    __syncthreads();
  }
}

// Sums down the columns of every table, in place: a block takes 64 columns,
// each of its 16 waves a run of rows (their total first, then the running
// sums from the waves before).
constexpr int kColWaves = 16;
__global__ __launch_bounds__(64 * kColWaves) void k_sat_cols(int H, int W, double* sat, long long stride) {
  __shared__ double part[kColWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + lane, cc = min(c, W);
  double* o = sat + stride * (blockIdx.y / 3) + (size_t)(blockIdx.y % 3) * (H + 1) * (W + 1) + cc;
  const int run = (H + kColWaves) / kColWaves;  // ceil((H + 1) / kColWaves) rows
  const int r0 = wave * run, r1 = min(r0 + run, H + 1);
  double sum = 0.0;
#pragma unroll 4
  for (int r = r0; r < r1; ++r) sum += o[(size_t)r * (W + 1)];
  part[wave][lane] = sum;
  __syncthreads();
  double at = 0.0;
  for (int w = 0; w < wave; ++w) at += part[w][lane];
  if (c > W) return;
  for (int r = r0; r < r1; r += 4) {
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = r + k < r1 ? o[(size_t)(r + k) * (W + 1)] : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      at += v[k];
      if (r + k < r1) o[(size_t)(r + k) * (W + 1)] = at;
    }
  }
}

hipError_t launch_background_tables(const SceneDev& s, const BgTablesDev& B, hipStream_t st) {
  const int H = s.cam.H, W = s.cam.W;
  hipLaunchKernelGGL(k_bg_rows, dim3(H + 1, B.n), dim3(kBlock), 0, st, s, B);
  hipLaunchKernelGGL(k_sat_cols, dim3((W + 64) / 64, 3 * B.n), dim3(64 * kColWaves), 0, st, H, W, B.sat, B.stride);
  return hipGetLastError();
}

}  // namespace b3d
