// Dense-grid DVR (the uncompressed reference renderer), dense point sampling,
// Philox point sampling, grid casts, and the precision dispatch of the
// network launchers.
#include <stdio.h>

#include <atomic>
#include <cmath>
#include <mutex>

#include "fvsrn_common.hpp"

namespace fvsrn_detail {

namespace {

__device__ inline void tf_eval_d(const TFDev& tf, float d, float rgba[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) rgba[q] = tf.base[q];
  for (int j = 0; j < tf.n_seg; ++j) {
    const float w = __builtin_amdgcn_fmed3f(fmaf(d, tf.inv[j], tf.off[j]), 0.0f, 1.0f);
#pragma unroll
    for (int q = 0; q < 4; ++q) rgba[q] = fmaf(w, tf.delta[j][q], rgba[q]);
  }
}

__device__ inline int xcd_block_d(int nblocks) {
  const int b = blockIdx.x;
  if (nblocks % 8 != 0) return b;
  const int per = nblocks / 8;
  return (b % 8) * per + b / 8;
}

// ---------------------------------------------------------- dense DVR

__device__ inline float dense_sample(const float* vol, int nx, int ny, int nz, float px, float py,
                                     float pz) {
  int ix, iy, iz;
  float fx, fy, fz;
  axis_cell(px, nx, ix, fx);
  axis_cell(py, ny, iy, fy);
  axis_cell(pz, nz, iz, fz);
  const long long sy = nx, sz = (long long)nx * ny;
  const float* b = vol + iz * sz + iy * sy + ix;
  const float c00 = b[0] + fx * (b[1] - b[0]);
  const float c10 = b[sy] + fx * (b[sy + 1] - b[sy]);
  const float c01 = b[sz] + fx * (b[sz + 1] - b[sz]);
  const float c11 = b[sz + sy] + fx * (b[sz + sy + 1] - b[sz + sy]);
  const float c0 = c00 + fy * (c10 - c00);
  const float c1 = c01 + fy * (c11 - c01);
  return c0 + fz * (c1 - c0);
}

constexpr int kDenseThreads = 256;

// Tile of a wave of the dense march: a step takes S = 2^ls consecutive
// segments of R = 128 / S rays (ls >= 1), in two passes over G = 64 / S rays
// each. Rays are numbered pass by pass, row by row within a pass's block; the
// second pass's block lies below the first's.
struct DenseTile {
  int ls;
  __host__ __device__ int rays() const { return 128 >> ls; }
  __host__ __device__ int lw() const { return (7 - ls) / 2; }  // log2 of the tile's edges
  __host__ __device__ int lh() const { return (6 - ls) / 2 + 1; }
  __device__ int x(int r) const { return r & ((1 << lw()) - 1); }
  __device__ int y(int r) const { return r >> lw(); }
};

// Dense DVR. The volume is read through L1 lookups, one per 128-byte line that
// a group of four lanes touches, and with one segment of 8x8 rays per wave
// these bound the march (27 per load of 64 lanes, one per CU and cycle). A
// wave therefore takes four segments of 4x4 rays per load: its lanes are as
// close in depth as they are across, and the lanes of a group are kept
// together along x, the volume's contiguous axis -- neighbouring pixels, or,
// where the view looks along x (the forward direction's x beyond 0.6), two
// segments of one ray. Each lane takes its samples through the transfer
// function and leaves colour and transmittance in LDS, from where the ray's
// own lane composites them in order: the image is the same, bit for bit,
// whatever the tile. A step has two passes, which hide each other's loads (one
// pass: 11.3 ms for 8 x 1024^2, four: 9.9). 256^3 volume, 1024^2 views, before
// and now: along z 1.22 -> 1.22 ms, 22 degrees off 1.47 -> 1.27, 45 1.66 -> 1.46,
// 67 1.72 -> 1.36, along x 1.64 -> 1.25, an orbit of eight 10.3 -> 9.1 (the VALU
// and the lookups are then about even); small launches: launch_render_dense.
template <bool PHONG, bool BIG>
__global__ __launch_bounds__(kDenseThreads, PHONG ? 4 : 5) void dense_march_kernel(const float* vol, int nx, int ny, int nz, TFDev tf,
                                                                    ViewBatch vb, MarchDev m, float* out,
                                                                    unsigned long long* stats, int tiles_x,
                                                                    int tiles_y, DenseTile dt) {
  constexpr int Q = 2;
  __shared__ f4 rays[kDenseThreads / 64][3][64];
  __shared__ f4 samples[kDenseThreads / 64][128];  // [segment][ray]: colour, transmittance (< 0: none)
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tiles_per_view = tiles_x * tiles_y;
  const int tile = __builtin_amdgcn_readfirstlane(xcd_block_d(gridDim.x) * (kDenseThreads / 64) + wave);
  if (tile >= tiles_per_view * vb.n_views) return;
  const int S = 1 << dt.ls, R = dt.rays(), G = 64 >> dt.ls;
  f4(*rw)[64] = rays[wave];
  f4* sw = samples[wave];
  __amdgpu_buffer_rsrc_t rsrc;
  if constexpr (!BIG) rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vol), 0, nx * ny * nz * 4, 0x00020000);
  // the rows along x of the cell around p, and p's fractions in it
  auto cell_rows = [&](const float p[3], f2 row[4], float f[3]) {
    int c[3];
    axis_cell(p[0], nx, c[0], f[0]);
    axis_cell(p[1], ny, c[1], f[1]);
    axis_cell(p[2], nz, c[2], f[2]);
    if constexpr (BIG) {
      const float* b = vol + ((long long)c[2] * ny + c[1]) * nx + c[0];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float* e = b + (k & 1 ? nx : 0) + (k >> 1 ? (long long)nx * ny : 0);
        row[k] = f2{e[0], e[1]};
      }
    } else {
      const unsigned at = ((unsigned)(c[2] * ny + c[1]) * (unsigned)nx + (unsigned)c[0]) * 4u;
      const unsigned sy = (unsigned)nx * 4u, sz = (unsigned)ny * sy;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        row[k] = __builtin_bit_cast(
            f2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, (k & 1 ? sy : 0u) + (k >> 1 ? sz : 0u), 0));
    }
  };
  auto trilinear = [](const f2 row[4], const float f[3]) {
    const float c00 = row[0][0] + f[0] * (row[0][1] - row[0][0]);
    const float c10 = row[1][0] + f[0] * (row[1][1] - row[1][0]);
    const float c01 = row[2][0] + f[0] * (row[2][1] - row[2][0]);
    const float c11 = row[3][0] + f[0] * (row[3][1] - row[3][0]);
    const float c0 = c00 + f[1] * (c10 - c00);
    const float c1 = c01 + f[1] * (c11 - c01);
    return c0 + f[2] * (c1 - c0);
  };
  auto sample = [&](float x, float y, float z) {
    const float p[3] = {x, y, z};
    f2 row[4];
    float f[3];
    cell_rows(p, row, f);
    return trilinear(row, f);
  };
  const bool fixed = m.fixed_steps > 0;
  const float hx = 2.0f / (float)(nx - 1), hy = 2.0f / (float)(ny - 1), hz = 2.0f / (float)(nz - 1);
  const int v = tile / tiles_per_view, tr = tile % tiles_per_view;
  const CamDev& cam = vb.cam[v];
  // a lane's ray within the pass and its segment: segment bits at either end of the lane index
  const int low = dt.ls > 0 && fabs(cam.fwd[0]) > 0.6 ? 1 : 0;
  const int rl = (lane >> low) & (G - 1), sl = (lane & ((1 << low) - 1)) | (lane >> (6 - dt.ls + low) << low);
  const int px = ((tr % tiles_x) << dt.lw()) + dt.x(lane), py = ((tr / tiles_x) << dt.lh()) + dt.y(lane);
  const bool owner = lane < R && px < vb.width && py < vb.height;
  int nseg = 0;
  if (lane < R) {
    const Ray r = make_ray(cam, owner ? px : 0, owner ? py : 0, vb.width, vb.height, m);
    nseg = owner && r.hit ? r.nseg : 0;
    rw[0][lane] = f4{r.o[0], r.o[1], r.o[2], r.t0};
    rw[1][lane] = f4{r.d[0], r.d[1], r.d[2], r.ds};
    rw[2][lane] = f4{r.t1, __int_as_float(nseg), 0.0f, 0.0f};
  }
  float T = 1.0f, Cr = 0.0f, Cg = 0.0f, Cb = 0.0f, A = 0.0f;
  int n = 0;
  bool active = nseg > 0;
  for (int i0 = 0;; i0 += S) {
    if (!__builtin_amdgcn_ballot_w64(active)) break;
    wave_lds_sync();
    const int i = i0 + sl;
    float len[Q], d[Q], px3[Q][3];
    bool has[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int r = q * G + rl;
      const f4 ro = rw[0][r], rd = rw[1][r], re = rw[2][r];
      const float a0 = ro[3] + (float)i * rd[3];
      float a1 = ro[3] + (float)(i + 1) * rd[3];
      if (!fixed) a1 = fminf(a1, re[0]);
      const float tm = 0.5f * (a0 + a1);
      len[q] = a1 - a0;
      has[q] = i < __float_as_int(re[1]) && len[q] > 0.0f;
#pragma unroll
      for (int a = 0; a < 3; ++a) px3[q][a] = ro[a] + tm * rd[a];
    }
    f2 rows[Q][4];
    float fr[Q][3];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (has[q]) cell_rows(px3[q], rows[q], fr[q]);
#pragma unroll
    for (int q = 0; q < Q; ++q) d[q] = has[q] ? trilinear(rows[q], fr[q]) : 0.0f;
    float rgba[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c) rgba[q][c] = tf.base[c];
    for (int j = 0; j < tf.n_seg; ++j)
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float w = __builtin_amdgcn_fmed3f(fmaf(d[q], tf.inv[j], tf.off[j]), 0.0f, 1.0f);
#pragma unroll
        for (int c = 0; c < 4; ++c) rgba[q][c] = fmaf(w, tf.delta[j][c], rgba[q][c]);
      }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int r = q * G + rl;
      if constexpr (PHONG) {
        if (m.phong && has[q]) {
          const float sx = px3[q][0], sy = px3[q][1], sz = px3[q][2];
          const float gx = (sample(sx + hx, sy, sz) - sample(sx - hx, sy, sz)) / (2.0f * hx);
          const float gy = (sample(sx, sy + hy, sz) - sample(sx, sy - hy, sz)) / (2.0f * hy);
          const float gz = (sample(sx, sy, sz + hz) - sample(sx, sy, sz - hz)) / (2.0f * hz);
          const float gl = sqrtf(gx * gx + gy * gy + gz * gz);
          if (gl >= 1e-6f) {
            const f4 r1 = rw[1][r];
            const float ndl = fabsf(gx * r1[0] + gy * r1[1] + gz * r1[2]) / gl;
            const float spec = m.ks * powf(ndl, m.shininess);
            const float k = m.ka + m.kd * ndl;
            rgba[q][0] = rgba[q][0] * k + spec;
            rgba[q][1] = rgba[q][1] * k + spec;
            rgba[q][2] = rgba[q][2] * k + spec;
          }
        }
      }
      sw[sl * R + r] = f4{rgba[q][0], rgba[q][1], rgba[q][2], has[q] ? fast_exp(-rgba[q][3] * len[q]) : -1.0f};
    }
    wave_lds_sync();
    for (int k = 0; k < S; ++k) {
      const f4 e = sw[k * R + (lane & (R - 1))];
      active = active && !(e[3] < 0.0f);
      const float trn = active ? e[3] : 1.0f;
      const float ta = T * (1.0f - trn);
      // PHONG: not by a weight of 0, since behind the ray's end a shade may be infinite
      Cr = active || !PHONG ? fmaf(ta, e[0], Cr) : Cr;
      Cg = active || !PHONG ? fmaf(ta, e[1], Cg) : Cg;
      Cb = active || !PHONG ? fmaf(ta, e[2], Cb) : Cb;
      A += ta;
      T *= trn;
      n += active ? 1 : 0;
      active = active && !(T < m.ert_eps);
    }
    active = active && i0 + S < nseg;
    if (lane < R && !active) rw[2][lane][1] = __int_as_float(0);  // an ended ray takes no more samples
  }
  if (owner)
    reinterpret_cast<float4*>(out)[((long long)v * vb.height + py) * vb.width + px] = make_float4(Cr, Cg, Cb, A);
  if (stats) {
    unsigned mine = (unsigned)n, hit = nseg > 0 ? 1u : 0u;
    for (int off = 32; off > 0; off >>= 1) {
      mine += (unsigned)__shfl_xor((int)mine, off, 64);
      hit += (unsigned)__shfl_xor((int)hit, off, 64);
    }
    if (lane == 0) {
      atomicAdd(stats, (unsigned long long)mine);
      atomicAdd(stats + 1, (unsigned long long)hit);
      atomicAdd(stats + 2, (unsigned long long)mine);
    }
  }
}

// Samples (out, nullable) and one-voxel central-difference gradients (out_g,
// nullable) of the dense grid, as the dense renderer shades.
__global__ void dense_points_kernel(const float* vol, int nx, int ny, int nz, const float* xyz,
                                    long long n, float* out, float* out_g) {
  const float hx = 2.0f / (float)(nx - 1), hy = 2.0f / (float)(ny - 1), hz = 2.0f / (float)(nz - 1);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const float x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
    if (out) out[i] = dense_sample(vol, nx, ny, nz, x, y, z);
    if (out_g) {
      out_g[3 * i] = (dense_sample(vol, nx, ny, nz, x + hx, y, z) - dense_sample(vol, nx, ny, nz, x - hx, y, z)) /
                     (2.0f * hx);
      out_g[3 * i + 1] =
          (dense_sample(vol, nx, ny, nz, x, y + hy, z) - dense_sample(vol, nx, ny, nz, x, y - hy, z)) / (2.0f * hy);
      out_g[3 * i + 2] =
          (dense_sample(vol, nx, ny, nz, x, y, z + hz) - dense_sample(vol, nx, ny, nz, x, y, z - hz)) / (2.0f * hz);
    }
  }
}

// --------------------------------------------------------- utilities

__device__ inline void philox_round(uint32_t c[4], const uint32_t k[2]) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t hi0 = __umulhi(M0, c[0]), lo0 = M0 * c[0];
  const uint32_t hi1 = __umulhi(M1, c[2]), lo1 = M1 * c[2];
  const uint32_t n0 = hi1 ^ c[1] ^ k[0], n2 = hi0 ^ c[3] ^ k[1];
  c[0] = n0;
  c[1] = lo1;
  c[2] = n2;
  c[3] = lo0;
}

}  // namespace

// Philox4x32-10 (Salmon et al., SC'11) of counter (i mod 2^32, i div 2^32,
// c_lo, c_hi) and key (k0, k1): four 32-bit outputs in c.
__device__ void philox4x32_10(long long i, uint32_t c_lo, uint32_t c_hi, uint32_t k0, uint32_t k1, uint32_t c[4]) {
  c[0] = (uint32_t)i;
  c[1] = (uint32_t)((unsigned long long)i >> 32);
  c[2] = c_lo;
  c[3] = c_hi;
  uint32_t k[2] = {k0, k1};
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k[0] += 0x9E3779B9u;
      k[1] += 0xBB67AE85u;
    }
    philox_round(c, k);
  }
}

namespace {

__global__ void sample_points_kernel(uint32_t k0, uint32_t k1, uint32_t c_lo, uint32_t c_hi,
                                     long long n, float* xyz) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    uint32_t c[4];
    philox4x32_10(i, c_lo, c_hi, k0, k1, c);
    const float s = 1.0f / 8388608.0f;  // 2^-23
    xyz[3 * i + 0] = -1.0f + (float)(c[0] >> 8) * s;
    xyz[3 * i + 1] = -1.0f + (float)(c[1] >> 8) * s;
    xyz[3 * i + 2] = -1.0f + (float)(c[2] >> 8) * s;
  }
}

__global__ void cast_f16_kernel(const float* src, _Float16* dst, long long count) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    dst[i] = (_Float16)src[i];
}

__global__ void cast_bf16_kernel(const float* src, __bf16* dst, long long count) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    dst[i] = (__bf16)src[i];
}

// SSIM map (Wang et al. 2004); the 11 x 11 Gaussian window is the outer product
// of the normalised 1-D weights. A workgroup owns a tile of 64 x 16 outputs and
// keeps its 74 x 26 input pixels of both images in LDS; a thread takes four
// neighbouring outputs, whose window rows share 14 inputs and their products.
// Bound by its FP32 FMAs (1,815 per output): two 800 x 600 pairs 148 -> 67 us
// against one thread per output reading both images through L1. The window's
// sums are taken row by row over all 121 taps. Rows first, then columns (22 taps)
// ran in 18 us; the variance terms cancel, so that it moves the map by 8e-5 of its
// norm, in the one case measured to a third of this order's error against FP64.
struct Window11 {
  float g[11];
};
constexpr int kSsimW = 64, kSsimH = 16, kSsimIW = kSsimW + 10, kSsimIH = kSsimH + 10;

__global__ __launch_bounds__(256) void ssim_kernel(const float4* a, const float4* b, int W, int H, int n, Window11 win,
                                                   float* out) {
  __shared__ float in[2][3][kSsimIH][kSsimIW];
  const int WO = W - 10, HO = H - 10, tx = (WO + kSsimW - 1) / kSsimW, ty = (HO + kSsimH - 1) / kSsimH;
  const int t = threadIdx.x;
  const int ox = 4 * (t % (kSsimW / 4)), oy = t / (kSsimW / 4);  // this thread's outputs ox .. ox + 3
  for (long long tile = blockIdx.x; tile < (long long)n * tx * ty; tile += gridDim.x) {
    const int x0 = (int)(tile % tx) * kSsimW, y0 = (int)((tile / tx) % ty) * kSsimH;
    const long long img = tile / ((long long)tx * ty);
    for (int e = t; e < kSsimIH * kSsimIW; e += 256) {
      const int x = e % kSsimIW, y = e / kSsimIW;
      const long long p = (img * H + min(y0 + y, H - 1)) * W + min(x0 + x, W - 1);
      const float4 va = a[p], vb = b[p];
      in[0][0][y][x] = va.x;
      in[0][1][y][x] = va.y;
      in[0][2][y][x] = va.z;
      in[1][0][y][x] = vb.x;
      in[1][1][y][x] = vb.y;
      in[1][2][y][x] = vb.z;
    }
    __syncthreads();
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int ch = 0; ch < 3; ++ch) {
      float m[4][5] = {};
      for (int i = 0; i < 11; ++i) {
        const float *ra = &in[0][ch][oy + i][ox], *rb = &in[1][ch][oy + i][ox];
        float w[11];
#pragma unroll
        for (int j = 0; j < 11; ++j) w[j] = win.g[i] * win.g[j];
#pragma unroll
        for (int k = 0; k < 14; ++k) {
          const float pa = ra[k], pb = rb[k];
          const float v[5] = {pa, pb, pa * pa, pb * pb, pa * pb};
#pragma unroll
          for (int o = 0; o < 4; ++o)
            if (k >= o && k - o < 11)
#pragma unroll
              for (int q = 0; q < 5; ++q) m[o][q] = fmaf(w[k >= o && k - o < 11 ? k - o : 0], v[q], m[o][q]);
        }
      }
      const float C1 = 1e-4f, C2 = 9e-4f;
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        const float mx = m[o][0], my = m[o][1];
        const float sx = m[o][2] - mx * mx, sy = m[o][3] - my * my, sxy = m[o][4] - mx * my;
        s[o] += ((2.0f * mx * my + C1) * (2.0f * sxy + C2)) / ((mx * mx + my * my + C1) * (sx + sy + C2));
      }
    }
#pragma unroll
    for (int o = 0; o < 4; ++o)
      if (x0 + ox + o < WO && y0 + oy < HO) out[(img * HO + y0 + oy) * WO + x0 + ox + o] = s[o] * (1.0f / 3.0f);
    __syncthreads();
  }
}

// uint8 quantisation (Sec. 4.2). One workgroup per channel finds the
// channel's minimum and maximum (order-independent, so exact) and writes
// (lo, (hi - lo) / 255); then every value is encoded as
// round-half-even((x - lo) / scale), clamped to [0, 255], in FP32.
__global__ __launch_bounds__(256) void channel_range_kernel(const float* src, long long n, int channels,
                                                            float* dequant) {
  __shared__ float s_lo[256], s_hi[256];
  const int ch = blockIdx.x, t = threadIdx.x;
  float lo = src[ch], hi = src[ch];
  for (long long i = t; i < n; i += blockDim.x) {
    const float x = src[i * channels + ch];
    lo = fminf(lo, x);
    hi = fmaxf(hi, x);
  }
  s_lo[t] = lo;
  s_hi[t] = hi;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if (t < h) {
      s_lo[t] = fminf(s_lo[t], s_lo[t + h]);
      s_hi[t] = fmaxf(s_hi[t], s_hi[t + h]);
    }
    __syncthreads();
  }
  if (t == 0) {
    dequant[2 * ch] = s_lo[0];
    dequant[2 * ch + 1] = (s_hi[0] - s_lo[0]) / 255.0f;
  }
}

__global__ void encode_u8_kernel(const float* src, long long count, int channels, const float* dequant,
                                 unsigned char* codes) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % channels);
    const float lo = dequant[2 * ch], scale = dequant[2 * ch + 1];
    float q = 0.0f;
    if (scale > 0.0f) q = fminf(fmaxf(rintf((src[i] - lo) / scale), 0.0f), 255.0f);
    codes[i] = (unsigned char)q;
  }
}

}  // namespace

thread_local char g_hip_err[256];


int check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    snprintf(g_hip_err, sizeof(g_hip_err), "%s", hipGetErrorString(e));
    return 2;
  }
  return 0;
}

int grid_blocks(long long work, int per_block, int cap) {
  long long b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

int device_cus() {
  static int cus = 0;
  if (!cus) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
    if (cus <= 0) cus = 256;
  }
  return cus;
}

namespace {
__device__ __align__(256) unsigned int tile_queues[2 * kTileQueueSlots];
}  // namespace

RayEnds ray_ends(const TFDev& tf, const MarchDev& m) {
  double kappa = tf.base[3], most = kappa, least = kappa;
  for (int j = 0; j < tf.n_seg; ++j) {
    kappa += tf.delta[j][3];
    most = fmax(most, kappa);
    least = fmin(least, kappa);
  }
  const double ds = m.fixed_steps > 0 ? 3.4641016 / m.fixed_steps : m.step;  // the longest segment
  // (the sum of the deltas is off by the rounding of FP32 differences)
  auto segments = [&](double k) {
    return m.ert_eps > 0.0f && k > 1e-6 * most ? fmax(1.0, -log((double)m.ert_eps) / (k * ds)) : HUGE_VAL;
  };
  return {segments(most), segments(least)};
}

unsigned int* tile_queue_slot() {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static unsigned int* base[kMaxDevices] = {};
  static std::atomic<unsigned int> next{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    snprintf(g_hip_err, sizeof(g_hip_err), "no current device for the tile queue");
    return nullptr;
  }
  unsigned int* b = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!base[dev]) {
      void* p = nullptr;
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(tile_queues));
      if (e != hipSuccess || !p) {
        snprintf(g_hip_err, sizeof(g_hip_err), "tile queue: %s", hipGetErrorString(e));
        return nullptr;
      }
      base[dev] = static_cast<unsigned int*>(p);
    }
    b = base[dev];
  }
  return b + 2 * (next.fetch_add(1u) % kTileQueueSlots);
}

// ------------------------------------------ adaptive resampling (Sec. 5.4)

namespace {

// Position inside voxel v of a G^3 grid over [-1,1]^3 (x fastest) from three
// random words: p_a = fma((float)i_a + u_a, 2/G, -1), u_a = (r_a >> 8) 2^-24.
__device__ inline void voxel_position(int G, long long v, const uint32_t* r, float* p) {
  const long long iv[3] = {v % G, (v / G) % G, v / ((long long)G * G)};
  const float step = 2.0f / (float)G;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float u = (float)(r[a] >> 8) * 5.9604644775390625e-8f;  // 2^-24
    p[a] = fmaf((float)iv[a] + u, step, -1.0f);
  }
}

__global__ void voxel_points_kernel(uint32_t k0, uint32_t k1, uint32_t c_lo, uint32_t c_hi, int G, int per_voxel,
                                    long long n, float* xyz) {
  for (long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x; j < n;
       j += (long long)gridDim.x * blockDim.x) {
    uint32_t c[4];
    philox4x32_10(j, c_lo, c_hi, k0, k1, c);
    voxel_position(G, j / per_voxel, c, xyz + 3 * j);
  }
}

// E[v] = mean over the voxel's points of |network density - trilinear target|.
__global__ void error_reduce_kernel(const float* d, const float* vol, int nx, int ny, int nz, const float* xyz,
                                    long long n_voxels, int per_voxel, float* E) {
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n_voxels;
       v += (long long)gridDim.x * blockDim.x) {
    float s = 0.0f;
    for (int k = 0; k < per_voxel; ++k) {
      const long long j = v * per_voxel + k;
      s += fabsf(d[j] - dense_sample(vol, nx, ny, nz, xyz[3 * j], xyz[3 * j + 1], xyz[3 * j + 2]));
    }
    E[v] = s / (float)per_voxel;
  }
}

// Largest weight (bits of non-negative floats order like unsigned integers;
// entries that are not >= 0 count as 0). emax must start at 0.
__global__ void weight_max_kernel(const float* E, long long nv, unsigned* emax) {
  unsigned m = 0;
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nv;
       v += (long long)gridDim.x * blockDim.x) {
    const float e = E[v];
    if (e >= 0.0f) m = max(m, __float_as_uint(e));
  }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0 && m) atomicMax(emax, m);
}

constexpr int kScanThreads = 256, kScanItems = 8, kScanBlock = kScanThreads * kScanItems;

// Integer weights q_v = floor(E_v * (2^24 / max E)) and their inclusive
// prefix sums within each block of kScanBlock voxels; block totals to S.
__global__ __launch_bounds__(kScanThreads) void weight_scan_kernel(const float* E, long long nv, const unsigned* emax,
                                                                   unsigned long long* Q, unsigned long long* S) {
  __shared__ unsigned long long part[kScanThreads];
  const float em = __uint_as_float(*emax);
  const float scale = em > 0.0f ? 16777216.0f / em : 0.0f;
  const long long base = (long long)blockIdx.x * kScanBlock + (long long)threadIdx.x * kScanItems;
  unsigned long long q[kScanItems], run = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const long long v = base + k;
    const float e = v < nv ? E[v] : 0.0f;
    run += (e >= 0.0f) ? (unsigned long long)floorf(e * scale) : 0ull;
    q[k] = run;
  }
  part[threadIdx.x] = run;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {  // inclusive scan of the thread totals
    const unsigned long long x = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0ull;
    __syncthreads();
    part[threadIdx.x] += x;
    __syncthreads();
  }
  const unsigned long long before = threadIdx.x ? part[threadIdx.x - 1] : 0ull;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < nv) Q[base + k] = q[k] + before;
  if (threadIdx.x == kScanThreads - 1) S[blockIdx.x] = part[threadIdx.x];
}

// Exclusive prefix sums of the block totals (one workgroup, in place).
__global__ __launch_bounds__(kScanThreads) void block_offsets_kernel(unsigned long long* S, long long nb) {
  __shared__ unsigned long long part[kScanThreads];
  unsigned long long carry = 0;
  for (long long b0 = 0; b0 < nb; b0 += kScanThreads) {
    const long long b = b0 + threadIdx.x;
    const unsigned long long x = b < nb ? S[b] : 0ull;
    part[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
      const unsigned long long y = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0ull;
      __syncthreads();
      part[threadIdx.x] += y;
      __syncthreads();
    }
    if (b < nb) S[b] = carry + part[threadIdx.x] - x;
    const unsigned long long total = part[kScanThreads - 1];
    __syncthreads();
    carry += total;
  }
}

__global__ void add_offsets_kernel(unsigned long long* Q, long long nv, const unsigned long long* S) {
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nv;
       v += (long long)gridDim.x * blockDim.x)
    Q[v] += S[v / kScanBlock];
}

// Point i (Philox counter words c_lo, c_hi): voxel v with
// Q[v-1] <= (r0 total) >> 32 < Q[v] (all weights zero: v = (r0 nv) >> 32),
// position inside it from r1..r3.
__device__ inline void draw_weighted(uint32_t k0, uint32_t k1, uint32_t c_lo, uint32_t c_hi,
                                     const unsigned long long* Q, unsigned long long total, int G, long long nv,
                                     long long i, float* out) {
  uint32_t c[4];
  philox4x32_10(i, c_lo, c_hi, k0, k1, c);
  long long v;
  if (total == 0) {
    v = (long long)(((unsigned long long)c[0] * (unsigned long long)nv) >> 32);
  } else {
    const unsigned long long target = __umul64hi((unsigned long long)c[0] << 32, total);
    long long lo = 0, hi = nv - 1;
    while (lo < hi) {
      const long long mid = (lo + hi) >> 1;
      if (Q[mid] > target) hi = mid;
      else lo = mid + 1;
    }
    v = lo;
  }
  voxel_position(G, v, c + 1, out);
}

__global__ void weighted_points_kernel(uint32_t k0, uint32_t k1, uint32_t c_lo, uint32_t c_hi,
                                       const unsigned long long* Q, int G, long long nv, long long n, float* xyz) {
  const unsigned long long total = Q[nv - 1];
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    draw_weighted(k0, k1, c_lo, c_hi, Q, total, G, nv, i, xyz + 3 * i);
}

// Several grids' draws in one launch: point i of the batch belongs to grid
// k with start[k] <= i < start[k + 1], draws with counter + k and local
// index i - start[k] from the prefix sums at ws + k stride bytes.
struct MultiDraw {
  int n;
  long long start[kMaxDrawGrids + 1];
};

__global__ void weighted_points_multi_kernel(uint32_t k0, uint32_t k1, unsigned long long counter, const char* ws,
                                             unsigned long long stride, int G, long long nv, MultiDraw md,
                                             float* xyz) {
  const long long n = md.start[md.n];
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    int k = 0;
#pragma unroll
    for (int j = 1; j < kMaxDrawGrids; ++j) k += (j < md.n && i >= md.start[j]) ? 1 : 0;
    const unsigned long long* Q = reinterpret_cast<const unsigned long long*>(ws + (unsigned long long)k * stride);
    const unsigned long long ck = counter + (unsigned long long)k;
    draw_weighted(k0, k1, (uint32_t)ck, (uint32_t)(ck >> 32), Q, Q[nv - 1], G, nv, i - md.start[k], xyz + 3 * i);
  }
}

__global__ void zero_u32_kernel(unsigned* p) { *p = 0u; }

}  // namespace

int launch_voxel_points(uint64_t seed, uint64_t counter, int G, int per_voxel, float* xyz, void* stream) {
  const long long n = (long long)G * G * G * per_voxel;
  hipLaunchKernelGGL(voxel_points_kernel, dim3(grid_blocks(n, 256, device_cus() * 16)), dim3(256), 0,
                     (hipStream_t)stream, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)counter,
                     (uint32_t)(counter >> 32), G, per_voxel, n, xyz);
  return check_launch();
}

int launch_error_reduce(const float* d, const float* vol, int nx, int ny, int nz, const float* xyz,
                        long long n_voxels, int per_voxel, float* E, void* stream) {
  hipLaunchKernelGGL(error_reduce_kernel, dim3(grid_blocks(n_voxels, 256, device_cus() * 16)), dim3(256), 0,
                     (hipStream_t)stream, d, vol, nx, ny, nz, xyz, n_voxels, per_voxel, E);
  return check_launch();
}

size_t weighted_points_workspace_bytes(long long nv) {
  const long long nb = (nv + kScanBlock - 1) / kScanBlock;
  return (size_t)(nv + nb) * 8 + 16;
}

int launch_weighted_points(uint64_t seed, uint64_t counter, const float* E, int G, long long n, float* xyz,
                           void* workspace, void* stream) {
  const hipStream_t st = (hipStream_t)stream;
  const long long nv = (long long)G * G * G, nb = (nv + kScanBlock - 1) / kScanBlock;
  unsigned long long* Q = (unsigned long long*)workspace;
  unsigned long long* S = Q + nv;
  unsigned* emax = (unsigned*)(S + nb);
  int rc = 0;
  if (E) {  // else the prefix sums of an earlier call are in the workspace
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, st, emax);
    if ((rc = check_launch())) return rc;
    hipLaunchKernelGGL(weight_max_kernel, dim3(grid_blocks(nv, 256, device_cus() * 8)), dim3(256), 0, st, E, nv,
                       emax);
    if ((rc = check_launch())) return rc;
    hipLaunchKernelGGL(weight_scan_kernel, dim3((unsigned)nb), dim3(kScanThreads), 0, st, E, nv, emax, Q, S);
    if ((rc = check_launch())) return rc;
    hipLaunchKernelGGL(block_offsets_kernel, dim3(1), dim3(kScanThreads), 0, st, S, nb);
    if ((rc = check_launch())) return rc;
    hipLaunchKernelGGL(add_offsets_kernel, dim3(grid_blocks(nv, 256, device_cus() * 8)), dim3(256), 0, st, Q, nv,
                       S);
    if ((rc = check_launch())) return rc;
  }
  if (n == 0) return 0;
  hipLaunchKernelGGL(weighted_points_kernel, dim3(grid_blocks(n, 256, device_cus() * 16)), dim3(256), 0, st,
                     (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)counter, (uint32_t)(counter >> 32), Q, G, nv,
                     n, xyz);
  return check_launch();
}

int launch_weighted_points_multi(uint64_t seed, uint64_t counter, int G, int n_grids, const int64_t* n_per_grid,
                                 float* xyz, const void* workspace, size_t stride, void* stream) {
  MultiDraw md;
  md.n = n_grids;
  md.start[0] = 0;
  for (int k = 0; k < n_grids; ++k) md.start[k + 1] = md.start[k] + n_per_grid[k];
  for (int k = n_grids + 1; k <= kMaxDrawGrids; ++k) md.start[k] = md.start[n_grids];
  const long long n = md.start[n_grids];
  if (n == 0) return 0;
  hipLaunchKernelGGL(weighted_points_multi_kernel, dim3(grid_blocks(n, 256, device_cus() * 16)), dim3(256), 0,
                     (hipStream_t)stream, (uint32_t)seed, (uint32_t)(seed >> 32), (unsigned long long)counter,
                     (const char*)workspace, (unsigned long long)stride, G, (long long)G * G * G, md, xyz);
  return check_launch();
}

const char* last_hip_error() { return g_hip_err; }

int launch_render(const NetDev& net, int prec, const TFDev& tf, const ViewBatch& views, const MarchDev& m,
                  float* out, unsigned long long* stats, void* stream) {
  switch (prec) {
    case kF32: return launch_render_p0(net, tf, views, m, out, stats, stream);
    case kF16: return launch_render_p1(net, tf, views, m, out, stats, stream);
    case kBF16: return launch_render_p2(net, tf, views, m, out, stats, stream);
  }
  return 1;
}

int launch_points(const NetDev& net, int prec, const float* xyz, long long n, int key, float key_w, float* out_d,
                  float* out_g, int gmode, void* stream) {
  switch (prec) {
    case kF32: return launch_points_p0(net, xyz, n, key, key_w, out_d, out_g, gmode, stream);
    case kF16: return launch_points_p1(net, xyz, n, key, key_w, out_d, out_g, gmode, stream);
    case kBF16: return launch_points_p2(net, xyz, n, key, key_w, out_d, out_g, gmode, stream);
  }
  return 1;
}

int launch_render_dense(const float* vol, int nx, int ny, int nz, const TFDev& tf, const ViewBatch& vb,
                        const MarchDev& m, float* out, unsigned long long* stats, void* stream) {
  // Segments per step and ray: 4 while that gives 48 tiles per CU, more in
  // smaller launches, whose rays would leave the GPU idle (ms at 4 / 8 / 16 /
  // 64 segments: two 800 x 600 views 1.20 / 1.18 / 1.38 / 3.39, one of 512^2
  // 0.59 / 0.54 / 0.54 / 1.21, 200 x 150 0.24 / 0.15 / 0.11 / 0.16, 40 x 40
  // 0.27 / 0.16 / 0.10 / 0.06; before 1.31, 1.03, 0.45 and 0.60). Phong starts at
  // 8 (two 800 x 600 views 7.8 / 7.5 / 7.7, before 9.4): its seven samples keep
  // the lanes' loads in flight. Where every ray ends early (RayEnds) no more
  // than an eighth of its segments at over a wave per SIMD, down to 2, where a wave
  // sets up 64 rays (ends after 4 samples, 1536x1152: Phong 0.27 -> 0.15 ms, before
  // 0.16); where a ray may end early, no more than a quarter of them in the largest
  // launches, whose rays need no splitting.
  const RayEnds ends = ray_ends(tf, m);
  DenseTile dt = {m.phong ? 3 : 2};
  const double chord = m.fixed_steps > 0 ? m.fixed_steps : 3.4641016 / m.step;
  auto tiles_at = [&](int ls) {
    const DenseTile t = {ls};
    const long long tw = 1 << t.lw(), th = 1 << t.lh();
    return ((vb.width + tw - 1) / tw) * ((vb.height + th - 1) / th) * vb.n_views;
  };
  const bool solid = ends.last < HUGE_VAL;
  double limit = solid ? ends.last / 8 : HUGE_VAL;
  if (!solid && tiles_at(2) >= device_cus() * 192ll) limit = ends.first / 4;
  while (dt.ls > 1 && (double)(1 << dt.ls) > limit) --dt.ls;
  while (dt.ls < 6 && tiles_at(dt.ls) < device_cus() * (dt.ls <= 2 ? 48ll : (dt.ls == 3 ? 12ll : 4ll)) &&
         (double)(4 << dt.ls) <= chord &&
         ((double)(2 << dt.ls) <= limit || tiles_at(dt.ls + 1) <= device_cus() * 4ll))
    ++dt.ls;
  if (tiles_at(dt.ls) > 1ll << 25) dt.ls = 1;  // tiles of 64 rays near the grid's limit
  const int tw = 1 << dt.lw(), th = 1 << dt.lh();
  const int tx = (vb.width + tw - 1) / tw, ty = (vb.height + th - 1) / th;
  const long long tiles = (long long)tx * ty * vb.n_views;
  long long blocks = (tiles + 3) / 4;
  if (blocks % 8) blocks += 8 - blocks % 8;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kDenseThreads), 0, (hipStream_t)stream, vol, nx, ny, nz, tf,
                       vb, m, out, stats, tx, ty, dt);
  };
  const bool big = (long long)nx * ny * nz >= (1ll << 29);  // 2^31 bytes
  // (colours that are not finite are composited as a shade's are)
  bool finite = true;
  for (int q = 0; q < 4; ++q) {
    finite = finite && std::isfinite(tf.base[q]);
    for (int j = 0; j < tf.n_seg; ++j) finite = finite && std::isfinite(tf.delta[j][q]);
  }
  if (m.phong || !finite) big ? go(dense_march_kernel<true, true>) : go(dense_march_kernel<true, false>);
  else big ? go(dense_march_kernel<false, true>) : go(dense_march_kernel<false, false>);
  return check_launch();
}

int launch_dense_points(const float* vol, int nx, int ny, int nz, const float* xyz, long long n, float* out,
                        float* out_g, void* stream) {
  const int blocks = grid_blocks(n, 256, device_cus() * 16);
  hipLaunchKernelGGL(dense_points_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, vol, nx, ny, nz,
                     xyz, n, out, out_g);
  return check_launch();
}

int launch_sample_points(uint64_t seed, uint64_t counter, long long n, float* xyz, void* stream) {
  const int blocks = grid_blocks(n, 256, device_cus() * 16);
  hipLaunchKernelGGL(sample_points_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, (uint32_t)seed,
                     (uint32_t)(seed >> 32), (uint32_t)counter, (uint32_t)(counter >> 32), n, xyz);
  return check_launch();
}

int launch_ssim(const float* a, const float* b, int width, int height, int n_images, float* out, void* stream) {
  Window11 win;
  double g[11], sum = 0.0;
  for (int i = 0; i < 11; ++i) {
    g[i] = exp(-(double)((i - 5) * (i - 5)) / (2.0 * 1.5 * 1.5));
    sum += g[i];
  }
  for (int i = 0; i < 11; ++i) win.g[i] = (float)(g[i] / sum);
  const long long tiles = (long long)n_images * ((height - 10 + kSsimH - 1) / kSsimH) * ((width - 10 + kSsimW - 1) / kSsimW);
  hipLaunchKernelGGL(ssim_kernel, dim3(grid_blocks(tiles, 1, device_cus() * 64)), dim3(256), 0,
                     (hipStream_t)stream, (const float4*)a, (const float4*)b, width, height, n_images, win, out);
  return check_launch();
}

int launch_quantize(const float* src, long long n, int channels, unsigned char* codes, float* dequant,
                    void* stream) {
  hipLaunchKernelGGL(channel_range_kernel, dim3(channels), dim3(256), 0, (hipStream_t)stream, src, n, channels,
                     dequant);
  int rc = check_launch();
  if (rc) return rc;
  const long long count = n * channels;
  hipLaunchKernelGGL(encode_u8_kernel, dim3(grid_blocks(count, 256, device_cus() * 16)), dim3(256), 0,
                     (hipStream_t)stream, src, count, channels, (const float*)dequant, codes);
  return check_launch();
}

int launch_cast(const float* src, void* dst, long long count, int dst_dtype, void* stream) {
  const int blocks = grid_blocks(count, 256, device_cus() * 16);
  if (dst_dtype == kF16)
    hipLaunchKernelGGL(cast_f16_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, src,
                       (_Float16*)dst, count);
  else
    hipLaunchKernelGGL(cast_bf16_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, src, (__bf16*)dst,
                       count);
  return check_launch();
}

}  // namespace fvsrn_detail
