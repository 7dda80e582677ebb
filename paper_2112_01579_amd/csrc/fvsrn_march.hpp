// Fused fV-SRN ray-march and point-evaluation kernels, templated on the
// network configuration and shading mode; the per-precision units
// (fvsrn_march.hip, fvsrn_adjoint.hip) instantiate and dispatch them.
//
// Render: one wavefront owns a tile of rays -- 8x8 pixels without shading,
// 4x4 pixels (four lanes per ray: value and three tangents) for forward-mode
// gradients, 4x2 pixels (eight lanes per ray: centre and six central-difference
// neighbours) for finite-difference gradients; a network that predicts its own
// gradient (four outputs) and the adjoint (reverse-mode) gradient shade from
// 8x8 tiles like the unshaded render. Per march step every lane builds its
// input row, the wave runs the MLP on the matrix cores, and the ray-owning
// lanes map the density through the transfer function and composite front to
// back (Sec. 3, Sec. 4), stopping when the transmittance falls below the
// termination threshold.
#pragma once
#include "fvsrn_adjoint.hpp"
#include "fvsrn_split.hpp"

namespace fvsrn_detail {

namespace {

// Shading modes of the render kernel: none, forward-mode gradient, central
// differences, the network's predicted gradient, the adjoint (Sec. 6).
enum { kShadeNone = 0, kShadeFwd = 1, kShadeFD = 2, kShadePred = 3, kShadeAdj = 4 };

constexpr int kLdsBytes = 160 * 1024;
constexpr int kRayBytes = 9 * 8 * kWave;  // a wave's FP64 rays in LDS (split render)

// FP32 sine networks with the octave features evaluate on the FP16 matrix
// cores (fvsrn_split.hpp) wherever values are needed, and for the adjoint of up
// to kSplitAdjLayers layers while its two sets of weight fragments leave LDS
// for at least a wave per SIMD of the render, whose waves also keep their rays
// there (10.5 KB a wave; c = 48: up to H = 3, with F = 16 up to 2). The points, which take
// 6 KB a wave, follow the same rule: at c = 48, F = 8, H = 3 their eight waves take
// 197 us for 10^6 gradients against 276 on the FP32 MFMA; one layer more would
// leave them four, which has not been measured. Forward-mode tangents, the other
// adjoints and the other activations stay on the FP32 MFMA.
template <class CF, int MODE, int HH = 0>
constexpr bool use_split() {
  return CF::P == kF32 && CF::ACT == kSine && CF::TE == 0 && !CF::FM && MODE != kShadeFwd &&
         (MODE != kShadeAdj || (HH > 0 && HH <= kSplitAdjLayers &&
                                SplitGeo<CF>::weight_bytes(HH) + SplitAdjGeo<CF>::back_bytes(HH) +
                                        4 * (SplitGeo<CF>::WAVE_BYTES + kRayBytes + SplitAdjGeo<CF>::GRAD_BYTES) <=
                                    kLdsBytes));
}

// Waves per workgroup cap (sets the VGPR budget through the launch bounds):
// value-mode networks with the packed FP16 latent path fit 4 waves per SIMD
// (<= 128 VGPRs), other value-mode networks 3 (<= 168). Forward mode: 3 for
// the c = 32 and c = 48 FP16 networks on a packed grid (spills of a few
// registers; with the persistent launch the third wave hides more than the
// spills cost: c = 48 measured 122 -> 106 ms per frame), 2 otherwise.
// Central differences add the neighbour offsets and the gradient gather to
// the value-mode network; with F = 16 channels gathered in FP32 (c = 48, or
// an FP16 network on an FP32 grid) that needs 2 waves per SIMD, c = 48 with
// the packed latent path 3. The adjoint keeps every layer's activation
// derivatives of two N-tiles in registers: 3 waves per SIMD for the c = 32
// FP16 network on a packed grid (151 -> 138 ms on the study views), 2
// otherwise (c = 48 measured 47 -> 48 ms at 3).
// FP32 networks off the split path add the FP64 ray of their sample positions
// (about 10 registers).
template <class CF, int MODE, bool POINTS = false, int HH = 0>
constexpr int max_waves() {
  if (use_split<CF, MODE, HH>()) return MODE == kShadeAdj ? 8 : 12;
  if (MODE == kShadeAdj) return (CF::P == kF16 && CF::C == 32 && CF::G16) ? 12 : 8;
  if (MODE == kShadeFwd) return (CF::P == kF16 && CF::C <= 48 && CF::G16) ? 12 : 8;
  if (MODE == kShadeFD) {
    if (CF::F == 16 && (CF::C == 48 || (CF::P != kF32 && !CF::G16))) return 8;
    return (CF::G16 && CF::C == 32) ? 16 : 12;
  }
  // FP32 c = 48 network with F = 16: the FP64 sample positions need a few
  // more registers than 168
  if (CF::P == kF32 && CF::C == 48 && CF::F == 16) return 8;
  // point evaluation on an FP16 grid holds the corners over the feature build
  if (POINTS && CF::GK == 1) return 12;
  return CF::G16 ? 16 : 12;
}

// Render tile geometry per shading mode: log2 of the lanes per ray, and of the
// tile's edges in rays when a wave takes 2^sh segments of a ray per step
// (unshaded: 8x8 rays, then 8x4, 4x4, ...).
template <int MODE>
struct TileShape {
  static constexpr int LOG_LPR = (MODE == kShadeFwd) ? 2 : (MODE == kShadeFD ? 3 : 0);
  static constexpr int LPR = 1 << LOG_LPR;
  __host__ __device__ static constexpr int log_w(int sh) { return (7 - LOG_LPR - sh) / 2; }
  __host__ __device__ static constexpr int log_h(int sh) { return (6 - LOG_LPR - sh) / 2; }
};
// LDS bytes of a workgroup besides its waves' input tiles: the forward weight
// fragments, and for the adjoint the transposed ones.
template <class CF, int MODE, int HH = 0>
__host__ __device__ int fixed_lds_bytes(int H) {
  using G = typename CF::G;
  if constexpr (use_split<CF, MODE, HH>())
    return SplitGeo<CF>::weight_bytes(H) + (MODE == kShadeAdj ? SplitAdjGeo<CF>::back_bytes(H) : 0);
  else return G::weight_bytes(H) + (MODE == kShadeAdj ? G::back_bytes(H) : 0);
}

// LDS bytes of one wave's input tile; the split render also keeps its lanes'
// FP64 rays there, which would cost 18 registers over the MLP.
template <class CF, int MODE, bool POINTS = false, int HH = 0>
constexpr int wave_lds_bytes() {
  if constexpr (use_split<CF, MODE, HH>())
    return SplitGeo<CF>::WAVE_BYTES + (POINTS ? 0 : kRayBytes) +
           (MODE == kShadeAdj ? SplitAdjGeo<CF>::GRAD_BYTES : 0);
  else return CF::G::FEAT_BYTES;
}

// Workgroups of wpb waves and shm bytes of LDS that a CU holds at once, by LDS
// and by the VGPR budget of max_waves. The CU deals a workgroup's waves out
// to its four SIMDs from the first one on, so a workgroup of w waves takes
// ceil(w / 4) of the first SIMD's wave slots: two workgroups of 6 waves do
// not fit where one of 12 does (measured: the second one waited for the
// first, 24.7 against 18.8 ms for a 1024^2 view of the FP32 study network).
template <class CF, int MODE, bool POINTS = false, int HH = 0>
int blocks_per_cu(int wpb, size_t shm) {
  const int by_lds = (int)(kLdsBytes / shm), by_regs = max_waves<CF, MODE, POINTS, HH>() / 4 / ((wpb + 3) / 4);
  return by_lds < by_regs ? by_lds : by_regs;
}

// Waves per workgroup. The VGPR budget of max_waves allows that many waves
// on a CU; every workgroup holds the weights once plus one input tile per
// wave in LDS. Pick the size that puts the most waves on a CU and, among
// sizes that reach it, the smallest: several smaller workgroups per CU let
// the dispatcher replace a finished one while another still runs its long
// rays (measured: 3 x 4 waves beat 1 x 12 waves by 12% on the BF16 path).
template <class CF, int MODE, bool POINTS = false, int HH = 0>
int waves_per_block(int H) {
  constexpr int cap = max_waves<CF, MODE, POINTS, HH>();
  const int wb = fixed_lds_bytes<CF, MODE, HH>(H);
  int best = 0, best_waves = 0;
  for (int w = 1; w <= cap; ++w) {
    const int waves =
        w * blocks_per_cu<CF, MODE, POINTS, HH>(w, (size_t)wb + w * wave_lds_bytes<CF, MODE, POINTS, HH>());
    if (waves > best_waves) {
      best = w;
      best_waves = waves;
    }
  }
  return best;
}

// Workgroups that the GPU holds at once.
template <class CF, int MODE, bool POINTS = false, int HH = 0>
long long resident_blocks(int wpb, size_t shm) {
  return (long long)device_cus() * blocks_per_cu<CF, MODE, POINTS, HH>(wpb, shm);
}

// ----------------------------------------------------- TF, camera, march

__device__ inline void tf_eval(const TFDev& tf, float d, float rgba[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) rgba[q] = tf.base[q];
  for (int j = 0; j < tf.n_seg; ++j) {
    const float w = __builtin_amdgcn_fmed3f(fmaf(d, tf.inv[j], tf.off[j]), 0.0f, 1.0f);
#pragma unroll
    for (int q = 0; q < 4; ++q) rgba[q] = fmaf(w, tf.delta[j][q], rgba[q]);
  }
}

// Segment i of a ray: midpoint parameter and length, the segment ending at
// t_end (the chord's end, or +inf for fixed-count marches: the last of their
// equal segments already ends there).
__device__ inline void segment(const Ray& r, int i, float t_end, float& tm, float& len) {
  const float a0 = fmaf((float)i, r.ds, r.t0);
  len = fminf(a0 + r.ds, t_end) - a0;
  tm = fmaf(0.5f, len, a0);
}

// Headlight Blinn-Phong (Sec. 6): light and view along -dir, normal = the
// normalized density gradient.
__device__ inline void phong(float rgba[4], float gx, float gy, float gz, const float dir[3], const MarchDev& m) {
  const float g2 = gx * gx + gy * gy + gz * gz;
  if (g2 >= 1e-12f) {  // |g| >= 1e-6
    // |n . l| with n = g / |g| by the hardware reciprocal square root, and
    // |n . l|^shininess as exp2(shininess * log2(.)) on the hardware
    // transcendentals (the library sqrt, divide and powf cost about 200
    // instructions per sample); the floor keeps log2 finite, so 0^0 = 1
    const float ndl = fabsf(gx * dir[0] + gy * dir[1] + gz * dir[2]) * __builtin_amdgcn_rsqf(g2);
    const float spec = m.ks * __builtin_amdgcn_exp2f(m.shininess * __builtin_amdgcn_logf(fmaxf(ndl, 1e-30f)));
    const float k = m.ka + m.kd * ndl;
    rgba[0] = fmaf(rgba[0], k, spec);
    rgba[1] = fmaf(rgba[1], k, spec);
    rgba[2] = fmaf(rgba[2], k, spec);
  }
}

// Front-to-back compositing of one segment (exact Beer-Lambert).
struct Accum {
  float T, C[3], A;
};

__device__ inline void composite(Accum& acc, const float rgba[4], float len) {
  const float trn = fast_exp(-rgba[3] * len);
  const float ta = acc.T * (1.0f - trn);
  acc.C[0] = fmaf(ta, rgba[0], acc.C[0]);
  acc.C[1] = fmaf(ta, rgba[1], acc.C[1]);
  acc.C[2] = fmaf(ta, rgba[2], acc.C[2]);
  acc.A += ta;
  acc.T *= trn;
}

// ------------------------------------------------------------- kernels

// A step of a wave takes 64 samples (16 in forward mode, 8 for central
// differences): one segment of each of its tile's rays, or,
// with seg_shift > 0 (small launches, see segments_log2), 2^seg_shift
// consecutive segments of fewer rays, composited by a prefix product over the
// ray's lanes.
// Persistent: as many workgroups as the CUs hold at once, each wave taking the
// tile of its own index (neighbours, whose rays are alike, on different CUs),
// then tiles from a device-wide counter until none is left (queue[0]: the next
// tile; queue[1]: waves done, so that the last one sets both back to zero). A
// launch with a wave per tile has no queue: the counter is one address for all
// XCDs and serves a wave in about 12 ns, which bounds launches of rays that end
// at once (128 x 96 of an opaque volume, 16 segments per step, 3,072 tiles: 117 us
// with the queue, 18 without; a 64^2 x 128 step view 75 and 47).
// Tile costs vary (empty, short and long rays): a static share of tiles per
// wave was measured 30% slower, and one tile per wave keeps a workgroup's
// LDS until its slowest wave ends, so the CUs ran at two thirds of their
// wave slots on average.
// HH: the network's layer count, compiled in for the adjoint (its saved
// activation derivatives are registers); 0 for the other modes.
// SEG: several segments per step (its code in the sample loop costs the
// unshaded and forward-mode kernels 3% where it does not run; the adjoint is
// compiled with it alone).
template <class CF, int MODE, int HH = 0, bool SEG = MODE == kShadeAdj>
__global__ __launch_bounds__((max_waves<CF, MODE, false, HH>() * 64)) void march_kernel(NetDev nd, TFDev tf, ViewBatch vb,
                                                                                  MarchDev m, float* out,
                                                                                  unsigned long long* stats,
                                                                                  unsigned int* queue,
                                                                                  int tiles_x, int tiles_y,
                                                                                  int seg_shift) {
  using G = typename CF::G;
  using E = typename CF::E;
  constexpr bool GRAD = MODE == kShadeFwd;  // network run in forward (tangent) mode
  constexpr bool FD = MODE == kShadeFD;
  constexpr int LPR = TileShape<MODE>::LPR;
  constexpr bool ADJ = MODE == kShadeAdj;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr bool SPLIT = use_split<CF, MODE, HH>();
  if constexpr (SPLIT) stage_split<CF>(nd, smem);
  else stage_weights<CF>(nd, smem);
  // transposed fragments (adjoint)
  char* bsm = smem + (SPLIT ? SplitGeo<CF>::weight_bytes(nd.H) : G::weight_bytes(nd.H));
  if constexpr (ADJ && SPLIT) stage_split_adj<CF>(nd, bsm);
  else if constexpr (ADJ) stage_backward_adj<CF>(nd, bsm);
  __syncthreads();
  // the wave index is wave-uniform; saying so keeps the tile, its camera and
  // the latent grid's buffer resource in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  const int tiles_per_view = tiles_x * tiles_y;
  const int n_tiles = tiles_per_view * vb.n_views;
  const int sh = SEG ? seg_shift : 0;                // log2 of the segments a ray takes per step
  const int q = lane % LPR;                          // role of the lane within its sample
  const int sl = (lane / LPR) & ((1 << sh) - 1);     // the sample's segment of its ray's step
  const int rl = (lane / LPR) >> sh;                 // ray within the tile
  const int lw = TileShape<MODE>::log_w(sh), lh = TileShape<MODE>::log_h(sh);
  const LaneRole role = GRAD ? grad_role(q) : value_role();
  // central differences: lane q = 1..6 evaluates the sample moved by +-h along
  // axis (q-1)/2 (odd q: +h); q = 0 and 7 evaluate the sample itself
  const float fh = (q & 1) ? m.fd_step : -m.fd_step;
  const float fd_off[3] = {FD && (q == 1 || q == 2) ? fh : 0.0f, FD && (q == 3 || q == 4) ? fh : 0.0f,
                           FD && (q == 5 || q == 6) ? fh : 0.0f};
  const float inv_2h = FD ? 0.5f / m.fd_step : 0.0f;
  const bool fixed = m.fixed_steps > 0;
  char* wlds = smem + fixed_lds_bytes<CF, MODE, HH>(nd.H) + wave * wave_lds_bytes<CF, MODE, false, HH>();
  E* feat = reinterpret_cast<E*>(wlds);
  E* myrow = feat + lane * G::ROW;
  SplitTile st = {reinterpret_cast<f4*>(wlds), reinterpret_cast<f4*>(wlds) + kWave};
  double* lray = reinterpret_cast<double*>(wlds + 2 * kWave * sizeof(f4)) + lane;  // SPLIT: this lane's ray
  f4* lgrad = reinterpret_cast<f4*>(wlds + 2 * kWave * sizeof(f4) + kRayBytes);    // and the partial gradients
  unsigned long long n_samp = 0, n_hit = 0, iters = 0;
  const int n_waves = gridDim.x * wpb;
  for (int tile = wave * gridDim.x + blockIdx.x; tile < n_tiles;
       tile = queue ? n_waves + next_tile(queue, lane) : n_tiles) {
    const int v = tile / tiles_per_view;
    const int tr = tile % tiles_per_view;
    const int px = ((tr % tiles_x) << lw) + (rl & ((1 << lw) - 1));
    const int py = ((tr / tiles_x) << lh) + (rl >> lw);
    const CamDev& cam = vb.cam[v];
    const LatentSrc ls = make_latent_src(nd, cam.key, cam.key_w);
    const bool in_img = px < vb.width && py < vb.height;
    // FP32 networks take every sample position from the FP64 ray, rounded
    // once: an FP32 o + t d (the eye a few units from the box) is off by a
    // few 1e-7, which the highest Fourier octaves turn into visible density
    // and shading-normal errors; FP16/BF16 rounding dwarfs it
    constexpr bool kPosF64 = CF::P == kF32;
    const RayD rayd = make_ray_d(cam, in_img ? px : 0, in_img ? py : 0, vb.width, vb.height, m);
    const Ray ray = round_ray(rayd);
    if constexpr (SPLIT) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lray[a * kWave] = rayd.o[a];
        lray[(3 + a) * kWave] = rayd.d[a];
      }
      lray[6 * kWave] = rayd.t0;
      lray[7 * kWave] = rayd.t1;
      lray[8 * kWave] = rayd.ds;
      wave_lds_sync();
    }
    bool active = in_img && ray.hit && ray.nseg > 0;
    float tfe[G::TIN > 0 ? G::TIN : 1];  // the view's time inputs (time-encoded networks)
    if constexpr (G::TIN > 0) time_features<CF::TE>(cam.tau, tfe);
    Accum acc = {1.0f, {0.0f, 0.0f, 0.0f}, 0.0f};
    const float t_end = fixed ? INFINITY : ray.t1;
    // position and length of segment ii. A lane whose ray has ended keeps
    // sampling its (finite) ray past the end: the cell clamps keep its loads
    // inside the grid and its result is not composited. The FP64 positions
    // of FP32 networks are zeroed for such lanes.
    auto sample_at = [&](int ii, bool act, float& sx, float& sy, float& sz, float& len) {
      if constexpr (kPosF64) {
        float pp[3];
        if constexpr (SPLIT) {
          const RayD r = {{lray[0], lray[kWave], lray[2 * kWave]},
                          {lray[3 * kWave], lray[4 * kWave], lray[5 * kWave]},
                          lray[6 * kWave], lray[7 * kWave], lray[8 * kWave], 0, true};
          segment_d(r, ii, fixed, fd_off, pp, len);
        } else {
          segment_d(rayd, ii, fixed, fd_off, pp, len);
        }
        sx = act ? pp[0] : 0.0f;
        sy = act ? pp[1] : 0.0f;
        sz = act ? pp[2] : 0.0f;
      } else {
        float tm;
        segment(ray, ii, t_end, tm, len);
        sx = fmaf(tm, ray.d[0], ray.o[0]);
        sy = fmaf(tm, ray.d[1], ray.o[1]);
        sz = fmaf(tm, ray.d[2], ray.o[2]);
        if constexpr (FD) {
          sx += fd_off[0];
          sy += fd_off[1];
          sz += fd_off[2];
        }
      }
    };
    int i = sl;  // this lane's next segment of its ray
    active = active && (sh == 0 || i < ray.nseg);
    while (__builtin_amdgcn_ballot_w64(active)) {
      ++iters;
      float len, sx, sy, sz;
      sample_at(i, active, sx, sy, sz, len);
      if constexpr (SPLIT) st.put(lane, ls, CF::F, sx, sy, sz);
      else write_features<CF, GRAD>(myrow, ls, role, sx, sy, sz, tfe, nd.fm);
      wave_lds_sync();
      f4 yo;
      float ga[3] = {0.0f, 0.0f, 0.0f};
      if constexpr (ADJ && SPLIT) {
        yo[0] = mlp_split_adj<CF, HH>(smem, bsm, st, lgrad, ls);
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int a = 0; a < 3; ++a) ga[a] += lgrad[4 * lane + k][a];
      } else if constexpr (ADJ) {
        // the network and its adjoint; each row then holds dy/d(input row)
        yo[0] = mlp_tile_adj<CF, HH>(smem, bsm, feat);
        wave_lds_sync();
        input_vjp<CF>(myrow, ls, sx, sy, sz, ga);
      } else if constexpr (SPLIT) {
        yo = mlp_split<CF>(smem, st, ls, nd.H);
      } else {
        yo = mlp_tile<CF, GRAD>(smem, feat, nd.H, role);
      }
      wave_lds_sync();
      const float y = yo[0];
      float dens, gx = 0.0f, gy = 0.0f, gz = 0.0f;
      if constexpr (ADJ) {
        dens = sigmoid_f(y);
        const float sg = dens * (1.0f - dens);
        gx = sg * ga[0];
        gy = sg * ga[1];
        gz = sg * ga[2];
      } else if constexpr (MODE == kShadePred) {
        // outputs 1..3 are the gradient itself
        dens = sigmoid_f(y);
        gx = yo[1];
        gy = yo[2];
        gz = yo[3];
      } else if constexpr (GRAD) {
        // the quad's value lane holds the logit, lanes 1..3 its derivatives
        const float y0 = quad_bcast0(y);
        const float t1 = quad_bcast<1>(y), t2 = quad_bcast<2>(y), t3 = quad_bcast<3>(y);
        dens = sigmoid_f(y0);
        const float sg = dens * (1.0f - dens);
        gx = sg * t1;
        gy = sg * t2;
        gz = sg * t3;
      } else if constexpr (FD) {
        // gather the seven densities of the ray's lane group
        const float dl = sigmoid_f(y);
        const int b = lane & ~7;
        dens = __shfl(dl, b, 64);
        gx = (__shfl(dl, b + 1, 64) - __shfl(dl, b + 2, 64)) * inv_2h;
        gy = (__shfl(dl, b + 3, 64) - __shfl(dl, b + 4, 64)) * inv_2h;
        gz = (__shfl(dl, b + 5, 64) - __shfl(dl, b + 6, 64)) * inv_2h;
      } else {
        dens = sigmoid_f(y);
      }
      // branch-free: a lane without a sample composites a zero-length
      // segment, which changes nothing (transmittance factor exp(0) = 1)
      const bool comp = active && len > 0.0f;
      float rgba[4];
      tf_eval(tf, dens, rgba);
      if (m.phong) {
        if constexpr (SPLIT) {
          const float dir[3] = {(float)lray[3 * kWave], (float)lray[4 * kWave], (float)lray[5 * kWave]};
          phong(rgba, gx, gy, gz, dir, m);
        } else {
          phong(rgba, gx, gy, gz, ray.d, m);
        }
      }
      if (sh == 0) {
        composite(acc, rgba, comp ? len : 0.0f);
        i += comp ? 1 : 0;
        active = comp && !(acc.T < m.ert_eps) && i < ray.nseg;
      } else {
        // the ray's 2^sh segments front to back: each lane's transmittance
        // from the product of those before it, its colour into the lane's
        // own sum; a segment behind the one that ends the ray is left out
        const float trn = fast_exp(-rgba[3] * (comp ? len : 0.0f));
        float inc = trn;
        for (int d = 1; d < (1 << sh); d <<= 1) {
          const float up = __shfl_up(inc, d * LPR, 64);
          inc *= sl >= d ? up : 1.0f;
        }
        const float before = __shfl_up(inc, LPR, 64), last = __shfl(inc, lane | (((1 << sh) - 1) * LPR), 64);
        const float T = sl ? acc.T * before : acc.T;
        const bool in = comp && !(sl && T < m.ert_eps);
        if (in) {  // not by a weight of 0: behind the ray's end a shade may be infinite
          const float ta = T * (1.0f - trn);
#pragma unroll
          for (int a = 0; a < 3; ++a) acc.C[a] = fmaf(ta, rgba[a], acc.C[a]);
          acc.A += ta;
        }
        acc.T *= last;
        n_samp += in && q == 0 ? 1ull : 0ull;
        i += 1 << sh;
        active = active && !(acc.T < m.ert_eps) && i < ray.nseg;
      }
    }
    for (int d = 1; d < (1 << sh); d <<= 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) acc.C[a] += __shfl_xor(acc.C[a], d * LPR, 64);
      acc.A += __shfl_xor(acc.A, d * LPR, 64);
    }
    const bool owner = q == 0 && sl == 0;
    if (in_img && owner) {
      float4* o = reinterpret_cast<float4*>(out) + ((long long)v * vb.height + py) * vb.width + px;
      *o = make_float4(acc.C[0], acc.C[1], acc.C[2], acc.A);
    }
    if (sh == 0) n_samp += owner ? (unsigned long long)i : 0ull;
    n_hit += (owner && in_img && ray.hit && ray.nseg > 0) ? 1ull : 0ull;
  }
  if (stats) {
    for (int off = 32; off > 0; off >>= 1) {
      n_samp += __shfl_xor(n_samp, off, 64);
      n_hit += __shfl_xor(n_hit, off, 64);
    }
    if (lane == 0 && (n_samp | n_hit | iters)) {
      atomicAdd(stats, n_samp);
      atomicAdd(stats + 1, n_hit);
      atomicAdd(stats + 2, iters * (unsigned long long)(64 / LPR));
    }
  }
  if (queue) release_queue(queue, lane, n_waves);
}

// Point evaluation (PM): kShadeNone -- density, and with out_g set outputs
// 1..3 of a 4-output network (its predicted gradient); kShadeFwd -- density
// and forward-mode gradient; kShadeAdj -- density and adjoint gradient (HH:
// layer count, as for the render kernel).
template <class CF, int PM, int HH = 0>
__global__ __launch_bounds__((max_waves<CF, PM, true, HH>() * 64)) void points_kernel(NetDev nd, const float* xyz, long long n,
                                                                            int key, float key_w, float* out_d,
                                                                            float* out_g) {
  using G = typename CF::G;
  using E = typename CF::E;
  constexpr bool GRAD = PM == kShadeFwd;
  constexpr bool ADJ = PM == kShadeAdj;
  constexpr int PER = GRAD ? 16 : 64;  // points per wave step
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr bool SPLIT = use_split<CF, PM, HH>();
  if constexpr (SPLIT) stage_split<CF>(nd, smem);
  else stage_weights<CF>(nd, smem);
  char* bsm = smem + (SPLIT ? SplitGeo<CF>::weight_bytes(nd.H) : G::weight_bytes(nd.H));
  if constexpr (ADJ && SPLIT) stage_split_adj<CF>(nd, bsm);
  else if constexpr (ADJ) stage_backward_adj<CF>(nd, bsm);
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  char* wlds = smem + fixed_lds_bytes<CF, PM, HH>(nd.H) + wave * wave_lds_bytes<CF, PM, true, HH>();
  E* feat = reinterpret_cast<E*>(wlds);
  E* myrow = feat + lane * G::ROW;
  SplitTile st = {reinterpret_cast<f4*>(wlds), reinterpret_cast<f4*>(wlds) + kWave};
  const LaneRole role = GRAD ? grad_role(lane & 3) : value_role();
  const LatentSrc ls = make_latent_src(nd, key, key_w);
  float tfe[G::TIN > 0 ? G::TIN : 1];  // time inputs of the evaluation time
  if constexpr (G::TIN > 0) time_features<CF::TE>(nd.tau, tfe);
  const long long nchunks = (n + PER - 1) / PER;
  const int waves = blockDim.x >> 6;
  const long long stride = (long long)gridDim.x * waves;
  // The next chunk's positions are read once this chunk's input rows are
  // built: the HBM read then runs behind this chunk's MLP instead of in
  // series with the latent gather that it addresses.
  float nx = 0.0f, ny = 0.0f, nz = 0.0f;
  auto load_pos = [&](long long cc) {
    const long long j = cc * PER + (GRAD ? (lane >> 2) : lane);
    nx = ny = nz = 0.0f;
    if (cc < nchunks && j < n) {
      nx = xyz[3 * j];
      ny = xyz[3 * j + 1];
      nz = xyz[3 * j + 2];
    }
  };
  long long c = (long long)blockIdx.x * waves + wave;
  load_pos(c);
  for (; c < nchunks; c += stride) {
    const long long idx = c * PER + (GRAD ? (lane >> 2) : lane);
    const bool ok = idx < n;
    const float x = nx, y = ny, z = nz;
    if constexpr (SPLIT) st.put(lane, ls, CF::F, x, y, z);
    else write_features<CF, GRAD, CF::P != kF32 && CF::GK != 2 && !GRAD>(myrow, ls, role, x, y, z, tfe, nd.fm);
    wave_lds_sync();
    load_pos(c + stride);
    if constexpr (ADJ) {
      float o, ga[3] = {0.0f, 0.0f, 0.0f};
      if constexpr (SPLIT) {
        f4* lgrad = reinterpret_cast<f4*>(wlds + 2 * kWave * sizeof(f4));
        o = mlp_split_adj<CF, HH>(smem, bsm, st, lgrad, ls);
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int a = 0; a < 3; ++a) ga[a] += lgrad[4 * lane + k][a];
      } else {
        o = mlp_tile_adj<CF, HH>(smem, bsm, feat);
        wave_lds_sync();
        input_vjp<CF>(myrow, ls, x, y, z, ga);
      }
      wave_lds_sync();
      const float d = sigmoid_f(o), sg = d * (1.0f - d);
      if (ok) {
        if (out_d) out_d[idx] = d;
        out_g[3 * idx] = sg * ga[0];
        out_g[3 * idx + 1] = sg * ga[1];
        out_g[3 * idx + 2] = sg * ga[2];
      }
      continue;
    }
    f4 oo;
    if constexpr (SPLIT) oo = mlp_split<CF>(smem, st, ls, nd.H);
    else oo = mlp_tile<CF, GRAD>(smem, feat, nd.H, role);
    wave_lds_sync();
    const float o = oo[0];
    if constexpr (GRAD) {
      const float d = sigmoid_f(quad_bcast0(o));
      if (ok) {
        if (role.is_val) {
          if (out_d) out_d[idx] = d;
        } else {
          out_g[3 * idx + role.axis] = d * (1.0f - d) * o;
        }
      }
    } else if (ok) {
      if (out_d) out_d[idx] = sigmoid_f(o);
      if (out_g) {
        out_g[3 * idx] = oo[1];
        out_g[3 * idx + 1] = oo[2];
        out_g[3 * idx + 2] = oo[3];
      }
    }
  }
}

// ------------------------------------------------------------ launchers

// log2 of the consecutive segments of a ray that one step of a wave takes
// (see march_kernel), for `slots` waves resident on the GPU. Tiles of one
// segment per ray leave a small launch with idle waves and serial rays, and
// a middle-sized one with few tiles per wave and a long tail, so a ray takes
// more segments
//  * while that leaves no more tiles than wave slots (idle waves cost nothing);
//  * beyond, until there are 32 tiles per wave slot, up to 16 while the
//    one-segment tiles are under 4 per slot, else up to 4, and no more than the
//    segments that can end a ray (RayEnds), falling to an eighth of them at
//    two tiles per slot: a ray that ends early leaves the rest of its step unused,
//    and every tile costs a ray set-up and a draw. At least 4, or 2 from one to two
//    tiles per slot, where the transfer function has a transparent part: the
//    longest rays then set the time;
//  * never so many that a chord has under 4 steps.
// Measured, one segment against the rule's, ms per launch (a fitted network's
// densities, 256 steps per unit): 64^2 x 128 steps FP32 0.561 -> 0.047 (16); FP16 study
// network 320x240 2.67 -> 0.55, 512x384 2.88 -> 1.19 (16; 8: 1.22), 1024x768 4.5 (16)
// and 4.3 (8), 8 x 1024^2 52.2 (1; 4: 52.3, 16: 54.9); 1920x1080 c = 48 adjoint 48.1 ->
// 44.9 (4; 8: 44.6). Rays that end after 3 to 4 samples, before these limits
// and with them: FP16 320x240 0.318 -> 0.023 (one segment 0.058), 1024x768 2.33 -> 0.21
// (0.25); after 18 samples 1024x768 2.33 -> 0.38 (0.35).
template <int MODE>
int segments_log2(const ViewBatch& vb, const MarchDev& m, const RayEnds& ends, long long slots) {
  const int lw = TileShape<MODE>::log_w(0), lh = TileShape<MODE>::log_h(0);
  const long long tiles =
      (long long)((vb.width + (1 << lw) - 1) >> lw) * ((vb.height + (1 << lh) - 1) >> lh) * vb.n_views;
  const double chord = m.fixed_steps > 0 ? m.fixed_steps : 3.4641016 / m.step;  // segments of the longest
  const int most = tiles >= 4 * slots ? 2 : (lw + lh < 4 ? lw + lh : 4);
  double limit = ends.first / fmin(8.0, fmax(1.0, 4.0 * (double)tiles / (double)slots));
  if (ends.last < HUGE_VAL) limit = fmin(limit, ends.last / 8);
  else if (tiles < 2 * slots) limit = fmax(limit, tiles < slots ? 4 : 2);
  int sh = 0;
  while (sh < most && (double)(8 << sh) <= chord &&
         ((tiles << (sh + 1)) <= slots || ((tiles << sh) < 32 * slots && (double)(2 << sh) <= limit)))
    ++sh;
  return sh;
}

template <class CF, int MODE, int HH, bool SEG>
void launch_march(long long blocks, int wpb, size_t shm, const NetDev& nd, const TFDev& tf, const ViewBatch& vb,
                  const MarchDev& m, float* out, unsigned long long* stats, unsigned int* queue, int tx, int ty, int sh,
                  hipStream_t st) {
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)march_kernel<CF, MODE, HH, SEG>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    attr = true;
  }
  hipLaunchKernelGGL((march_kernel<CF, MODE, HH, SEG>), dim3((unsigned)blocks), dim3(wpb * 64), shm, st, nd, tf, vb, m,
                     out, stats, queue, tx, ty, sh);
}

template <class CF, int MODE, int HH = 0>
int launch_render_t(const NetDev& nd, const TFDev& tf, const ViewBatch& vb, const MarchDev& m, float* out,
                    unsigned long long* stats, hipStream_t st) {
  const int wpb = waves_per_block<CF, MODE, false, HH>(nd.H);
  if (wpb < 1) return kLaunchNoLds;
  const size_t shm =
      (size_t)fixed_lds_bytes<CF, MODE, HH>(nd.H) + (size_t)wpb * wave_lds_bytes<CF, MODE, false, HH>();
  // the workgroups the CUs hold at once, fewer for small launches
  const long long resident = resident_blocks<CF, MODE, false, HH>(wpb, shm);
  const int sh = segments_log2<MODE>(vb, m, ray_ends(tf, m), resident * wpb);
  const int tw = 1 << TileShape<MODE>::log_w(sh), th = 1 << TileShape<MODE>::log_h(sh);
  const int tx = (vb.width + tw - 1) / tw, ty = (vb.height + th - 1) / th;
  const long long tiles = (long long)tx * ty * vb.n_views;
  if (tiles > 0x7fffffffLL) return kLaunchTooLarge;
  const long long want = (tiles + wpb - 1) / wpb;
  const long long blocks = want < resident ? want : resident;
  if (blocks < 1) return 0;
  unsigned int* queue = nullptr;
  if (tiles > blocks * wpb && !(queue = tile_queue_slot())) return 2;
  if (sh > 0 || MODE == kShadeAdj)
    launch_march<CF, MODE, HH, true>(blocks, wpb, shm, nd, tf, vb, m, out, stats, queue, tx, ty, sh, st);
  else
    launch_march<CF, MODE, HH, MODE == kShadeAdj>(blocks, wpb, shm, nd, tf, vb, m, out, stats, queue, tx, ty, 0, st);
  return check_launch();
}

template <class CF, int PM, int HH = 0>
int launch_points_t(const NetDev& nd, const float* xyz, long long n, int key, float key_w, float* out_d,
                    float* out_g, hipStream_t st) {
  constexpr int PER = PM == kShadeFwd ? 16 : 64;
  const int wpb = waves_per_block<CF, PM, true, HH>(nd.H);
  if (wpb < 1) return kLaunchNoLds;
  const size_t shm = (size_t)fixed_lds_bytes<CF, PM, HH>(nd.H) + (size_t)wpb * wave_lds_bytes<CF, PM, true, HH>();
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)points_kernel<CF, PM, HH>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kLdsBytes);
    attr = true;
  }
  // persistent: the workgroups the GPU holds at once walk the chunks (equal
  // cost), so the weights are staged once per workgroup and no workgroup
  // waits for another to release its LDS
  const int blocks = grid_blocks((n + PER - 1) / PER, wpb, (int)resident_blocks<CF, PM, true, HH>(wpb, shm));
  hipLaunchKernelGGL((points_kernel<CF, PM, HH>), dim3(blocks), dim3(wpb * 64), shm, st, nd, xyz, n, key, key_w,
                     out_d, out_g);
  return check_launch();
}

}  // namespace

}  // namespace fvsrn_detail
