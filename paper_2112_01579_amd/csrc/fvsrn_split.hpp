// Value-mode evaluation of an FP32 sine network on the FP16 matrix cores.
//
// The FP32 MFMA runs at 1/16 of the FP16 rate, so an FP32 network on it is
// bound by the matrix cores (study network: 360 16x16x4 MFMAs = 11,520 cycles
// per 64 samples). Every operand here is instead the sum of two FP16 values,
// x = hi + lo with hi = fp16(x), lo = fp16(x - hi), and each product is
// hi hi + hi lo + lo hi, accumulated in FP32 (lo lo, at most 2^-22 of the
// product, is left out): 132 FP16 MFMAs and 40 FP32 ones = 3,400 cycles.
// Two FP16 mantissas and the sign of lo hold 23 of FP32's 24 bits, provided
// that lo stays clear of FP16's smallest step of 2^-24:
//  * B operands are sines and cosines (the hidden activations and the Fourier
//    features), at most 1: the split is off by at most 2^-24, half of the
//    sine instruction's own error;
//  * A operands are weights, scaled per output row by the power of two that
//    puts the row's largest into [2^13, 2^14); the accumulator is multiplied
//    by the inverse (exact) in the FMA that adds the bias. A hidden row that
//    holds an infinity or NaN is not scaled and gives NaN, as the sine of the
//    infinite sum does in FP32. An output row with infinities becomes their
//    signs times an infinite scale: the logit is infinite and the density 0 or 1, as
//    in FP32 (several infinities: by the sign of their channels' sum).
//  * inputs without a bound -- the latent vector and the position -- and their
//    weights stay on the FP32 MFMA, where they are off the VALU's path.
// A sine of 2^-k so keeps 23 - k bits (its low half ends at 2^-25). Measured
// against FP64 (2^19 points, six seeds, relative L2) the densities' error is 0.95 to 0.99
// of the FP32 MFMA's on average and at most 1.05 for one seed, with all weights doubled
// 0.87 to 0.92: one K32 step rounds its accumulator once, eight K4 steps eight times.
//
// The kernel is then VALU-bound (the sines, the splits, the corner sums), and
// the input rows are built in the layout in which the MFMA reads them: lane
// 16 g + n of an N-tile builds quarter g of the features and of the latent
// channels of the tile's sample n, so that only the sample's position, cell
// and fractions go through LDS (32 bytes a sample instead of a 272-byte row:
// 12 waves per CU instead of 7). Measured, before and now: 10^6 random points
// of the study network 145 -> 71 us, 2^24 points 2.14 -> 0.98 ms (17 G/s), its
// trained 8 x 1024^2 orbit 331 -> 158 ms; VALU busy 75% and MFMA 44% in the render.
#pragma once
#include "fvsrn_net.hpp"

namespace fvsrn_detail {

template <class CF>
struct SplitGeo {
  static constexpr int C = CF::C, F = CF::F, L = CF::L;
  static constexpr int MT = C / 16;            // M-tiles of a hidden layer
  static constexpr int HS = (MT + 1) / 2;      // K32 steps of a hidden layer (zero past C)
  static constexpr int OCT = L / 4;            // octaves per lane group
  static constexpr int NF = 6 * OCT;           // Fourier features per lane group
  static constexpr int S0 = (NF + 7) / 8;      // K32 steps of the Fourier features
  static constexpr int Q = F / 4;              // K4 steps of the latent vector; one more for x y z 1
  static constexpr int FRAG = 2 * kWave * 16;  // bytes of one hi and one lo fragment
  static constexpr int W0F = MT * S0 * FRAG, W0L = MT * (Q + 1) * kWave * 4;
  static constexpr int L0 = W0F + W0L + C * 4;            // Fourier fragments, FP32 fragments, row scales
  static constexpr int WH = MT * HS * FRAG;
  static constexpr int HID = WH + 2 * C * 4;              // fragments, row scales, biases
  static constexpr int WO = 4 * HS * FRAG;
  static constexpr int OUT = WO + 32;                     // fragments, row scales, biases
  __host__ __device__ static constexpr int weight_bytes(int H) { return L0 + (H - 1) * HID + OUT; }
  static constexpr int WAVE_BYTES = 2 * kWave * 16;       // position and cell of a wave's samples
};

// hi + lo of a pair. A mixed-precision FMA forms a - hi without converting hi
// back, which the compiler selects only while it does not know that the factor
// is -1. (Written as instructions, which also round to FP16, the pair took two
// instead of three, but the compiler places wait states between an MFMA and
// the vector instructions that reuse its registers only where it selects them
// itself; it also schedules these better: a 1024 x 768 view of the study
// network 11.35 -> 11.15 ms, 10^6 points 73 -> 71 us.)
__device__ inline void split2(float a, float b, h2& hi, h2& lo) {
  float neg = -1.0f;
  asm("" : "+s"(neg));
  hi = __builtin_convertvector((f2{a, b}), h2);
  lo = h2{(_Float16)__builtin_fmaf((float)hi[0], neg, a), (_Float16)__builtin_fmaf((float)hi[1], neg, b)};
}

// The power of two that undoes a row's scale, from the row's largest weight.
__device__ inline float row_unscale(float m) {
  const int e = (int)(__float_as_uint(m) >> 23);  // m >= 0 or NaN
  if (e == 0 || e >= 255) return 1.0f;
  const int k = e - 127 - 13;
  return __uint_as_float((unsigned)((k < -100 ? -100 : k) + 127) << 23);
}
__device__ inline float pow2_inverse(float p) { return __uint_as_float((254u << 23) - __float_as_uint(p)); }

// Weights in LDS. K slot j of step s in lane group g is channel 32 s + 4 g + j
// for j < 4 and 32 s + 16 + 4 g + j - 4 otherwise, the order in which a D
// fragment packs into a B fragment.
template <class CF>
__device__ void stage_split(const NetDev& nd, char* smem) {
  using SG = SplitGeo<CF>;
  constexpr int C = SG::C, F = SG::F, L = SG::L, MT = SG::MT, HS = SG::HS, S0 = SG::S0, Q = SG::Q;
  constexpr int K0 = 3 + F + 6 * L;
  const int H = nd.H, NO = nd.NO;
  const float* w = nd.weights;
  const int tid = threadIdx.x, nt = blockDim.x;
  auto layer = [&](int i) { return w + (long long)C * K0 + C + (long long)(i - 1) * (C * C + C); };  // W_i, i >= 1
  auto hid = [&](int i) { return smem + SG::L0 + (i - 1) * SG::HID; };
  char* out = smem + SG::L0 + (H - 1) * SG::HID;
  // row scales: 16 lanes per row find its largest weight
  const int rows = C * H + 4;
  for (int r = tid >> 4; r < rows; r += nt >> 4) {
    const int i = r / C, o = r % C, l = tid & 15;
    const float sc = i < H ? kInv2Pi : 1.0f;
    const float* row = i == 0 ? w + (long long)o * K0 + 3 + F : layer(i) + (long long)o * C;
    const int cols = i == 0 ? 6 * L : ((i < H || o < NO) ? C : 0);
    float m = 0.0f;
    for (int k = l; k < cols; k += 16) {
      const float a = fabsf(row[k] * sc);
      m = a > m || !(a == a) ? a : m;
    }
    for (int off = 8; off > 0; off >>= 1) {
      const float a = __shfl_xor(m, off, 64);
      m = a > m || !(a == a) ? a : m;
    }
    if (l == 0) {
      float* dst = reinterpret_cast<float*>(i == 0 ? smem + SG::W0F + SG::W0L : (i < H ? hid(i) + SG::WH : out + SG::WO));
      dst[o] = i == H && !(m < HUGE_VALF) ? m : row_unscale(m);
    }
  }
  __syncthreads();
  // one thread per lane of a fragment: its 8 K slots, hi and lo
  auto put = [](char* base, int frag, int lane, const float v[8]) {
    h8* p = reinterpret_cast<h8*>(base + frag * SG::FRAG) + lane;
    h8 hi, lo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      hi[j] = (_Float16)v[j];
      lo[j] = (_Float16)(v[j] - (float)hi[j]);
    }
    p[0] = hi;
    p[kWave] = lo;
  };
  // K slots of row o (C weights from `row`, 16-byte aligned) in step s of lane group g
  auto load8k = [&](const float* row, int s, int g, float sc, float v[8]) {
    const f4 a = *reinterpret_cast<const f4*>(row + 32 * s + 4 * g);
    const f4 b = 32 * s + 16 < C ? *reinterpret_cast<const f4*>(row + 32 * s + 16 + 4 * g) : f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = a[j] * sc;
      v[4 + j] = b[j] * sc;
    }
  };
  const float* s0 = reinterpret_cast<const float*>(smem + SG::W0F + SG::W0L);
  for (int e = tid; e < MT * S0 * kWave; e += nt) {
    const int lane = e & 63, s = (e >> 6) % S0, mt = (e >> 6) / S0;
    const int o = 16 * mt + (lane & 15);
    const float up = pow2_inverse(s0[o]);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // feature f of group g: octave g OCT + f / 6, sine (x, y, z) then cosine
      const int f = 8 * s + j, k = (lane >> 4) * SG::OCT + f / 6, a = f % 6;
      const int col = a < 3 ? 3 * k + a : 3 * L + 3 * k + (a - 3);
      v[j] = f < SG::NF ? w[(long long)o * K0 + 3 + F + col] * kInv2Pi * up : 0.0f;
    }
    put(smem, e >> 6, lane, v);
  }
  float* wl = reinterpret_cast<float*>(smem + SG::W0F);
  for (int e = tid; e < MT * (Q + 1) * kWave; e += nt) {
    const int lane = e & 63, q = (e >> 6) % (Q + 1), mt = (e >> 6) / (Q + 1);
    const int o = 16 * mt + (lane & 15), g = lane >> 4;
    const float v = q < Q ? w[(long long)o * K0 + 3 + Q * g + q]
                          : (g < 3 ? w[(long long)o * K0 + g] : w[(long long)C * K0 + o]);
    wl[e] = v * kInv2Pi;
  }
  for (int i = 1; i < H; ++i) {
    const float* Wi = layer(i);
    char* p = hid(i);
    float* sb = reinterpret_cast<float*>(p + SG::WH);
    for (int e = tid; e < MT * HS * kWave; e += nt) {
      const int lane = e & 63, s = (e >> 6) % HS, mt = (e >> 6) / HS;
      const int o = 16 * mt + (lane & 15);
      float v[8];
      load8k(Wi + o * C, s, lane >> 4, kInv2Pi, v);
      const float up = pow2_inverse(sb[o]);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] *= up;
      put(p, e >> 6, lane, v);
    }
    for (int e = tid; e < C; e += nt) sb[C + e] = Wi[C * C + e] * kInv2Pi;
  }
  const float* Wo = layer(H);
  float* so = reinterpret_cast<float*>(out + SG::WO);
  for (int e = tid; e < 4 * HS * kWave; e += nt) {
    const int lane = e & 63, s = (e >> 6) % HS, t = (e >> 6) / HS;
    const int o = (lane & 15) - 4 * t;  // output o of N-tile t sits in row 4t + o
    float v[8] = {};
    if (o >= 0 && o < NO) {
      // a row with infinities: they become +-1, the others (all but) 0
      const bool inf = so[o] == HUGE_VALF;
      const float most = inf ? 1.0f : 65504.0f;
      load8k(Wo + o * C, s, lane >> 4, inf ? 0x1p-126f : pow2_inverse(so[o]), v);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = __builtin_amdgcn_fmed3f(v[j], -most, most);
    }
    put(out, e >> 6, lane, v);
  }
  if (tid < 4) so[4 + tid] = tid < NO ? Wo[NO * C + tid] : 0.0f;
}

// A sample's position and cell, read by the four lanes that build its inputs.
struct SplitTile {
  f4* pos;   // x, y, z, 1
  f4* cell;  // element offset of the cell's first vertex (bits), fractions

  __device__ inline void put(int lane, const LatentSrc& ls, int F, float x, float y, float z) {
    int ix, iy, iz;
    float fx, fy, fz;
    axis_cell(x, ls.R, ix, fx);
    axis_cell(y, ls.R, iy, fy);
    axis_cell(z, ls.R, iz, fz);
    const unsigned R = (unsigned)ls.R, sx = (unsigned)F, sy = R * sx, sz = R * sy;
    pos[lane] = f4{x, y, z, 1.0f};
    cell[lane] = f4{__uint_as_float(vertex_offset(ix, iy, iz, sx, sy, sz)), fx, fy, fz};
  }
};

// Channels [g F/4, (g + 1) F/4) of one keyframe's latent vector of a cell
// (quarter g), in two phases so that the features are built while the
// corner loads are in flight. D: the grid's storage type.
template <int F, int D>
struct QuarterGather {
  static constexpr int Q = F / 4;  // channels
  static_assert(Q == 2 || Q == 4, "F = 8 or 16");
  static constexpr int BYTES = Q * (D == kF32 ? 4 : (D == kF16 ? 2 : 1)), DW = (BYTES + 3) / 4;
  unsigned raw[8][DW];

  __device__ inline void load(const void* grid, const LatentSrc& ls, int g, unsigned base, const unsigned off[8]) {
    constexpr unsigned esz = D == kF32 ? 4 : (D == kF16 ? 2 : 1);
    const __amdgpu_buffer_rsrc_t r = grid_rsrc(grid, ls.bytes);
    const unsigned at = (base + (unsigned)(Q * g)) * esz;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const unsigned so = off[c] * esz;
      if constexpr (BYTES == 16) {
        const uint4 v = load16(r, at, so);
        raw[c][0] = v.x, raw[c][1] = v.y, raw[c][2] = v.z, raw[c][3] = v.w;
      } else if constexpr (BYTES == 8) {
        const uint2 v = load8(r, at, so);
        raw[c][0] = v.x, raw[c][1] = v.y;
      } else if constexpr (BYTES == 4) {
        raw[c][0] = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, at, so, 0);
      } else {
        raw[c][0] = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, at, so, 0);
      }
    }
  }

  // d[c] = u . corner c (a uint8 grid's offsets drop out of the derivative)
  __device__ inline void dot(const float* u, int g, const float* dq, float d[8]) const {
    float us[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) us[j] = D == kU8 ? u[j] * dq[2 * (Q * g + j) + 1] : u[j];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      d[c] = 0.0f;
#pragma unroll
      for (int j = 0; j < Q; ++j) d[c] = fmaf(us[j], value(c, j), d[c]);
    }
  }

  // channel j of corner c (a code of a uint8 grid)
  __device__ inline float value(int c, int j) const {
    if constexpr (D == kU8) return (float)((raw[c][0] >> (8 * j)) & 0xffu);
    else if constexpr (D == kF16) return (float)__builtin_bit_cast(h2, raw[c][j / 2])[j % 2];
    else return __uint_as_float(raw[c][j]);
  }

  // z += sum over corners of w * corner
  __device__ inline void add(const float w[8], int g, const float* dq, float* z) const {
    if constexpr (D == kU8) {
      float acc[Q] = {}, wsum = 0.0f;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
#pragma unroll
        for (int j = 0; j < Q; ++j) acc[j] = fmaf(w[c], value(c, j), acc[j]);
        wsum += w[c];
      }
      const float* d = dq + 2 * Q * g;
#pragma unroll
      for (int j = 0; j < Q; ++j) z[j] += fmaf(d[2 * j + 1], acc[j], d[2 * j] * wsum);
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int j = 0; j < Q; ++j) z[j] = fmaf(w[c], value(c, j), z[j]);
    }
  }
};

// Layer 0's B operands of N-tiles tp, tp + 1: the Fourier features (hi, lo),
// the latent channels and the position's component of this lane's group.
template <class CF, int D, int NT, int NS>
__device__ inline void split_inputs(const SplitTile& st, const LatentSrc& ls, int tp, h8 bh[NT][NS], h8 bl[NT][NS],
                                    float z[NT][CF::F / 4], float tail[NT]) {
  using SG = SplitGeo<CF>;
  constexpr int F = SG::F, S0 = SG::S0, Q = SG::Q;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, n = lane & 15;
  // The corner loads run with a vertex's channels in adjacent lanes (lane
  // 4 s + q: quarter q of sample s), so that one L1 lookup serves four lanes;
  // in the operands' layout each lane's load is a lookup of its own, and
  // random points were bound by them (36 per point, one per CU and cycle).
  const int gs = lane >> 2, gq = lane & 3;
  const unsigned R = (unsigned)ls.R;
  unsigned off[8];
  corner_offsets((unsigned)F, R * F, R * R * F, off);
  // revolutions of this group's first octave per world unit
  const float oct = 0.5f * (float)(1 << (SG::OCT * g));
  QuarterGather<F, D> qg[NT];
  f4 cf[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    cf[u] = st.cell[16 * (tp + u) + gs];
    qg[u].load(ls.g0, ls, gq, __float_as_uint(cf[u][0]), off);
  }
  // keep the features below between the loads and their use
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const f4 p = st.pos[16 * (tp + u) + n];
    float f[8 * S0];
#pragma unroll
    for (int j = SG::NF; j < 8 * S0; ++j) f[j] = 0.0f;
#pragma unroll
    for (int k = 0; k < SG::OCT; ++k)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float ph = p[a] * (oct * (float)(1 << k));
        f[6 * k + a] = sin_rev(ph);
        f[6 * k + 3 + a] = cos_rev(ph);
      }
#pragma unroll
    for (int s = 0; s < S0; ++s)
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        h2 hi = {}, lo = {};
        if (8 * s + j < SG::NF) split2(f[8 * s + j], f[8 * s + j + 1], hi, lo);
        bh[u][s][j] = hi[0];
        bh[u][s][j + 1] = hi[1];
        bl[u][s][j] = lo[0];
        bl[u][s][j + 1] = lo[1];
      }
    tail[u] = reinterpret_cast<const float*>(st.pos + 16 * (tp + u) + n)[g];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const float x0 = 1.0f - cf[u][1], y0 = 1.0f - cf[u][2], z0 = 1.0f - cf[u][3];
    const float xy[4] = {x0 * y0, cf[u][1] * y0, x0 * cf[u][2], cf[u][1] * cf[u][2]};
#pragma unroll
    for (int j = 0; j < Q; ++j) z[u][j] = 0.0f;
#pragma unroll
    for (int key = 0; key < 2; ++key) {
      if (key == 1 && !ls.g1) break;
      const float kw = key == 0 ? ls.w0 : ls.w1, za = z0 * kw, zb = cf[u][3] * kw;
      float w[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) w[c] = xy[c & 3] * (c < 4 ? za : zb);
      if (key == 1) qg[u].load(ls.g1, ls, gq, __float_as_uint(cf[u][0]), off);
      qg[u].add(w, gq, key == 0 ? ls.dq0 : ls.dq1, z[u]);
    }
    // quarter g of sample n from lane 4 n + g
#pragma unroll
    for (int j = 0; j < Q; ++j)
      z[u][j] = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (4 * n + g), __float_as_int(z[u][j])));
  }
}

// A pair of N-tiles on its way through the network: the B operands (hi, lo) and
// the accumulators.
template <class CF>
struct SplitPair {
  using SG = SplitGeo<CF>;
  using P16 = PrecT<kF16>;
  using P32 = PrecT<kF32>;
  static constexpr int MT = SG::MT, HS = SG::HS, S0 = SG::S0, Q = SG::Q, NT = 2, NS = HS > S0 ? HS : S0;
  f4 acc[NT][MT], lin[NT][MT];  // row-scaled; layer 0: latent, position and bias
  h8 bh[NT][NS], bl[NT][NS];

  // hi hi + hi lo + lo hi of one K32 step
  __device__ inline void mma3(const h8* frag, int s, f4 c[NT]) const {
    const int lane = threadIdx.x & 63;
    const h8 ah = frag[lane], al = frag[kWave + lane];
#pragma unroll
    for (int u = 0; u < NT; ++u) c[u] = P16::mma(al, bh[u][s], c[u]);
#pragma unroll
    for (int u = 0; u < NT; ++u) c[u] = P16::mma(ah, bl[u][s], c[u]);
#pragma unroll
    for (int u = 0; u < NT; ++u) c[u] = P16::mma(ah, bh[u][s], c[u]);
  }

  template <int STEPS>
  __device__ inline void product(const h8* frags) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      f4 c[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) c[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < STEPS; ++s) mma3(frags + (mt * STEPS + s) * 2 * kWave, s, c);
#pragma unroll
      for (int u = 0; u < NT; ++u) acc[u][mt] = c[u];
    }
  }

  // layer 0 of N-tiles tp, tp + 1: inputs and products
  __device__ inline void layer0(const char* wsm, const SplitTile& st, const LatentSrc& ls, int tp) {
    const int lane = threadIdx.x & 63;
    const float* WL = reinterpret_cast<const float*>(wsm + SG::W0F);
    float z[NT][Q], tail[NT];
    if (ls.dtype == kF32) split_inputs<CF, kF32, NT, NS>(st, ls, tp, bh, bl, z, tail);
    else if (ls.dtype == kF16) split_inputs<CF, kF16, NT, NS>(st, ls, tp, bh, bl, z, tail);
    else split_inputs<CF, kU8, NT, NS>(st, ls, tp, bh, bl, z, tail);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float* wl = WL + mt * (Q + 1) * kWave + lane;
#pragma unroll
      for (int u = 0; u < NT; ++u) lin[u][mt] = P32::mma(wl[Q * kWave], tail[u], f4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < NT; ++u) lin[u][mt] = P32::mma(wl[q * kWave], z[u][q], lin[u][mt]);
    }
    product<S0>(reinterpret_cast<const h8*>(wsm));
  }

  __device__ inline void hidden(const char* p) { product<HS>(reinterpret_cast<const h8*>(p)); }

  // The next B operands: sin of the layer's pre-activations (revolutions), row
  // scales (then biases) at `us`; with DER also act' (cos) into der.
  template <bool DER>
  __device__ inline void pack(const f4* us, bool first, f4 (*der)[MT]) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
#pragma unroll
      for (int s = 0; s < HS; ++s) {
        bh[u][s] = bl[u][s] = h8{};
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const int mt = 2 * s + v;
          if (mt >= MT) continue;
          const f4 sc = us[4 * mt + g], ad = first ? lin[u][mt] : us[SG::C / 4 + 4 * mt + g];
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            const float r0 = fmaf(acc[u][mt][j], sc[j], ad[j]), r1 = fmaf(acc[u][mt][j + 1], sc[j + 1], ad[j + 1]);
            h2 hi, lo;
            split2(sin_rev(r0), sin_rev(r1), hi, lo);
            if constexpr (DER) {
              der[u][mt][j] = cos_rev(r0);
              der[u][mt][j + 1] = cos_rev(r1);
            }
            bh[u][s][4 * v + j] = hi[0];
            bh[u][s][4 * v + j + 1] = hi[1];
            bl[u][s][4 * v + j] = lo[0];
            bl[u][s][4 * v + j + 1] = lo[1];
          }
        }
      }
    }
  }

  // the output layer at p, into out
  __device__ inline void output(const char* p, int tp, f4 out[NT]) const {
    const h8* WO = reinterpret_cast<const h8*>(p) + (threadIdx.x & 63);
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const h8* frag = WO + ((tp + u) * HS + s) * 2 * kWave;
        const h8 ah = frag[0], al = frag[kWave];
        out[u] = P16::mma(al, bh[u][s], out[u]);
        out[u] = P16::mma(ah, bl[u][s], out[u]);
        out[u] = P16::mma(ah, bh[u][s], out[u]);
      }
  }
};

// The network on the wave's 64 samples; returns the output pre-activations of
// this lane's own sample.
template <class CF>
__device__ inline f4 mlp_split(const char* wsm, const SplitTile& st, const LatentSrc& ls, int H) {
  using SG = SplitGeo<CF>;
  constexpr int NT = 2;
  f4 out[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) out[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  for (int tp = 0; tp < 4; tp += NT) {
    SplitPair<CF> sp;
    sp.layer0(wsm, st, ls, tp);
    sp.template pack<false>(reinterpret_cast<const f4*>(wsm + SG::W0F + SG::W0L), true, nullptr);
    const char* p = wsm + SG::L0;
    for (int i = 1; i < H; ++i) {
      sp.hidden(p);
      sp.template pack<false>(reinterpret_cast<const f4*>(p + SG::WH), false, nullptr);
      p += SG::HID;
    }
    sp.output(p, tp, out);
  }
  const f4* so = reinterpret_cast<const f4*>(wsm + SG::L0 + (H - 1) * SG::HID + SG::WO);
  const f4 us = so[0], bo = so[1];
  f4 y = out[0] + out[1];
#pragma unroll
  for (int j = 0; j < 4; ++j) y[j] = fmaf(y[j], us[j], bo[j]);
  return y;
}

// ------------------------------------------------------------- adjoint
//
// Reverse-mode gradient of an FP32 sine network of up to kSplitAdjLayers
// layers (Sec. 6). The forward pass is mlp_split's, keeping every layer's act'
// in registers. The deltas have no bound, so the backward products take three
// BF16 values per operand (x = b0 + b1 + b2 to 27 bits, any exponent) and the
// six largest of their products: 6/16 of the FP32 MFMA's cycles. W_0^T's rows
// are ordered so that lane 16 g + n receives the derivatives of the inputs that it
// built (its Fourier features, its latent channels, the position's component
// g) and contracts them with the inputs' Jacobian itself; the four partial
// gradients of a sample meet in LDS. Measured, FP32 MFMA and here: gradients at 10^6
// points of the study network 324 -> 161 us (65,537 points 38 -> 28, of which
// 20 are the weights' way into LDS), at c = 48, F = 16, H = 2 416 -> 215, an 800 x 600
// Phong view of the study network 34.4 -> 16.5 ms; bound by the VALU
// (sines, splits; 60% busy) and by 8 waves per CU. Against FP64 the gradients' error is
// 0.75 to 0.80 of the FP32 MFMA's (c = 32 networks, six seeds).
// Above four layers the derivatives do not fit in registers.
constexpr int kSplitAdjLayers = 4;

template <class CF>
struct SplitAdjGeo {
  using SG = SplitGeo<CF>;
  static constexpr int SLOTS = SG::NF + SG::Q + 1;  // inputs per lane group: features, channels, one of x y z
  static constexpr int MB = (SLOTS + 3) / 4;        // M-tiles of W_0^T: slot 4 m + j of group g in row 4 g + j
  static constexpr int FRAG = 3 * kWave * 16;       // b0, b1, b2
  static constexpr int WB = SG::MT * SG::HS * FRAG;
  static constexpr int WB0 = MB * SG::HS * FRAG;
  __host__ __device__ static constexpr int back_bytes(int H) { return (H - 1) * WB + WB0 + SG::C * 4; }
  static constexpr int GRAD_BYTES = 4 * kWave * 16;  // a wave's partial gradients [sample][group]
};

// b0 + b1 + b2 of eight values.
__device__ inline void split3(const float v[8], b8& b0, b8& b1, b8& b2) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    b0[j] = (__bf16)v[j];
    const float r = v[j] - (float)b0[j];
    b1[j] = (__bf16)r;
    b2[j] = (__bf16)(r - (float)b1[j]);
  }
}

template <class CF>
__device__ void stage_split_adj(const NetDev& nd, char* p) {
  using SG = SplitGeo<CF>;
  using SA = SplitAdjGeo<CF>;
  constexpr int C = SG::C, F = SG::F, L = SG::L, MT = SG::MT, HS = SG::HS, Q = SG::Q;
  constexpr int K0 = 3 + F + 6 * L;
  const int H = nd.H;
  const float* w = nd.weights;
  const int tid = threadIdx.x, nt = blockDim.x;
  // a fragment's lane: rows r, K slots of step s; value(row, output channel)
  auto stage = [&](char* base, int mtiles, auto value) {
    for (int e = tid; e < mtiles * HS * kWave; e += nt) {
      const int lane = e & 63, s = (e >> 6) % HS, m = (e >> 6) / HS;
      const int g = lane >> 4;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ch = 32 * s + (j < 4 ? 4 * g + j : 16 + 4 * g + (j - 4));
        v[j] = ch < C ? value(m, lane & 15, ch) : 0.0f;
      }
      b8 b0, b1, b2;
      split3(v, b0, b1, b2);
      b8* f = reinterpret_cast<b8*>(base + (e >> 6) * SA::FRAG) + lane;
      f[0] = b0;
      f[kWave] = b1;
      f[2 * kWave] = b2;
    }
  };
  for (int i = 1; i < H; ++i) {
    const float* Wi = w + (long long)C * K0 + C + (long long)(i - 1) * (C * C + C);
    stage(p + (i - 1) * SA::WB, MT, [&](int m, int r, int ch) { return Wi[ch * C + 16 * m + r]; });
  }
  p += (H - 1) * SA::WB;
  stage(p, SA::MB, [&](int m, int r, int ch) {
    const int g = r >> 2, slot = 4 * m + (r & 3);
    int col;  // column of W_0
    if (slot < SG::NF) {
      const int k = g * SG::OCT + slot / 6, a = slot % 6;
      col = 3 + F + (a < 3 ? 3 * k + a : 3 * L + 3 * k + (a - 3));
    } else if (slot < SG::NF + Q) {
      col = 3 + Q * g + (slot - SG::NF);
    } else {
      col = slot == SG::NF + Q && g < 3 ? g : -1;
    }
    return col < 0 ? 0.0f : w[(long long)ch * K0 + col];
  });
  float* wo = reinterpret_cast<float*>(p + SA::WB0);
  const float* Wo = w + (long long)C * K0 + C + (long long)(H - 1) * (C * C + C);
  for (int e = tid; e < C; e += nt) wo[e] = Wo[e];
}

// The latent channels' share of a sample's gradient, this lane's quarter gq of
// the channels: ul = dy/d(channel). The trilinear weights are differentiated
// per axis, zero outside the domain.
template <class CF, int D>
__device__ inline void split_latent_vjp(const SplitTile& st, const LatentSrc& ls, int s, int gq, const float* ul,
                                        float t[3]) {
  constexpr int F = CF::F, Q = F / 4;
  const unsigned R = (unsigned)ls.R;
  unsigned off[8];
  corner_offsets((unsigned)F, R * F, R * R * F, off);
  const f4 cf = st.cell[s], p = st.pos[s];
  const float scale = 0.5f * (float)(ls.R - 1);
  float d3[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) d3[a] = (p[a] < -1.0f || p[a] > 1.0f) ? 0.0f : scale;
  const float X[2] = {1.0f - cf[1], cf[1]}, Y[2] = {1.0f - cf[2], cf[2]}, Z[2] = {1.0f - cf[3], cf[3]};
  t[0] = t[1] = t[2] = 0.0f;
#pragma unroll
  for (int key = 0; key < 2; ++key) {
    if (key == 1 && !ls.g1) break;
    QuarterGather<F, D> qg;
    qg.load(key == 0 ? ls.g0 : ls.g1, ls, gq, __float_as_uint(cf[0]), off);
    float d[8];
    qg.dot(ul, gq, key == 0 ? ls.dq0 : ls.dq1, d);
    float v[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int lo = i & 1, hi = i >> 1;
      v[0] = fmaf(Y[lo] * Z[hi], d[1 + 2 * lo + 4 * hi] - d[2 * lo + 4 * hi], v[0]);
      v[1] = fmaf(X[lo] * Z[hi], d[lo + 2 + 4 * hi] - d[lo + 4 * hi], v[1]);
      v[2] = fmaf(X[lo] * Y[hi], d[lo + 2 * hi + 4] - d[lo + 2 * hi], v[2]);
    }
    const float kw = key == 0 ? ls.w0 : ls.w1;
#pragma unroll
    for (int a = 0; a < 3; ++a) t[a] = fmaf(kw * d3[a], v[a], t[a]);
  }
}

// The network and its gradient on the wave's 64 samples: returns the logit of
// this lane's own sample and leaves its partial gradients (of the logit) in
// grad[4 lane .. 4 lane + 3].
template <class CF, int HH>
__device__ inline float mlp_split_adj(const char* wsm, const char* bsm, const SplitTile& st, f4* grad,
                                      const LatentSrc& ls) {
  using SG = SplitGeo<CF>;
  using SA = SplitAdjGeo<CF>;
  using P16 = PrecT<kF16>;
  using PB = PrecT<kBF16>;
  constexpr int MT = SG::MT, HS = SG::HS, NT = 2;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, n = lane & 15;
  const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  const float oct = 0.5f * (float)(1 << (SG::OCT * g));
  const f4* wo = reinterpret_cast<const f4*>(bsm + (HH - 1) * SA::WB + SA::WB0);
  f4 out[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) out[u] = zero;
  for (int tp = 0; tp < 4; tp += NT) {
    SplitPair<CF> sp;
    sp.layer0(wsm, st, ls, tp);
    f4 der[HH][NT][MT];
    const char* p = wsm + SG::L0;
#pragma unroll
    for (int i = 0; i < HH; ++i) {
      if (i > 0) {
        sp.hidden(p);
        sp.template pack<true>(reinterpret_cast<const f4*>(p + SG::WH), false, der[i]);
        p += SG::HID;
      } else {
        sp.template pack<true>(reinterpret_cast<const f4*>(wsm + SG::W0F + SG::W0L), true, der[0]);
      }
    }
    sp.output(p, tp, out);
    // backward: e_i = dy/dh_{i+1} * act'(x_i), dy/dh_i = W_i^T e_i
    f4 e[NT][MT];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) e[u][mt] = wo[4 * mt + g] * der[HH - 1][u][mt];
    b8 b[3][NT][HS];
    auto split_e = [&]() {
#pragma unroll
      for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int s = 0; s < HS; ++s) {
          float v[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] = 2 * s + j / 4 < MT ? e[u][2 * s + j / 4 < MT ? 2 * s + j / 4 : 0][j % 4] : 0.0f;
          split3(v, b[0][u][s], b[1][u][s], b[2][u][s]);
        }
    };
    // rows of one M-tile: the six largest products, smallest first
    auto mma6 = [&](const char* base, f4 c[NT]) {
#pragma unroll
      for (int u = 0; u < NT; ++u) c[u] = zero;
#pragma unroll
      for (int s = 0; s < HS; ++s) {
        const b8* f = reinterpret_cast<const b8*>(base + s * SA::FRAG) + lane;
        const b8 a0 = f[0], a1 = f[kWave], a2 = f[2 * kWave];
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = PB::mma(a2, b[0][u][s], c[u]);
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = PB::mma(a1, b[1][u][s], c[u]);
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = PB::mma(a0, b[2][u][s], c[u]);
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = PB::mma(a1, b[0][u][s], c[u]);
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = PB::mma(a0, b[1][u][s], c[u]);
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = PB::mma(a0, b[0][u][s], c[u]);
      }
    };
#pragma unroll
    for (int i = HH - 1; i >= 1; --i) {
      split_e();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f4 c[NT];
        mma6(bsm + (i - 1) * SA::WB + mt * HS * SA::FRAG, c);
#pragma unroll
        for (int u = 0; u < NT; ++u) e[u][mt] = c[u] * der[i - 1][u][mt];
      }
    }
    split_e();
    float v[NT][4 * SA::MB];  // dy/d(input) of this lane's slots
#pragma unroll
    for (int m = 0; m < SA::MB; ++m) {
      f4 c[NT];
      mma6(bsm + (HH - 1) * SA::WB + m * HS * SA::FRAG, c);
#pragma unroll
      for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][4 * m + j] = c[u][j];
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int s0 = 16 * (tp + u);
      const f4 pp = st.pos[s0 + n];
      float ga[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) ga[a] = g == a ? v[u][SG::NF + SG::Q] : 0.0f;
#pragma unroll
      for (int k = 0; k < SG::OCT; ++k) {
        const float wk = k2Pi * (oct * (float)(1 << k));
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const float ph = pp[a] * (oct * (float)(1 << k));
          ga[a] = fmaf(wk, fmaf(v[u][6 * k + a], cos_rev(ph), -v[u][6 * k + 3 + a] * sin_rev(ph)), ga[a]);
        }
      }
      // channels to the lane that holds the quarter's corners, and back
      float ul[SG::Q], t[3];
#pragma unroll
      for (int j = 0; j < SG::Q; ++j)
        ul[j] = __int_as_float(
            __builtin_amdgcn_ds_bpermute(4 * (16 * (lane & 3) + (lane >> 2)), __float_as_int(v[u][SG::NF + j])));
      const int s = s0 + (lane >> 2), gq = lane & 3;
      if (ls.dtype == kF32) split_latent_vjp<CF, kF32>(st, ls, s, gq, ul, t);
      else if (ls.dtype == kF16) split_latent_vjp<CF, kF16>(st, ls, s, gq, ul, t);
      else split_latent_vjp<CF, kU8>(st, ls, s, gq, ul, t);
#pragma unroll
      for (int a = 0; a < 3; ++a)
        ga[a] += __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (4 * n + g), __float_as_int(t[a])));
      grad[4 * (s0 + n) + g] = f4{ga[0], ga[1], ga[2], 0.0f};
    }
  }
  const f4* so = reinterpret_cast<const f4*>(wsm + SG::L0 + (HH - 1) * SG::HID + SG::WO);
  return fmaf(out[0][0] + out[1][0], so[0][0], so[1][0]);
}

}  // namespace fvsrn_detail
