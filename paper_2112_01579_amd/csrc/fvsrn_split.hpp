// Value-mode evaluation of an FP32 sine network on the FP16 matrix cores.
//
// The FP32 MFMA runs at 1/16 of the FP16 rate, so an FP32 network on it is
// bound by the matrix cores (study network: 360 16x16x4 MFMAs = 11,520 cycles
// per 64 samples). Every operand here is instead the sum of two FP16 values,
// x = hi + lo with hi = fp16(x), lo = fp16(x - hi), and each product is
// hi hi + hi lo + lo hi, accumulated in FP32 (lo lo, below 2^-24 of the
// product, is left out): 132 FP16 MFMAs and 40 FP32 ones = 3,400 cycles.
// Two FP16 mantissas and the sign of lo hold 23 of FP32's 24 bits, provided
// that lo stays clear of FP16's smallest step of 2^-24:
//  * B operands are sines and cosines (the hidden activations and the Fourier
//    features), at most 1: the split is off by at most 2^-24, half of the
//    sine instruction's own error;
//  * A operands are weights, scaled per output row by the power of two that
//    puts the row's largest into [2^13, 2^14); the accumulator is multiplied
//    by the inverse (exact) in the FMA that adds the bias. (A row that holds
//    an infinity or NaN is not scaled and gives NaN.)
//  * inputs without a bound -- the latent vector and the position -- and their
//    weights stay on the FP32 MFMA, where they are off the VALU's path.
// Measured against FP64 (see the tests) the densities are no further off than
// the FP32 MFMA's: one K32 step rounds its accumulator once, eight K4 steps
// eight times.
//
// The kernel is then VALU-bound (the sines, the splits, the corner sums), and
// the input rows are built in the layout in which the MFMA reads them: lane
// 16 g + n of an N-tile builds quarter g of the features and of the latent
// channels of the tile's sample n, so that only the sample's position, cell
// and fractions go through LDS (32 bytes a sample instead of a 272-byte row:
// 12 waves per CU instead of 7). Measured, before and now: 10^6 random points
// of the study network 145 -> 77 us, 2^24 points 2.14 -> 1.0 ms (17 G/s), its
// 8 x 1024^2 views 164 -> 80 ms; VALU busy 80% in the render.
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
  __host__ __device__ static int weight_bytes(int H) { return L0 + (H - 1) * HID + OUT; }
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
      dst[o] = row_unscale(m);
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
    if (o >= 0 && o < NO) load8k(Wo + o * C, s, lane >> 4, pow2_inverse(so[o]), v);
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

  // z += sum over corners of w * corner
  __device__ inline void add(const float w[8], int g, const float* dq, float* z) const {
    if constexpr (D == kU8) {
      float acc[Q] = {}, wsum = 0.0f;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
#pragma unroll
        for (int j = 0; j < Q; ++j) acc[j] = fmaf(w[c], (float)((raw[c][0] >> (8 * j)) & 0xffu), acc[j]);
        wsum += w[c];
      }
      const float* d = dq + 2 * Q * g;
#pragma unroll
      for (int j = 0; j < Q; ++j) z[j] += fmaf(d[2 * j + 1], acc[j], d[2 * j] * wsum);
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          float v;
          if constexpr (D == kF16) v = (float)__builtin_bit_cast(h2, raw[c][j / 2])[j % 2];
          else v = __uint_as_float(raw[c][j]);
          z[j] = fmaf(w[c], v, z[j]);
        }
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

// The network on the wave's 64 samples; returns the output pre-activations of
// this lane's own sample.
template <class CF>
__device__ inline f4 mlp_split(const char* wsm, const SplitTile& st, const LatentSrc& ls, int H) {
  using SG = SplitGeo<CF>;
  using P16 = PrecT<kF16>;
  using P32 = PrecT<kF32>;
  constexpr int C = SG::C, MT = SG::MT, HS = SG::HS, S0 = SG::S0, Q = SG::Q, NT = 2;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4;
  const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  const h8* W0 = reinterpret_cast<const h8*>(wsm);
  const float* WL = reinterpret_cast<const float*>(wsm + SG::W0F);
  const f4* U0 = reinterpret_cast<const f4*>(wsm + SG::W0F + SG::W0L);
  constexpr int NS = HS > S0 ? HS : S0;
  f4 out[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) out[u] = zero;
  for (int tp = 0; tp < 4; tp += NT) {
    f4 acc[NT][MT], lin[NT][MT];  // Fourier part (row-scaled); latent, position and bias
    h8 bh[NT][NS], bl[NT][NS];
    {
      float z[NT][Q], tail[NT];
      if (ls.dtype == kF32) split_inputs<CF, kF32, NT, NS>(st, ls, tp, bh, bl, z, tail);
      else if (ls.dtype == kF16) split_inputs<CF, kF16, NT, NS>(st, ls, tp, bh, bl, z, tail);
      else split_inputs<CF, kU8, NT, NS>(st, ls, tp, bh, bl, z, tail);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float* wl = WL + mt * (Q + 1) * kWave + lane;
#pragma unroll
        for (int u = 0; u < NT; ++u) lin[u][mt] = P32::mma(wl[Q * kWave], tail[u], zero);
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int u = 0; u < NT; ++u) lin[u][mt] = P32::mma(wl[q * kWave], z[u][q], lin[u][mt]);
      }
    }
    // hi hi + hi lo + lo hi of one K32 step
    auto mma3 = [&](const h8* frag, int s, f4 c[NT]) {
      const h8 ah = frag[lane], al = frag[kWave + lane];
#pragma unroll
      for (int u = 0; u < NT; ++u) c[u] = P16::mma(al, bh[u][s], c[u]);
#pragma unroll
      for (int u = 0; u < NT; ++u) c[u] = P16::mma(ah, bl[u][s], c[u]);
#pragma unroll
      for (int u = 0; u < NT; ++u) c[u] = P16::mma(ah, bh[u][s], c[u]);
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      f4 c[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) c[u] = zero;
#pragma unroll
      for (int s = 0; s < S0; ++s) mma3(W0 + (mt * S0 + s) * 2 * kWave, s, c);
#pragma unroll
      for (int u = 0; u < NT; ++u) acc[u][mt] = c[u];
    }
    // the next B operands: sin of the layer's pre-activations (revolutions)
    auto pack = [&](const f4* unscale, auto add) {
#pragma unroll
      for (int u = 0; u < NT; ++u) {
#pragma unroll
        for (int s = 0; s < HS; ++s) {
          bh[u][s] = bl[u][s] = h8{};
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const int mt = 2 * s + v;
            if (mt >= MT) continue;
            const f4 us = unscale[4 * mt + g], ad = add(u, mt);
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
              h2 hi, lo;
              split2(sin_rev(fmaf(acc[u][mt][j], us[j], ad[j])), sin_rev(fmaf(acc[u][mt][j + 1], us[j + 1], ad[j + 1])),
                     hi, lo);
              bh[u][s][4 * v + j] = hi[0];
              bh[u][s][4 * v + j + 1] = hi[1];
              bl[u][s][4 * v + j] = lo[0];
              bl[u][s][4 * v + j + 1] = lo[1];
            }
          }
        }
      }
    };
    pack(U0, [&](int u, int mt) { return lin[u][mt]; });
    const char* p = wsm + SG::L0;
    for (int i = 1; i < H; ++i) {
      const h8* WH = reinterpret_cast<const h8*>(p);
      const f4* SB = reinterpret_cast<const f4*>(p + SG::WH);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f4 c[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) c[u] = zero;
#pragma unroll
        for (int s = 0; s < HS; ++s) mma3(WH + (mt * HS + s) * 2 * kWave, s, c);
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[u][mt] = c[u];
      }
      pack(SB, [&](int, int mt) { return SB[C / 4 + 4 * mt + g]; });
      p += SG::HID;
    }
    const h8* WO = reinterpret_cast<const h8*>(p);
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const h8* frag = WO + ((tp + u) * HS + s) * 2 * kWave + lane;
        const h8 ah = frag[0], al = frag[kWave];
        out[u] = P16::mma(al, bh[u][s], out[u]);
        out[u] = P16::mma(ah, bl[u][s], out[u]);
        out[u] = P16::mma(ah, bh[u][s], out[u]);
      }
  }
  const f4* so = reinterpret_cast<const f4*>(wsm + SG::L0 + (H - 1) * SG::HID + SG::WO);
  const f4 us = so[0], bo = so[1];
  f4 y = out[0] + out[1];
#pragma unroll
  for (int j = 0; j < 4; ++j) y[j] = fmaf(y[j], us[j], bo[j]);
  return y;
}

}  // namespace fvsrn_detail
