// Forward and backward pass of a training step as one kernel per batch row
// block: the chain of layers that follow one another on the same rows runs in
// registers (train_engine.h), and memory sees only what the weight gradients
// need, each layer's input and the gradient at its pre-activation, written
// once.  (Layer by layer, each of the 2 n launches read its input back from
// memory and waited for the one before.)
#include "device_common.h"
#include "runtime.h"
#include "train_engine.h"
#include "train_kernels.h"

namespace nedf {
namespace {

using chain::kstep_off;
using chain::gstore;
using chain::gstore1;
using eng::u32x4;

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Broadcast of one lane half's values to both.
__device__ __forceinline__ float from_lo(float x) {
  return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false)[0]);
}
__device__ __forceinline__ float from_hi(float x) {
  return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false)[1]);
}

// Regression form: encoding, the hidden layers, head, loss (Eq. 6) and the
// data gradients of a workgroup's 32 NW rows.  N input components (6
// Pluecker, 3 xyz), K0 K-steps of the first layer.
//
// Bound by the matrix cores (without its stores the kernel takes 118 us at
// 65,536 rows and 8 layers, 130 GFLOP at 1.1 PFLOP/s) and by the writes of
// the layers' inputs and gradients (15 x 33.6 MB + 16.8 MB): 158 us with
// both.  One launch per layer and direction took 300 us for the same work
// (each read its input back), the step 473 us against 318 us now.  The ring,
// the biases and the head weights in LDS allow one workgroup per compute
// unit; 8 waves keep two on each SIMD, 4 serve the batches that would leave
// compute units without a workgroup (chain_line_waves).
template <int N, int K0, int NW>
__global__ __launch_bounds__(64 * NW, 1) void k_chain_line(ChainLineArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[chain::RING];
  __shared__ __attribute__((aligned(16))) float s_bias[NEDF_MAX_LAYERS * 256];
  __shared__ __attribute__((aligned(16))) float s_head[2 * 256];
  __shared__ __attribute__((aligned(16))) float s_red[NW * 512];
  __shared__ __attribute__((aligned(16))) uint8_t s_bits[2 * NW * 1024];
  __shared__ __attribute__((aligned(16))) float s_row[4][32 * NW];
  __shared__ float s_label[2][32 * NW];
  constexpr int NT = 64 * NW;
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5, wave = t >> 6;
  const size_t row = (size_t(blockIdx.x) * NW + wave) * 32 + (lane & 31);
  const int NH = a.n_hidden;
  for (int i = t; i < NH * 256; i += NT) s_bias[i] = a.bias[i >> 8][i & 255];
  for (int i = t; i < 512; i += NT) s_head[i] = a.head_w[i];
  int cur = 0;
  const uint32_t tile_off = chain::tile_off(lane);
  // ---- encoding: features in natural order [p, sin(2^0 pi p), cos(2^0 pi p), ...]
  u32x4 B0u[K0];
  {
    float mu = 0.f, alpha;
    const float o[3] = {a.o_l[3 * row], a.o_l[3 * row + 1], a.o_l[3 * row + 2]};
    const float d[3] = {a.d_l[3 * row], a.d_l[3 * row + 1], a.d_l[3 * row + 2]};
    float p[6], plo[6] = {0, 0, 0, 0, 0, 0}, tperp = 0.0f;
    {
      float pl[6], pllo[6];
      line_of_local(o, d, pl, pllo, tperp);
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        p[c] = N == 6 ? pl[c] : c < 3 ? o[c] : 0.0f;
        plo[c] = N == 6 ? pllo[c] : 0.0f;
      }
    }
    const bool h = a.hit[row] != 0;
    alpha = h ? 1.0f : 0.0f;
    if (h) mu = (tperp - a.depth[row]) / a.bound;
    const int n_in = N * (1 + 2 * a.enc_L);
    auto feature = [&](int f, float& s, float& x, float& xlo, int& cosine) __attribute__((always_inline)) {
      const int q = f < N ? 0 : f - N, level = q / (2 * N), w = q % (2 * N);
      const int c = f < N ? f : w % N;
      s = float(1 << level);
      x = p[c];
      xlo = plo[c];
      cosine = w >= N ? 1 : 0;
    };
#pragma unroll
    for (int ks = 0; ks < K0; ++ks) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // half 0 takes feature 16 ks + j, half 1 feature 16 ks + 8 + j
        const int fa = 16 * ks + j, fb = fa + 8;
        float sa, xa, la, sb, xb, lb;
        int ca, cb;
        feature(fa, sa, xa, la, ca);
        feature(fb, sb, xb, lb, cb);
        const float s = half ? sb : sa, x = half ? xb : xa, lo = half ? lb : la;
        const float w = sinpi_hw(s * x, s * lo, half ? cb : ca);
        const int f = half ? fb : fa;
        v[j] = f < N ? x : f < n_in ? w : 0.0f;
      }
      B0u[ks] = u32x4{chain::pack2(v[0], v[1]), chain::pack2(v[2], v[3]), chain::pack2(v[4], v[5]),
                      chain::pack2(v[6], v[7])};
      gstore(a.Hin + size_t(blockIdx.x) * (32 * NW * 16 * K0), wave * (1024u * K0) + tile_off + kstep_off(ks), B0u[ks]);
    }
    // the labels wait in LDS (registers are short in the layers)
    if (half == 0) {
      s_label[0][32 * wave + lane] = mu;
      s_label[1][32 * wave + lane] = alpha;
    }
  }
  __syncthreads();
  chain::prime<K0, NW>(a.w[0], lds, cur);
  const uint32_t bias0 = eng::lds_offset(reinterpret_cast<const uint8_t*>(s_bias));
  bf16x8_t X[16], Y[16];
  // a row's place in the H and G arrays, a lane's word of a block pair's bits
  // from the workgroup's first row on
  const uint32_t row_off = wave * 16384u + tile_off;
  const uint32_t bit_off = (uint32_t(wave) * 256u + lane) * 4u;
  const size_t layer_elems = size_t(a.B) * 256, layer_bits = size_t(a.B) * 32;
  uint16_t* const H0 = a.H + size_t(blockIdx.x) * (32 * NW * 256);
  uint16_t* const G0 = a.G + size_t(blockIdx.x) * (32 * NW * 256);
  uint8_t* const bits0 = a.bits + size_t(blockIdx.x) * (32 * NW * 32);
  uint32_t bits = 0;
  // ReLU of a block, rounded, as the next operand; stored unless it is the
  // last layer's.  A quarter is two packed words; two quarters make a K-step.
  uint32_t ew[4];
  auto relu_quarter = [&](int q, const f32x16_t& v) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      ew[2 * (q & 1) + i] = chain::pack2(fmaxf(v[4 * q + 2 * i], 0.f), fmaxf(v[4 * q + 2 * i + 1], 0.f));
  };
  auto fwd_store = [&](int l) __attribute__((always_inline)) {
    return [&, l](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
      relu_quarter(q, v);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t m = chain::positive_bits(ew[2 * (q & 1) + i], fb & 1, 2 * q + i);
        bits = (fb & 1) || 2 * q + i ? bits | m : m;
      }
      if (q & 1) {
        const u32x4 k = chain::to_operand(ew[0], ew[1], ew[2], ew[3]);
        Y[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, k);
        gstore(H0 + l * layer_elems, row_off + kstep_off(2 * fb + q / 2), k);
      }
      if ((fb & 1) && q == 3) gstore1(bits0 + l * layer_bits, bit_off + 256 * (fb / 2), bits);
    };
  };
  auto fwd_last = [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
    relu_quarter(q, v);
    if (q & 1) Y[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, chain::to_operand(ew[0], ew[1], ew[2], ew[3]));
  };
  auto advance = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) X[i] = Y[i];
  };
  {
    bf16x8_t B0[K0];
#pragma unroll
    for (int i = 0; i < K0; ++i) B0[i] = __builtin_bit_cast(bf16x8_t, B0u[i]);
    chain::layer<K0, 8, 16, NW, true, 2, 0, 0>(B0, a.w[0], NH > 1 ? a.w[1] : nullptr, lds, cur, bias0, fwd_store(0));
    advance();
  }
  for (int l = 1; l + 1 < NH; ++l) {
    chain::layer<16, 8, 16, NW, true, 2, 2, 2>(X, a.w[l], a.w[l + 1], lds, cur, bias0 + l * 1024, fwd_store(l));
    advance();
  }
  if (NH > 1) {
    // backward weights follow in the ring
    chain::layer<16, 8, 16, NW, true, 0, 2, 2>(X, a.w[NH - 1], a.wt[NH - 1], lds, cur, bias0 + (NH - 1) * 1024, fwd_last);
    advance();
  }
  // signs of H_{l-1}, copied a layer ahead, into two places by turns
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  auto bits_at = [&](int l) __attribute__((always_inline)) { return s_bits + ((l & 1) * NW + uwave) * 1024; };
  auto fetch_bits = [&](int l) __attribute__((always_inline)) {
    chain::copy_bits(bits0 + size_t(l) * layer_bits + uwave * 1024, bits_at(l));
  };
  if (NH > 1) fetch_bits(NH - 2);
  // ---- head and loss.  The two dot products take a row's features in order
  // in four quarters, (q0 + q1) + (q2 + q3); a quarter's groups of eight
  // features alternate between the lane halves.
  float g0, g1;
  {
    const float4* hw = reinterpret_cast<const float4*>(s_head);
    float s0[4] = {0.f, 0.f, 0.f, 0.f}, s1[4] = {0.f, 0.f, 0.f, 0.f};
    for (int m = 0; m < 4; ++m) {
#pragma unroll
      for (int side = 0; side < 2; ++side) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // K-step 4 q + m; selected by a compile-time chain over m
          u32x4 x = __builtin_bit_cast(u32x4, X[4 * q]);
#pragma unroll
          for (int c = 1; c < 4; ++c)
            if (m == c) x = __builtin_bit_cast(u32x4, X[4 * q + c]);
          const int k4 = (16 * (4 * q + m) + 8 * half) / 4;
          const float4 u0 = hw[k4], u1 = hw[k4 + 1], v0 = hw[64 + k4], v1 = hw[64 + k4 + 1];
          const float wa[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
          const float wb[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
          const uint32_t w4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s0[q] = fmaf(wa[2 * e], bf_lo(w4[e]), s0[q]);
            s1[q] = fmaf(wb[2 * e], bf_lo(w4[e]), s1[q]);
            s0[q] = fmaf(wa[2 * e + 1], bf_hi(w4[e]), s0[q]);
            s1[q] = fmaf(wb[2 * e + 1], bf_hi(w4[e]), s1[q]);
          }
          s0[q] = side == 0 ? from_lo(s0[q]) : from_hi(s0[q]);
          s1[q] = side == 0 ? from_lo(s1[q]) : from_hi(s1[q]);
        }
      }
    }
    const float invB = 1.0f / float(a.B);
    const float y0 = ((s0[0] + s0[1]) + (s0[2] + s0[3])) + a.head_b[0];
    const float y1 = ((s1[0] + s1[1]) + (s1[2] + s1[3])) + a.head_b[1];
    const float mu = s_label[0][32 * wave + (lane & 31)], alpha = s_label[1][32 * wave + (lane & 31)];
    const float e = y0 - mu;
    float v[4];
    v[0] = g0 = 2.0f * alpha * e * invB;
    v[1] = g1 = a.w_hit * (1.0f / (1.0f + expf(-y1)) - alpha) * invB;
    v[2] = alpha * e * e;
    v[3] = fmaxf(y1, 0.f) + log1pf(expf(-fabsf(y1))) - alpha * y1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (half == 0) s_row[q][32 * wave + lane] = v[q];
  }
  // head weight gradients, 64 features at a time: the wave's 32 x 64 values
  // change places in the ring's free slot (16-byte chunk c of row r at c ^ (r
  // % 8)), a lane adds two features over two groups of eight rows, and the
  // groups of a 128-row tile are then added in order
  {
    uint8_t* const place = lds + chain::next_slot(chain::next_slot(cur)) * chain::SLOT + wave * 4096;
    const int fp = lane & 31, r0 = 16 * half;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = lane & 31;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        *reinterpret_cast<u32x4*>(place + r * 128 + 16 * ((2 * m + half) ^ (r & 7))) =
            __builtin_bit_cast(u32x4, X[4 * q + m]);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        float s[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, gr[2][8];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < 8; i += 4) {
            const float4 g4 = *reinterpret_cast<const float4*>(&s_row[j][32 * wave + r0 + 8 * g + i]);
            gr[j][i] = g4.x;
            gr[j][i + 1] = g4.y;
            gr[j][i + 2] = g4.z;
            gr[j][i + 3] = g4.w;
          }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int rr = r0 + 8 * g + i;
          const uint32_t w =
              *reinterpret_cast<const uint32_t*>(place + rr * 128 + 16 * ((fp >> 2) ^ i) + 4 * (fp & 3));
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            s[j][0] = fmaf(gr[j][i], bf_lo(w), s[j][0]);
            s[j][1] = fmaf(gr[j][i], bf_hi(w), s[j][1]);
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
          *reinterpret_cast<float2*>(s_red + (4 * wave + 2 * half + g) * 128 + 64 * j + 2 * fp) =
              make_float2(s[j][0], s[j][1]);
      }
      __syncthreads();
      for (int i = t; i < NW / 4 * 128; i += NT) {
        const int tile = i >> 7, c = i & 127;
        float acc = 0.f;
#pragma unroll
        for (int g = 0; g < 16; ++g) acc += s_red[(16 * tile + g) * 128 + c];
        a.hpart[(size_t(blockIdx.x) * (NW / 4) + tile) * HEAD_PART + 256 * (c >> 6) + 64 * q + (c & 63)] = acc;
      }
      __syncthreads();
    }
  }
  // a tile's bias gradients and loss sums: one wave, lane l adds rows l and
  // l + 64, then a fixed butterfly
  if (wave < NW / 4) {
    const float invB = 1.0f / float(a.B);
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = s_row[q][128 * wave + lane] + s_row[q][128 * wave + lane + 64];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_xor(v[q], off);
    }
    if (lane == 0) {
      float* P = a.hpart + (size_t(blockIdx.x) * (NW / 4) + wave) * HEAD_PART;
      P[512] = v[0];
      P[513] = v[1];
      P[514] = (v[2] + a.w_hit * v[3]) * invB;
      P[515] = v[2] * invB;
      P[516] = v[3] * invB;
    }
  }
  // G = (g_mu W_0 + g_z W_1) * (h > 0); h again from its packed words (kept
  // unpacked from the dot products on, they spilled)
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) asm volatile("" : "+v"(X[ks]));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the first signs have landed
  {
    const float4* hw = reinterpret_cast<const float4*>(s_head);
    uint16_t* dst = G0 + size_t(NH - 1) * layer_elems;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      const u32x4 x = __builtin_bit_cast(u32x4, X[ks]);
      const int k4 = (16 * ks + 8 * half) / 4;
      const float4 u0 = hw[k4], u1 = hw[k4 + 1], z0 = hw[64 + k4], z1 = hw[64 + k4 + 1];
      const float wa[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
      const float wb[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
      const uint32_t w4[4] = {x.x, x.y, x.z, x.w};
      uint32_t o4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v0 = fmaf(g0, wa[2 * e], g1 * wb[2 * e]);
        const float v1 = fmaf(g0, wa[2 * e + 1], g1 * wb[2 * e + 1]);
        // a positive half has its sign bit clear and is not zero (h >= 0)
        o4[e] = chain::pack2(v0, v1) & chain::select_mask(w4[e]);
      }
      const u32x4 g = {o4[0], o4[1], o4[2], o4[3]};
      X[ks] = __builtin_bit_cast(bf16x8_t, g);
      gstore(dst, row_off + kstep_off(ks), g);
    }
  }
  // ---- data gradients: G_{l-1} = (G_l W_l) * (H_{l-1} > 0)
  for (int l = NH - 1; l > 0; --l) {
    uint32_t mb[4];
    chain::read_bits(mb, bits_at(l - 1));
    if (l > 1) fetch_bits(l - 2);
    uint16_t* dst = G0 + size_t(l - 1) * layer_elems;
    auto bwd = [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        ew[2 * (q & 1) + i] = chain::select_bits(chain::pack2(v[4 * q + 2 * i], v[4 * q + 2 * i + 1]), mb[fb / 2],
                                                 fb & 1, 2 * q + i);
      if (q & 1) {
        const u32x4 k = chain::to_operand(ew[0], ew[1], ew[2], ew[3]);
        Y[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, k);
        gstore(dst, row_off + kstep_off(2 * fb + q / 2), k);
      }
    };
    // the first of these layers follows 16 stores of G, the others a layer's six
    chain::layer<16, 8, 16, NW, false, 2, 2, 2>(X, a.wt[l], l > 1 ? a.wt[l - 1] : nullptr, lds, cur, 0u, bwd);
    advance();
  }
}

// Classifier form: the head (K outermost), the residual blocks, the tail with
// its loss (Eq. 6), and the data gradients with the skip path's float32
// gradient, of a workgroup's 32 NW rows (a wave's residual stream, skip
// gradient and two operands take more registers than two waves per SIMD
// leave).
//
// Bound by one wave's own instruction stream up to a round of workgroups (350
// us for 16 blocks from 256 rows on, 415 us at 16,384: about 1,000
// instructions beside the 128 matrix ops of a layer and nobody else on the
// SIMD), beyond it by the writes of the 67 arrays of B x 256 values that the
// weight gradients read.  With it the step takes 685 us at 16,384 rows
// against 1,519 us with a launch per layer and direction (and the float32
// gradient stream in memory).
constexpr int CLS_OUT = 1 + NEDF_CLS_COARSE + NEDF_CLS_FINE;
__device__ __forceinline__ float softplus_f(float z) { return fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))); }

template <int NW>
__global__ __launch_bounds__(64 * NW, 1) void k_chain_points(ChainPointsArgs a) {
  constexpr int K0 = 64;  // K-steps of the encoded input
  constexpr int NI = eng::dma_instr(chain::SLOT, NW);
  __shared__ __attribute__((aligned(16))) uint8_t lds[chain::RING];
  __shared__ __attribute__((aligned(16))) float s_bias[NEDF_TRAIN_MAX_LAYERS * 256];
  __shared__ float s_red[NW][2];
  __shared__ __attribute__((aligned(16))) uint8_t s_bits[2 * NW * 1024];
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5, wave = t >> 6;
  const int NB = a.n_blocks, tail = 2 * NB + 1;
  const uint32_t tile_off = chain::tile_off(lane);
  const uint32_t row_off = wave * 16384u + tile_off;
  const uint32_t bit_off = (uint32_t(wave) * 256u + lane) * 4u;
  const size_t elems = size_t(a.B) * 256, lbits = size_t(a.B) * 32;
  const size_t wg_elems = size_t(blockIdx.x) * (32 * NW * 256), wg_bits = size_t(blockIdx.x) * (32 * NW * 32);
  uint16_t *const H0 = a.H + wg_elems, *const A0 = a.A + wg_elems, *const G0 = a.G + wg_elems;
  // sign arrays: the head's output, then per block its two layers'
  uint8_t* const bits0 = a.bits + wg_bits;
  const uint8_t* X0 = reinterpret_cast<const uint8_t*>(a.X) + (size_t(blockIdx.x) * NW + wave) * (1024u * K0);
  for (int i = t; i < (tail + 1) * 256; i += 64 * NW) s_bias[i] = a.bias[i >> 8][i & 255];
  __syncthreads();
  const uint32_t bias0 = eng::lds_offset(reinterpret_cast<const uint8_t*>(s_bias));
  int cur = 0;
  bf16x8_t X[16], Y[16];
  uint32_t hw[64];  // the residual stream in accumulator order (two features a word)
  f32x16_t gh[8];  // the logits, then the skip path's gradient: float32, accumulator order
  uint32_t ew[4], bits = 0;
  // ---- head: all eight blocks at once, four K-steps per chunk
  {
    constexpr int NHC = K0 / 4;
    f32x16_t acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = f32x16_t{};
    eng::dma_chunk<chain::SLOT, NW>(a.w[0], lds);
    eng::dma_chunk<chain::SLOT, NW>(a.w[0] + chain::SLOT, lds + chain::SLOT);
    u32x4 xn[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) xn[i] = chain::gload(X0, tile_off + kstep_off(i));
    eng::dma_wait_barrier_n<NI>();
#pragma unroll 1
    for (int c = 0; c < NHC; ++c) {
      const int n2 = c + 2;
      uint8_t* nbuf = lds + chain::next_slot(chain::next_slot(cur)) * chain::SLOT;
      eng::dma_chunk<chain::SLOT, NW>(n2 < NHC ? a.w[0] + size_t(n2) * chain::SLOT
                                               : a.w[1] + size_t(n2 - NHC) * chain::SLOT, nbuf);
      bf16x8_t x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = __builtin_bit_cast(bf16x8_t, xn[i]);
      // the next chunk's inputs (the last chunk reads its own again)
      const uint32_t base = 4096u * uint32_t(c + 1 < NHC ? c + 1 : c);
#pragma unroll
      for (int i = 0; i < 4; ++i) xn[i] = chain::gload(X0, base + tile_off + kstep_off(i));
      const uint32_t fbase = eng::lds_offset(lds + cur * chain::SLOT) + uint32_t(lane) * 16u;
      u32x4 w[2][4];
      eng::static_for<4>([&](auto rc) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        w[0][r] = eng::lds_read16<r * 1024>(fbase);
      });
      eng::static_for<8>([&](auto fbc) __attribute__((always_inline)) {
        constexpr int fb = decltype(fbc)::value;
        u32x4(&cw)[4] = w[fb & 1];
        if constexpr (fb + 1 < 8) {
          eng::static_for<4>([&](auto rc) __attribute__((always_inline)) {
            constexpr int r = decltype(rc)::value;
            w[(fb + 1) & 1][r] = eng::lds_read16<((fb + 1) * 4 + r) * 1024>(fbase);
          });
          eng::lds_wait4<4>(cw[0], cw[1], cw[2], cw[3]);
        } else {
          eng::lds_wait4<0>(cw[0], cw[1], cw[2], cw[3]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[fb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, cw[r]), x[r], acc[fb], 0, 0, 0);
      });
      // chunk c + 1 has landed; the copies of c + 2 and this chunk's four
      // input loads, issued since the last barrier, may be in flight
      eng::dma_wait_barrier_n<NI + 4>();
      cur = chain::next_slot(cur);
    }
#pragma unroll
    for (int fb = 0; fb < 8; ++fb) {
      uint32_t w[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = 2 * i;
        const float2 b = *reinterpret_cast<const float2*>(s_bias + 32 * fb + 8 * (r / 4) + 4 * half + r % 4);
        w[i] = chain::pack2(fmaxf(acc[fb][r] + b.x, 0.f), fmaxf(acc[fb][r + 1] + b.y, 0.f));
        const uint32_t m = chain::positive_bits(w[i], fb & 1, i);
        bits = (fb & 1) || i ? bits | m : m;
        hw[8 * fb + i] = w[i];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const u32x4 k = chain::to_operand(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
        X[2 * fb + q] = __builtin_bit_cast(bf16x8_t, k);
        gstore(H0, row_off + kstep_off(2 * fb + q), k);
      }
      if (fb & 1) gstore1(bits0, bit_off + 256 * (fb / 2), bits);
    }
  }
  // ---- residual blocks: a = relu(W1 h + b1), h += relu(W2 a + b2)
  for (int k = 0; k < NB; ++k) {
    const int i1 = 1 + 2 * k, i2 = i1 + 1;
    uint16_t* Ak = A0 + k * elems;
    uint8_t* ba = bits0 + size_t(i1) * lbits;
    chain::layer<16, 8, 16, NW, true, 2, 2, 2>(
        X, a.w[i1], a.w[i2], lds, cur, bias0 + i1 * 1024, [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const uint32_t w = chain::pack2(fmaxf(v[4 * q + 2 * i], 0.f), fmaxf(v[4 * q + 2 * i + 1], 0.f));
            ew[2 * (q & 1) + i] = w;
            const uint32_t m = chain::positive_bits(w, fb & 1, 2 * q + i);
            bits = (fb & 1) || 2 * q + i ? bits | m : m;
          }
          if (q & 1) {
            const u32x4 kk = chain::to_operand(ew[0], ew[1], ew[2], ew[3]);
            Y[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, kk);
            gstore(Ak, row_off + kstep_off(2 * fb + q / 2), kk);
          }
          if ((fb & 1) && q == 3) gstore1(ba, bit_off + 256 * (fb / 2), bits);
        });
    uint16_t* Hn = H0 + (k + 1) * elems;
    uint8_t* br = bits0 + size_t(i2) * lbits;
    chain::layer<16, 8, 16, NW, true, 2, 2, 2>(
        Y, a.w[i2], a.w[i2 + 1], lds, cur, bias0 + i2 * 1024,
        [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float r0 = fmaxf(v[4 * q + 2 * i], 0.f), r1 = fmaxf(v[4 * q + 2 * i + 1], 0.f);
            const uint32_t m = chain::positive_bits(chain::pack2(r0, r1), fb & 1, 2 * q + i);
            bits = (fb & 1) || 2 * q + i ? bits | m : m;
            uint32_t& h = hw[8 * fb + 2 * q + i];
            h = chain::pack2(bf_lo(h) + r0, bf_hi(h) + r1);
            ew[2 * (q & 1) + i] = h;
          }
          if (q & 1) {
            const u32x4 kk = chain::to_operand(ew[0], ew[1], ew[2], ew[3]);
            X[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, kk);
            gstore(Hn, row_off + kstep_off(2 * fb + q / 2), kk);
          }
          if ((fb & 1) && q == 3) gstore1(br, bit_off + 256 * (fb / 2), bits);
        });
  }
  // signs, copied a layer ahead, into two places by turns; the layers take the
  // arrays from the last one down
  uint32_t mb[4];
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  auto bits_at = [&](int i) __attribute__((always_inline)) { return s_bits + ((i & 1) * NW + uwave) * 1024; };
  auto fetch_bits = [&](int i) __attribute__((always_inline)) {
    chain::copy_bits(bits0 + size_t(i) * lbits + uwave * 1024, bits_at(i));
  };
  fetch_bits(2 * NB);
  // ---- tail and loss: target bins from S of mu*; binary cross-entropy with
  // logits, bins averaged per level and counted for hits only
  {
    const size_t row = (size_t(blockIdx.x) * NW + wave) * 32 + (lane & 31);
    const float al = a.alpha[row];
    const float u = (a.mu[row] + 1.0f) * 0.5f;  // S: u = (mu + l) / 2l with mu* = mu / l
    const int c = min(max(int(floorf(float(NEDF_CLS_COARSE) * u)), 0), NEDF_CLS_COARSE - 1);
    const int f = min(max(int(floorf(float(NEDF_CLS_FINE) * (float(NEDF_CLS_COARSE) * u - float(c)))), 0),
                      NEDF_CLS_FINE - 1);
    const float invB = 1.0f / float(a.B);
    float lb = 0.f, lh = 0.f;
    uint16_t* Gt = G0 + size_t(tail) * elems;
    // the logits first: the loss's exponentials and logarithms need more
    // registers than a layer's reads in flight leave
    chain::layer<16, 8, 16, NW, true, 0, 2, 2>(
        X, a.w[tail], a.wt[tail], lds, cur, bias0 + tail * 1024,
        [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < 4; ++i) gh[fb][4 * q + i] = v[4 * q + i];
        });
#pragma unroll
    for (int fb = 0; fb < 8; ++fb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float g[4] = {0.f, 0.f, 0.f, 0.f};
        if (32 * fb + 8 * q < CLS_OUT) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int j = 32 * fb + 8 * q + 4 * half + i;
            const float z = gh[fb][4 * q + i];
            const float sg = 1.0f / (1.0f + expf(-z));
            const float sp = softplus_f(z);
            if (j == 0) {
              lh += sp - al * z;
              g[i] = a.w_hit * (sg - al) * invB;
            } else if (j <= NEDF_CLS_COARSE) {
              const float y = (j - 1 == c) ? 1.f : 0.f;
              lb += al * (sp - y * z) * (1.0f / NEDF_CLS_COARSE);
              g[i] = al * (sg - y) * (invB / NEDF_CLS_COARSE);
            } else if (j < CLS_OUT) {
              const float y = (j - 1 - NEDF_CLS_COARSE == f) ? 1.f : 0.f;
              lb += al * (sp - y * z) * (1.0f / NEDF_CLS_FINE);
              g[i] = al * (sg - y) * (invB / NEDF_CLS_FINE);
            }
          }
        }
        ew[2 * (q & 1)] = chain::pack2(g[0], g[1]);
        ew[2 * (q & 1) + 1] = chain::pack2(g[2], g[3]);
        if (q & 1) {
          const u32x4 kk = chain::to_operand(ew[0], ew[1], ew[2], ew[3]);
          Y[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, kk);
          gstore(Gt, row_off + kstep_off(2 * fb + q / 2), kk);
        }
      }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      lb += __shfl_xor(lb, off);
      lh += __shfl_xor(lh, off);
    }
    if (lane == 0) {
      s_red[wave][0] = lb;
      s_red[wave][1] = lh;
    }
  }
  __syncthreads();
  if (t == 0) {
    float lb = 0.f, lh = 0.f;
#pragma unroll
    for (int w = 0; w < NW; w += 2) {
      lb += s_red[w][0] + s_red[w + 1][0];
      lh += s_red[w][1] + s_red[w + 1][1];
    }
    float* P = a.lpart + size_t(blockIdx.x) * 3;
    P[0] = lb + a.w_hit * lh;
    P[1] = lb;
    P[2] = lh;
  }
  // ---- data gradients
  // a masked quarter of a block into `out` and the gradient array `dst`
  auto masked = [&](bf16x8_t(&out)[16], uint16_t* dst, int fb, int q, const float (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      ew[2 * (q & 1) + i] = chain::select_bits(chain::pack2(v[2 * i], v[2 * i + 1]), mb[fb / 2], fb & 1, 2 * q + i);
    if (q & 1) {
      const u32x4 kk = chain::to_operand(ew[0], ew[1], ew[2], ew[3]);
      out[2 * fb + q / 2] = __builtin_bit_cast(bf16x8_t, kk);
      gstore(dst, row_off + kstep_off(2 * fb + q / 2), kk);
    }
  };
  {
    chain::read_bits(mb, bits_at(2 * NB));
    fetch_bits(2 * NB - 1);
    uint16_t* dst = G0 + size_t(2 * NB) * elems;
    chain::layer<16, 8, 16, NW, false, 2, 2, 2>(
        Y, a.wt[tail], a.wt[2 * NB], lds, cur, 0u, [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
          float o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = gh[fb][4 * q + i] = v[4 * q + i];
          masked(X, dst, fb, q, o);
        });
  }
  for (int k = NB - 1; k >= 0; --k) {
    const int i1 = 1 + 2 * k, i2 = i1 + 1;
    chain::read_bits(mb, bits_at(i1));
    fetch_bits(i1 - 1);
    uint16_t* d1 = G0 + size_t(i1) * elems;
    chain::layer<16, 8, 16, NW, false, 2, 2, 2>(
        X, a.wt[i2], a.wt[i1], lds, cur, 0u, [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
          const float o[4] = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
          masked(Y, d1, fb, q, o);
        });
    // masked by the second layer of the block before, or by the head's output
    chain::read_bits(mb, bits_at(i1 - 1));
    if (k > 0) fetch_bits(i1 - 2);
    uint16_t* d0 = G0 + size_t(i1 - 1) * elems;
    chain::layer<16, 8, 16, NW, false, 2, 2, 2>(
        Y, a.wt[i1], k > 0 ? a.wt[i1 - 1] : nullptr, lds, cur, 0u,
        [&](int fb, int q, const f32x16_t& v) __attribute__((always_inline)) {
          float o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = gh[fb][4 * q + i] = v[4 * q + i] + gh[fb][4 * q + i];
          masked(X, d0, fb, q, o);
        });
  }
}

template <int N, int NW>
void launch_line(const ChainLineArgs& a, int k0, hipStream_t s) {
  const dim3 g(a.B / (32 * NW)), b(64 * NW);
  // xyz inputs of up to 12 levels have at most 75 features: always 8 K-steps
  if (N == 3 || k0 == 8) hipLaunchKernelGGL((k_chain_line<N, 8, NW>), g, b, 0, s, a);
  else if constexpr (N == 6) hipLaunchKernelGGL((k_chain_line<N, 16, NW>), g, b, 0, s, a);
}

}  // namespace

int chain_line_waves(int B, int cus) {
  const int r8 = (B / 256 + cus - 1) / cus, r4 = (B / 128 + cus - 1) / cus;
  return 9 * r8 <= 5 * r4 ? 8 : 4;
}

int chain_points_waves(int B, int cus) {
  const int r2 = (B / 64 + cus - 1) / cus, r4 = (B / 128 + cus - 1) / cus;
  return r2 <= r4 ? 2 : 4;
}

void launch_chain_line(const ChainLineArgs& a, int n_comp, int k0, int waves, hipStream_t s) {
  if (n_comp == 6) {
    if (waves == 8) launch_line<6, 8>(a, k0, s);
    else launch_line<6, 4>(a, k0, s);
  } else {
    if (waves == 8) launch_line<3, 8>(a, k0, s);
    else launch_line<3, 4>(a, k0, s);
  }
}

void launch_chain_points(const ChainPointsArgs& a, int waves, hipStream_t s) {
  if (waves == 2) hipLaunchKernelGGL((k_chain_points<2>), dim3(a.B / 64), dim3(128), 0, s, a);
  else hipLaunchKernelGGL((k_chain_points<4>), dim3(a.B / 128), dim3(256), 0, s, a);
}

}  // namespace nedf
