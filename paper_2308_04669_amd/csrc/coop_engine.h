// Feature-split evaluation of a 256-wide network: the workgroup's eight waves
// share 32 NB samples and each computes one 32-feature block of every layer
// (the register-resident engine of mlp_engine.h instead gives every wave 32
// samples of its own and all eight blocks).  Per pass a compute unit then does
// an eighth of the matrix work, so a call with few samples ends in a fraction
// of the time.  A wave's weights are used by no other wave: they go from L2
// straight into registers, one ring of 16 loads ahead of the matrix ops; the
// activations go through LDS once per layer, already in operand order (an
// accumulator block is two (BF16) or four (FP32) 1 KB operand reads of the
// next layer).  Every output is summed over K in the same order, and the head
// over features in the same order, as in the register-resident engine: the
// two give the same bits.
#pragma once
#include "mlp_engine.h"

namespace coop {

using eng::u32x4;
constexpr int NW = 8;
constexpr int THREADS = 64 * NW;

// LDS: two activation buffers of the widest layer input (the second one also
// takes the last layer's float32 activations with the first), the head rows,
// and one result per sample and head row.
template <int DT, int NB, int NOUT>
struct Lds {
  static constexpr int R = 256 / eng::Tr<DT>::KPS * eng::Tr<DT>::FRAG / 1024;  // 1 KB reads per layer
  static constexpr int ACT = R * 1024;                                          // one sample block's activations
  static constexpr int LAST = 8 * 4 * 1024;                                     // one block's float32 activations
  static constexpr int BUF = NB * (2 * ACT > LAST ? 2 * ACT : LAST);
  static constexpr int HEAD = NOUT * 8 * 128;
  static constexpr int BYTES = BUF + HEAD + NOUT * NB * 32 * 4;
};

// Every wave's LDS accesses done, then the barrier (outstanding global loads,
// the weights ahead, stay in flight).
__device__ __forceinline__ void barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef __attribute__((address_space(1))) const u32x4 gvec;
__device__ __forceinline__ u32x4 gload(const uint8_t* p) { return *(gvec*)p; }

// Evaluates the network at `blob` for 32 NB samples.  enc(nb, read) returns
// this lane's 16 bytes of operand read `read` of sample block nb's encoded
// input (called by wave read % 8).  Sample (nb, lane % 32)'s head value o,
// without the head bias, comes back in out[nb][o] on every wave.  `lds` is
// free when the workgroup enters and may be reused after the next barrier.
template <int DT, int KS0, int NHID, int NOUT, int NB, class ENC>
__device__ __forceinline__ void network(const nedf_blob_header* hb, const uint8_t* blob, uint8_t* lds, ENC&& enc,
                                        float (&out)[NB][NOUT]) {
  using T = eng::Tr<DT>;
  using L = Lds<DT, NB, NOUT>;
  constexpr int R = L::R;
  constexpr int R0 = KS0 * T::FRAG / 1024;
  static_assert(KS0 * T::FRAG % 1024 == 0 && R >= 16 && R % 16 == 0, "whole reads, whole rings");
  constexpr int PD = 16;  // loads ahead
  constexpr int CB0 = eng::chunk_bytes<DT>(KS0, 0), CBH = R * 1024 + 128, CBL = R * 1024 + 128 * (1 + NOUT);
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* s_out = reinterpret_cast<float*>(lds + L::BUF + L::HEAD);
  // this wave's chunk (output block `wave`) of layer l, at this lane's bytes
  auto chunk = [&](int l) __attribute__((always_inline)) {
    const int cb = l == 0 ? CB0 : l == NHID - 1 ? CBL : CBH;
    return blob + uniform_load_u64(&hb->off_layer[l]) + size_t(wave) * cb;
  };
  const uint8_t* w0 = chunk(0);
  u32x4 first[R0], ring[PD];
  f32x16_t bias;
  auto load_bias = [&](const uint8_t* p) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4 v = gload(p + 64 * half + 16 * i);
      bias[4 * i + 0] = __uint_as_float(v.x); bias[4 * i + 1] = __uint_as_float(v.y);
      bias[4 * i + 2] = __uint_as_float(v.z); bias[4 * i + 3] = __uint_as_float(v.w);
    }
  };
#pragma unroll
  for (int r = 0; r < R0; ++r) first[r] = gload(w0 + r * 1024 + lane * 16);
  load_bias(w0 + R0 * 1024);
  const uint8_t* wl = chunk(1);
#pragma unroll
  for (int r = 0; r < PD; ++r) ring[r] = gload(wl + r * 1024 + lane * 16);
  // encoded input into buffer 0, read r by wave r % 8
  eng::static_for<R0>([&](auto rc) __attribute__((always_inline)) {
    constexpr int r = decltype(rc)::value;
    if (wave == r % NW) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        *reinterpret_cast<u32x4*>(lds + nb * L::ACT + r * 1024 + lane * 16) = enc(nb, rc);
    }
  });
  barrier();
  f32x16_t acc[NB];
  auto mma_read = [&](const u32x4& a, const uint8_t* act, int r) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const u32x4 b = *reinterpret_cast<const u32x4*>(act + nb * L::ACT + r * 1024 + lane * 16);
#pragma unroll
      for (int i = 0; i < T::KPR; ++i) acc[nb] = T::mma(T::pick(a, i), T::pick(b, i), acc[nb]);
    }
  };
  // ReLU of the wave's block in operand order
  auto store_hidden = [&](uint8_t* act) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      constexpr int RB = R / 8;  // reads per block
      typename T::frag v[1][256 / T::KPS / 8];
      const f32x16_t one[1] = {acc[nb]};
      eng::epi_hidden<DT, 1, 256 / T::KPS / 8>(0, one, v, make_float2(1.f, 1.f));
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        u32x4 q;
        if constexpr (DT == 1) q = __builtin_bit_cast(u32x4, v[0][r]);
        else q = u32x4{__float_as_uint(v[0][4 * r]), __float_as_uint(v[0][4 * r + 1]), __float_as_uint(v[0][4 * r + 2]),
                       __float_as_uint(v[0][4 * r + 3])};
        *reinterpret_cast<u32x4*>(act + nb * L::ACT + (wave * RB + r) * 1024 + lane * 16) = q;
      }
    }
  };
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = bias;
#pragma unroll
  for (int r = 0; r < R0; ++r) mma_read(first[r], lds, r);
  load_bias(wl + R * 1024);
  store_hidden(lds + NB * L::ACT);
  barrier();
  for (int l = 1; l < NHID; ++l) {
    // the last layer's look-ahead reads its own weights again
    const uint8_t* wn = chunk(l + 1 < NHID ? l + 1 : l);
    const uint8_t* act = lds + (l & 1) * (NB * L::ACT);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = bias;
    load_bias(wn + R * 1024);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      mma_read(ring[r % PD], act, r);
      ring[r % PD] = gload((r + PD < R ? wl + (r + PD) * 1024 : wn + (r + PD - R) * 1024) + lane * 16);
    }
    if (l + 1 < NHID) {
      store_hidden(lds + ((l + 1) & 1) * (NB * L::ACT));
      barrier();
    } else {
      barrier();  // every wave has read its input: the activations' buffers take the float32 outputs
    }
    wl = wn;
  }
  // head: the last activations (float32) and this block's head rows to LDS,
  // then wave nb sums sample block nb over the features in order
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<float4*>(lds + nb * L::LAST + (wave * 4 + i) * 1024 + lane * 16) =
          make_float4(fmaxf(acc[nb][4 * i], 0.0f), fmaxf(acc[nb][4 * i + 1], 0.0f), fmaxf(acc[nb][4 * i + 2], 0.0f),
                      fmaxf(acc[nb][4 * i + 3], 0.0f));
  if (lane < 8 * NOUT) {
    const int o = lane >> 3, q = lane & 7;
    *reinterpret_cast<u32x4*>(lds + L::BUF + (o * 8 + wave) * 128 + q * 16) = gload(wl + R * 1024 + 128 * (1 + o) + q * 16);
  }
  barrier();
  if (wave < NB) {
    float s[NOUT];
#pragma unroll
    for (int o = 0; o < NOUT; ++o) s[o] = 0.f;
#pragma unroll 2
    for (int fb = 0; fb < 8; ++fb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(lds + wave * L::LAST + (fb * 4 + i) * 1024 + lane * 16);
#pragma unroll
        for (int o = 0; o < NOUT; ++o) {
          const float4 w = *reinterpret_cast<const float4*>(lds + L::BUF + (o * 8 + fb) * 128 + half * 64 + i * 16);
          s[o] = fmaf(w.x, v.x, s[o]);
          s[o] = fmaf(w.y, v.y, s[o]);
          s[o] = fmaf(w.z, v.z, s[o]);
          s[o] = fmaf(w.w, v.w, s[o]);
        }
      }
#pragma unroll
    for (int o = 0; o < NOUT; ++o) {
      s[o] += __shfl_xor(s[o], 32);
      if (lane < 32) s_out[(wave * NOUT + o) * 32 + lane] = s[o];
    }
  }
  barrier();
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int o = 0; o < NOUT; ++o) out[nb][o] = s_out[(nb * NOUT + o) * 32 + (lane & 31)];
}

// Operand read r of the encoded input for one sample (see eng::encode_input).
template <int DT, int N, int LV, class RC>
__device__ __forceinline__ u32x4 encode_read(const float (&p)[N], const float (&plo)[N], int half, RC) {
  constexpr int r = RC::value;
  if constexpr (DT == 1) {
    bf16x8_t v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = static_cast<__bf16>(eng::enc_slot<N, LV>(p, plo, 8 * r + j, half));
    return __builtin_bit_cast(u32x4, v);
  } else {
    u32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = __float_as_uint(eng::enc_slot<N, LV>(p, plo, 4 * r + j, half));
    return v;
  }
}

}  // namespace coop
