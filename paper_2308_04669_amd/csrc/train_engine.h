// Layer chain of the training kernels: a wave carries 32 batch rows through
// every layer of a 256-wide network in registers, as mlp_engine.h does for
// inference, and streams each layer's inputs for the weight gradients out to
// memory on the way.  Weights come packed as matrix-core fragments
// (train_layout.h) through a three-slot LDS ring of superchunks of two
// 32-feature output blocks.
//
// Operands are kept in natural feature order: lane half h of K-step ks holds
// features 16 ks + 8 h .. + 7.  An accumulator block holds, in lane half h,
// features 8 (r / 4) + 4 h + r % 4; two half-wave swaps per K-step turn the
// rounded block into the next layer's operand, which is then also a row's 16
// contiguous bytes.  The products are summed over K in order from zero, the
// bias added after: the same sums as a tile GEMM over the same K-steps gives.
#pragma once
#include "mlp_engine.h"
#include "train_layout.h"

namespace chain {

using eng::u32x4;
constexpr int KS = 16;                   // K-steps of a 256-wide layer
constexpr int SB = 2;                    // output blocks per superchunk
constexpr int SLOT = SB * KS * 1024;     // bytes of a ring slot
constexpr int RING = eng::NBUF * SLOT;

// Global memory at a wave-uniform base plus a lane's 32-bit byte offset (one
// address register per lane for every array of one row stride).
typedef __attribute__((address_space(1))) u32x4 gvec;
typedef __attribute__((address_space(1))) uint32_t gword;
typedef __attribute__((address_space(1))) char gbyte;
__device__ __forceinline__ void gstore(void* base, uint32_t off, u32x4 v) { *(gvec*)((gbyte*)base + off) = v; }
__device__ __forceinline__ void gstore1(void* base, uint32_t off, uint32_t v) { *(gword*)((gbyte*)base + off) = v; }
__device__ __forceinline__ u32x4 gload(const void* base, uint32_t off) { return *(gvec*)((gbyte*)base + off); }

// The arrays kept for the weight gradients are stored in tiles of 32 rows x
// 32 features, [row block][feature block][row][feature]: a K-step's store
// covers 32-byte pieces of a 2 KB tile (row-major 512-byte rows made it 32
// pieces 512 bytes apart: the address units were busy two thirds of the
// kernel, which took 189 us instead of 158 at 65,536 rows), and the weight
// gradients' loads take whole 256-byte runs of a tile (nedf_train_tile_row).
// Byte offsets: a lane's place in a tile, and K-step ks from its row block's
// start.
__device__ __forceinline__ uint32_t tile_off(int lane) {
  return uint32_t(nedf_train_tile_row(lane & 31)) * 64u + 16u * (lane >> 5);
}
__device__ __forceinline__ constexpr uint32_t kstep_off(int ks) { return uint32_t(ks >> 1) * 2048u + 32u * (ks & 1); }

__device__ __forceinline__ int next_slot(int s) { return s + 1 >= eng::NBUF ? s + 1 - eng::NBUF : s + 1; }

// The first two superchunks of a layer of K0 K-steps into slots `cur` and the
// next (a chain's start); the first has landed on return.
template <int K0, int NW>
__device__ __forceinline__ void prime(const uint8_t* w, uint8_t* lds, int cur) {
  constexpr int SCB = SB * K0 * 1024;
  eng::dma_chunk<SCB, NW>(w, lds + cur * SLOT);
  eng::dma_chunk<SCB, NW>(w + SCB, lds + next_slot(cur) * SLOT);
  eng::dma_wait_barrier_n<eng::dma_instr(SCB, NW)>();
}

// One layer of FB output blocks and K0 K-steps.  A block's sums (plus the
// bias with BIAS: float32 [256] at LDS byte address bias_addr) go to epi one
// block late, a quarter at a time, so that its vector work lies under the next
// block's matrix ops: epi(block, quarter, acc) may use registers 4 quarter ..
// 4 quarter + 3 of acc.  w_next: the following layer's weights (KN K-steps),
// or null at a chain's end.  On entry superchunk 0 is in slot `cur` and
// superchunk 1 on its way.
//
// epi stores ST times (0 or 2: after quarters 1 and 3) to global memory per
// block; the previous layer's PST times, SP stores of it lying after its last
// barrier.  The wait at the end of superchunk sc is for the copies of
// superchunk sc + 1.  Vector-memory operations retire in order, and a store
// takes about as long as a superchunk, so the wait leaves in flight all that
// was certainly issued after those copies (at the start of superchunk sc - 1,
// with the compiler kept from moving memory operations past them): the copies
// of superchunk sc + 2 and the stores of two superchunks.  A superchunk's
// last read group is consumed after its barrier, so that before the barrier
// lie PRE of its ST SB stores, both of the block before it and, with four
// read groups or more to a block, the first one of its own first block.
template <int K0, int FB, int KN, int NW, bool BIAS, int ST, int PST, int SP, class EPI>
__device__ __forceinline__ void layer(const bf16x8_t (&Bin)[K0], const uint8_t* w, const uint8_t* w_next, uint8_t* lds,
                                      int& cur, uint32_t bias_addr, EPI&& epi) {
  constexpr int NSC = FB / SB;
  static_assert(ST == 0 || ST == 2, "stores after quarters 1 and 3");
  static_assert(FB % SB == 0 && NSC >= 2 && K0 % 8 == 0 && KN % 8 == 0 && SB == 2, "layer shape");
  constexpr int SCB = SB * K0 * 1024, SCN = SB * KN * 1024;
  static_assert(SCB <= SLOT && SCN <= SLOT && SCB < 65536, "superchunk fits a slot");
  constexpr int G = 4, NG = K0 / G;
  // read groups of a block: its first fragments, the bias of the block
  // before, its other fragments
  constexpr int PER = NG + (BIAS ? 1 : 0);
  constexpr int E = SB * PER;  // read groups (4 reads each) per superchunk
  constexpr int D = 3;         // groups in flight
  const int lane = threadIdx.x & 63, half = lane >> 5;
  u32x4 ring[D][G];
  auto read_bias = [&](u32x4(&dst)[G], int fb) __attribute__((always_inline)) {
    const uint32_t b = bias_addr + uint32_t(fb * 128 + 16 * half);
    eng::static_for<4>([&](auto rc) __attribute__((always_inline)) {
      constexpr int r = decltype(rc)::value;
      dst[r] = eng::lds_read16<32 * r>(b);
    });
  };
  auto issue = [&](auto ec, uint32_t base, int sc) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value;
    if constexpr (e < E) {
      constexpr int k = e / PER, g = e % PER;
      u32x4(&dst)[G] = ring[e % D];
      if constexpr (BIAS && g == 1) {
        const int fb = sc * SB + k;
        read_bias(dst, fb > 0 ? fb - 1 : 0);
      } else {
        constexpr int f = g == 0 ? 0 : g - (BIAS ? 1 : 0);
        const uint32_t at = base + uint32_t(lane) * 16u;
        eng::static_for<4>([&](auto rc) __attribute__((always_inline)) {
          constexpr int r = decltype(rc)::value;
          dst[r] = eng::lds_read16<k * K0 * 1024 + (f * G + r) * 1024>(at);
        });
      }
    }
  };
  // the accumulators of consecutive blocks alternate; a block's stay in place
  // while the next one is multiplied
  f32x16_t acc2[2];
  auto add_bias = [&](f32x16_t& p, const u32x4(&cw)[G]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      p[4 * q + 0] += __uint_as_float(cw[q].x);
      p[4 * q + 1] += __uint_as_float(cw[q].y);
      p[4 * q + 2] += __uint_as_float(cw[q].z);
      p[4 * q + 3] += __uint_as_float(cw[q].w);
    }
  };
  auto consume = [&](auto ec, int sc, const u32x4(&cw)[G]) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value;
    constexpr int k = e / PER, g = e % PER;
    const int fb = sc * SB + k;
    f32x16_t &acc = acc2[k & 1], &prev = acc2[(k + 1) & 1];
    if constexpr (BIAS && g == 1) {
      if (fb > 0) add_bias(prev, cw);
    } else {
      constexpr int f = g == 0 ? 0 : g - (BIAS ? 1 : 0);
      if constexpr (f == 0) acc = f32x16_t{};
#pragma unroll
      for (int r = 0; r < G; ++r)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, cw[r]), Bin[f * G + r], acc, 0, 0, 0);
      // the quarters of the block before, spread over this block's groups
      // (from the second one on with BIAS, which the first one covers)
      if (fb > 0) {
        if constexpr (BIAS) {
          if constexpr (f > 0) {
#pragma unroll
            for (int q = (f - 1) * 4 / (NG - 1); q < f * 4 / (NG - 1); ++q) epi(fb - 1, q, prev);
          }
        } else {
#pragma unroll
          for (int q = f * 4 / NG; q < (f + 1) * 4 / NG; ++q) epi(fb - 1, q, prev);
        }
      }
      eng::static_for<G>([&](auto) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one matrix op
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);  // up to eight VALU ops
      });
    }
  };
  {
    const uint32_t base0 = eng::lds_offset(lds + cur * SLOT);
    eng::static_for<D>([&](auto ec) __attribute__((always_inline)) { issue(ec, base0, 0); });
  }
  eng::static_for<NSC>([&](auto scc) __attribute__((always_inline)) {
    constexpr int sc = decltype(scc)::value;
    uint8_t* nbuf = lds + next_slot(next_slot(cur)) * SLOT;
    constexpr bool own = sc + 2 < NSC;
    constexpr int NI = own ? eng::dma_instr(SCB, NW) : eng::dma_instr(SCN, NW);
    constexpr int OWN = NG >= 4 ? ST / 2 : 0, PRE = ST + OWN;
    constexpr int young = sc == 0 ? SB * PST + SP + OWN : sc == 1 ? OWN + (SB * ST - PRE) + PRE : SB * ST + PRE;
    bool issued = own;
    if constexpr (own) {
      eng::dma_chunk<SCB, NW>(w + size_t(sc + 2) * SCB, nbuf);
    } else if (w_next != nullptr) {
      eng::dma_chunk<SCN, NW>(w_next + size_t(sc + 2 - NSC) * SCN, nbuf);
      issued = true;
    }
    asm volatile("" ::: "memory");
    auto pass_barrier = [&]() __attribute__((always_inline)) {
      if (issued) eng::dma_wait_barrier_n<NI + young>();
      else eng::dma_wait_barrier();
    };
    const uint32_t base = eng::lds_offset(lds + cur * SLOT);
    eng::static_for<E>([&](auto ec) __attribute__((always_inline)) {
      constexpr int e = decltype(ec)::value;
      u32x4(&cw)[G] = ring[e % D];
      constexpr int after = (e + 1 < E ? 4 : 0) + (e + 2 < E ? 4 : 0);
      eng::lds_wait4<after>(cw[0], cw[1], cw[2], cw[3]);
      if constexpr (e + 1 < E) {
        consume(ec, sc, cw);
        issue(std::integral_constant<int, e + D>{}, base, sc);
      } else if constexpr (sc + 1 < NSC) {
        // every read of this superchunk has completed: pass the barrier, start
        // the next superchunk's reads, then this group's work covers them
        u32x4 tail[G] = {cw[0], cw[1], cw[2], cw[3]};
        pass_barrier();
        const uint32_t nbase = eng::lds_offset(lds + next_slot(cur) * SLOT);
        eng::static_for<D>([&](auto gc) __attribute__((always_inline)) { issue(gc, nbase, sc + 1); });
        asm volatile("" : "+v"(tail[0]), "+v"(tail[1]), "+v"(tail[2]), "+v"(tail[3]));
        consume(ec, sc, tail);
      } else {
        consume(ec, sc, cw);
      }
    });
    // the layer's end: the next layer's first superchunk must have landed
    if constexpr (sc + 1 == NSC) pass_barrier();
    cur = next_slot(cur);
  });
  if constexpr (BIAS) {
    u32x4(&cw)[G] = ring[0];
    read_bias(cw, FB - 1);
    eng::lds_wait4<0>(cw[0], cw[1], cw[2], cw[3]);
    add_bias(acc2[(FB - 1) & 1], cw);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) epi(FB - 1, q, acc2[(FB - 1) & 1]);
}

typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_t;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  const f32x2_t f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

// A wave's sign words of a layer, [block pair][lane], copied to its 1 KB of
// LDS a layer ahead and read there.  (As loads to registers they made the
// compiler drain every store and copy in flight, once per layer.)  The copy
// has landed once the wave has passed the barriers of a layer begun after it.
__device__ __forceinline__ void copy_bits(const uint8_t* src, uint8_t* dst) {
  const eng::gbyte* base = (const eng::gbyte*)src;
  uint32_t off = (threadIdx.x & 63) * 16u;
  asm volatile("" : "+s"(base), "+v"(off));
  __builtin_amdgcn_global_load_lds((const void*)(base + off), dst, 16, 0, 0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void read_bits(uint32_t (&m)[4], const uint8_t* src) {
  const uint32_t at = eng::lds_offset(src) + (threadIdx.x & 63) * 4u;
  asm volatile(
      "ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:256\n\tds_read_b32 %2, %4 offset:512\n\t"
      "ds_read_b32 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(m[0]), "=&v"(m[1]), "=&v"(m[2]), "=&v"(m[3])
      : "v"(at)
      : "memory");
}

// Half of a block's packed words (accumulator order, two features each) as
// one K-step of the next layer's operand.
__device__ __forceinline__ u32x4 to_operand(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
  auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
  auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
  return u32x4{a[0], b[0], a[1], b[1]};
}

// Which of a packed (non-negative) word's values are positive, as bits: two
// blocks share a word of bits per lane, word i of a block has its two at
// 15 - i and 31 - i (8 further down for the odd block).
__device__ __forceinline__ uint32_t positive_bits(uint32_t w, int odd, int i) {
  return ((w + 0x7FFF7FFFu) & 0x80008000u) >> (i + (odd ? 8 : 0));
}
__device__ __forceinline__ uint32_t select_bits(uint32_t w, uint32_t m, int odd, int i) {
  typedef __attribute__((__vector_size__(2 * sizeof(short)))) short s16x2_t;
  const s16x2_t t = __builtin_bit_cast(s16x2_t, m << (i + (odd ? 8 : 0)));
  const s16x2_t fifteen = {15, 15};
  return w & __builtin_bit_cast(uint32_t, t >> fifteen);
}

// Of a packed (non-negative) word's values: all ones where positive.
__device__ __forceinline__ uint32_t select_mask(uint32_t w) {
  return select_bits(0xFFFFFFFFu, positive_bits(w, 0, 0), 0, 0);
}

}  // namespace chain
