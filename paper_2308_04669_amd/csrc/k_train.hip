// Training of an intersection network (Eq. 6, training details of the paper:
// Adam, lr 5e-4): the split-K weight gradients of the arrays that the training
// chain (k_chain.hip) leaves, their reduction and Adam on float32 master
// weights; the classifier form's input encoding; and the calibration pass of
// FP8 networks.
#include <algorithm>
#include <cstring>

#include "device_common.h"
#include "mlp_engine.h"
#include "runtime.h"
#include "train_kernels.h"
#include "train_layout.h"

namespace nedf {
namespace {

__device__ __forceinline__ uint16_t bf16_bits(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}
__device__ __forceinline__ float bf16_val(uint16_t u) { return __uint_as_float(uint32_t(u) << 16); }

// ---- input encoding of the calibration pass --------------------------------------
// Features in natural order [p, sin(2^0 pi p), cos(2^0 pi p), ...] of the
// Pluecker (d, o x d) or xyz input, zero padded to Kpad.  One thread per sample
// and group of 8 features (one 16-byte store; a sample's row is written by
// consecutive threads).
// N: input components (6 Pluecker, 3 xyz), a constant so that the feature
// index arithmetic divides by constants.
template <int N>
__global__ void k_encode_rows(const float* o_l, const float* d_l, int B, int L, int Kpad, uint16_t* H) {
  const int groups = Kpad / 8;
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int s = tid / groups, grp = tid % groups;
  if (s >= B) return;
  const float o[3] = {o_l[3 * s], o_l[3 * s + 1], o_l[3 * s + 2]};
  const float d[3] = {d_l[3 * s], d_l[3 * s + 1], d_l[3 * s + 2]};
  float p[6], plo[6] = {0, 0, 0, 0, 0, 0}, tperp = 0.0f;
  constexpr int n = N;
  if constexpr (N == 6) {
    line_of_local(o, d, p, plo, tperp);
  } else {
    p[0] = o[0]; p[1] = o[1]; p[2] = o[2];
    p[3] = p[4] = p[5] = 0.0f;
  }
  uint32_t packed[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    float v2[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int f = 8 * grp + e + u;
      float v = 0.0f;
      if (f < n) {
        v = p[f];
      } else if (f < n * (1 + 2 * L)) {
        const int q = f - n, level = q / (2 * n), w = q % (2 * n), c = w % n;
        v = sinpi_hw(float(1 << level) * p[c], float(1 << level) * plo[c], w >= n ? 1 : 0);
      }
      v2[u] = v;
    }
    packed[e / 2] = uint32_t(bf16_bits(v2[0])) | (uint32_t(bf16_bits(v2[1])) << 16);
  }
  *reinterpret_cast<uint4*>(H + size_t(s) * Kpad + 8 * grp) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
}

// amax of |x| over n bfloat16 values (non-negative float bits order as
// unsigned integers).
__global__ void k_amax16(const uint16_t* x, size_t n, uint32_t* out) {
  float m = 0.f;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    m = fmaxf(m, fabsf(bf16_val(x[i])));
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) atomicMax(out, __float_as_uint(m));
}

__global__ void k_amax32(const float* x, size_t n, uint32_t* out) {
  float m = 0.f;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    m = fmaxf(m, fabsf(x[i]));
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) atomicMax(out, __float_as_uint(m));
}

// Scales {w_scale, a_scale} = amax / 448 per hidden layer (E4M3 largest finite).
__global__ void k_fp8_scales(const uint32_t* amax_w, const uint32_t* amax_a, int n_hidden, float* scales) {
  const int i = threadIdx.x;
  if (i >= n_hidden) return;
  const float w = __uint_as_float(amax_w[i]), a = __uint_as_float(amax_a[i]);
  scales[2 * i] = w > 0.f ? w / 448.0f : 1.0f;
  scales[2 * i + 1] = a > 0.f ? a / 448.0f : 1.0f;
}

// ---- GEMM of the calibration pass --------------------------------------------
// out16[M][N] = relu(sum_k A(m, k) B(n, k) + bias[n]) on 32x32x16 bf16 matrix
// cores with float32 accumulation, operands k-contiguous.  A workgroup
// computes a 128 x 256 tile with one wave per 64 x 64 block (2 x 2 blocks of
// 32 x 32); K runs in stages of 64, staged in LDS as [row][k] (rows padded to
// 72 elements, so that the 16-byte fragment reads of a wave's 16-lane groups
// fall on distinct banks) and double-buffered.  Global loads run two stages
// ahead of the matrix cores (two register sets), so a stage's loads have two
// stages of multiplies to arrive in.  The tile goes through LDS after the
// last stage and leaves as whole 16-byte row pieces.  M is a multiple of 128,
// N of 256 and K of 128.
constexpr int GT_BM = 128, GT_BN = 256, GT_BK = 64, GT_LD = 72;  // tile, K stage, LDS row stride (bf16)

struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  int M, N, K, lda, ldb;
  const float* bias;
  uint16_t* out16;  // [M][ldo]
  int ldo;
};

// Staging registers are plain 4 x 32-bit vectors (not the HIP vector
// classes, which the compiler keeps in memory here).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Register staging of one operand's stage (ROWS rows x 64 k) by NT threads.
template <int ROWS, int NT>
struct Stage {
  static constexpr int PER = ROWS * 8 / NT;  // 16-byte chunks per thread
  u32x4 v[PER];
  // chunk c = t + NT i: row c / 8, k 8 (c % 8)
  __device__ __forceinline__ void load(const uint16_t* X, int ld, int row0, int k0, int t) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = t + NT * i;
      v[i] = *reinterpret_cast<const u32x4*>(X + size_t(row0 + (c >> 3)) * ld + k0 + 8 * (c & 7));
    }
  }
  __device__ __forceinline__ void store(uint16_t* S, int t) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = t + NT * i;
      *reinterpret_cast<u32x4*>(S + (c >> 3) * GT_LD + 8 * (c & 7)) = v[i];
    }
  }
};

__global__ __launch_bounds__(512) void k_gemm(GemmArgs g) {
  constexpr int BM = GT_BM, BN = GT_BN;
  constexpr int NT = BN * 2;   // threads: 2 x (BN / 64) waves
  constexpr int WN = BN / 64;  // waves along N
  constexpr int SA = BM * GT_LD, SB = BN * GT_LD;
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * (SA + SB)];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int n_stages = g.K / GT_BK;
  // two register sets, named (not indexed) so that they stay in registers
  Stage<BM, NT> ra0, ra1;
  Stage<BN, NT> rb0, rb1;
  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16_t{};
  ra0.load(g.A, g.lda, m0, 0, t);
  rb0.load(g.B, g.ldb, n0, 0, t);
  ra1.load(g.A, g.lda, m0, GT_BK, t);
  rb1.load(g.B, g.ldb, n0, GT_BK, t);
  ra0.store(lds, t);
  rb0.store(lds + SA, t);
  __syncthreads();
  // one stage: multiply LDS buffer BUF; register set CUR (stage s, then
  // free) takes stage s + 2; set NXT (stage s + 1) goes to buffer BUF ^ 1.
  // Written out for each parity (a macro, not a function), so that both
  // register sets stay named registers.
#define NEDF_GEMM_STAGE(S_, BUF, RA_CUR, RB_CUR, RA_NXT, RB_NXT)                                           \
  {                                                                                                       \
    {                                                                                                     \
      /* unconditional (the last stage again past the end): a conditional */                            \
      /* load would keep the register set in memory */                                                    \
      const int kl = min((S_) + 2, n_stages - 1) * GT_BK;                                                 \
      RA_CUR.load(g.A, g.lda, m0, kl, t);                                                                 \
      RB_CUR.load(g.B, g.ldb, n0, kl, t);                                                                 \
    }                                                                                                     \
    const uint16_t* A_ = lds + (BUF) * (SA + SB) + (wm * 64 + (lane & 31)) * GT_LD;                        \
    const uint16_t* B_ = lds + (BUF) * (SA + SB) + SA + (wn * 64 + (lane & 31)) * GT_LD;                   \
    _Pragma("unroll") for (int ks = 0; ks < GT_BK / 16; ++ks) {                                           \
      bf16x8_t a[2], b[2];                                                                                \
      const int c_ = 2 * ks + (lane >> 5);                                                                \
      _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                       \
        a[i] = *reinterpret_cast<const bf16x8_t*>(A_ + 32 * i * GT_LD + 8 * c_);                          \
      _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                       \
        b[i] = *reinterpret_cast<const bf16x8_t*>(B_ + 32 * i * GT_LD + 8 * c_);                          \
      _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                       \
      _Pragma("unroll") for (int j = 0; j < 2; ++j)                                                       \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);              \
    }                                                                                                     \
    if ((S_) + 1 < n_stages) {                                                                            \
      RA_NXT.store(lds + ((BUF) ^ 1) * (SA + SB), t);                                                     \
      RB_NXT.store(lds + ((BUF) ^ 1) * (SA + SB) + SA, t);                                                \
    }                                                                                                     \
    __syncthreads();                                                                                      \
  }
  // operands swapped in the matrix-core call (B tile first): the accumulators
  // of lane l then hold row m = l % 32 of the block and, per group of four
  // registers, four consecutive columns
  // the stage count is even, so both copies run every iteration
#pragma unroll 1
  for (int s = 0; s < n_stages; s += 2) {
    NEDF_GEMM_STAGE(s, 0, ra0, rb0, ra1, rb1)
    NEDF_GEMM_STAGE(s + 1, 1, ra1, rb1, ra0, rb0)
  }
#undef NEDF_GEMM_STAGE
  // bfloat16 tile in LDS ([128][BN + 8]), then 16-byte row pieces.
  // Accumulator r of block (i, j): row 64 wm + 32 i + lane % 32, column
  // 64 wn + 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile
  constexpr int LO = BN + 8;
  static_assert(BM * LO <= 2 * (SA + SB), "output tile must fit the stage buffers");
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = wm * 64 + 32 * i + (lane & 31);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = wn * 64 + 32 * j + 8 * q + 4 * (lane >> 5);
        const float4 bb = *reinterpret_cast<const float4*>(g.bias + n0 + c);
        const float v0 = fmaxf(acc[i][j][4 * q] + bb.x, 0.f), v1 = fmaxf(acc[i][j][4 * q + 1] + bb.y, 0.f);
        const float v2 = fmaxf(acc[i][j][4 * q + 2] + bb.z, 0.f), v3 = fmaxf(acc[i][j][4 * q + 3] + bb.w, 0.f);
        *reinterpret_cast<uint2*>(lds + r * LO + c) =
            make_uint2(uint32_t(bf16_bits(v0)) | (uint32_t(bf16_bits(v1)) << 16),
                       uint32_t(bf16_bits(v2)) | (uint32_t(bf16_bits(v3)) << 16));
      }
  }
  __syncthreads();
  constexpr int CH = BM * BN / 8;  // 16-byte pieces of the tile
#pragma unroll
  for (int i = 0; i < CH / NT; ++i) {
    const int c = t + NT * i;
    const int r = c / (BN / 8), c8 = 8 * (c % (BN / 8));
    *reinterpret_cast<uint4*>(g.out16 + size_t(m0 + r) * g.ldo + n0 + c8) =
        *reinterpret_cast<const uint4*>(lds + r * LO + c8);
  }
}

// ---- weight gradients -----------------------------------------------------------
// dW_p = G_p^T X_p of several layers in one launch, over S batch splits, with
// the column sums of G_p (bias gradients).  M = width for every problem.
//
// A workgroup computes a 128 x 128 tile, a wave a 64 x 64 block of it.  Both
// operands lie with the batch (the product's k) outermost, in tiles of 32 x
// 32 (train_layout.h), which go to LDS as they are, by direct copies of 1 KB
// (the lanes put the samples in order on the way), 32 samples a stage in a
// ring of three, and are turned into fragments by transposing reads.  Bound by
// memory: 538 MB at 65,536 rows and 8 layers in 132 us (4.1 TB/s; 145 us when
// they were turned in registers, 32 byte permutes and an LDS write per 64
// values beside the products, and the column sums as many again in half of
// the waves), the classifier's 634 MB at 16,384 rows in 176 us (245).
//
// Three workgroups share a compute unit (48 KB of LDS each), so that the
// others' products cover one's waits, and a launch of up to 768 is one round.
struct WgradProb {
  const uint16_t* G;  // [B][M] in tiles
  const uint16_t* X;  // [B][ldx] in tiles, N = padded input width
  float* part;        // [S][M][N]
  float* colsum;      // [S][M]
  int ldx, N;
};
struct WgradBatch {
  WgradProb p[NEDF_TRAIN_MAX_LAYERS];
  int S, M, B;
};
constexpr int WG_TILE = 128;                  // rows and columns of a workgroup's tile
constexpr int WG_SLOT = 2 * WG_TILE * 32 * 2;  // bytes of a stage: 32 samples of both operands
constexpr int WG_SLOTS = 3;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// Of 16 lanes that read 16 values at each of four k (lane l: k l / 4, values
// 4 (l % 4) ..), lane i gets value i at the four k.
template <int OFF>
__device__ __forceinline__ u32x2 lds_read_tr(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}

__global__ __launch_bounds__(256, 3) void k_wgrad(WgradBatch wb) {
  // The tiles of one (problem, split) read the same rows of both operands.
  // Workgroups are handed to the 8 XCDs (each with its own L2) round-robin, so
  // consecutive logical ids lie on one XCD, an eighth of them on each: the
  // second read of an operand row is an L2 hit instead of an HBM read.  (A
  // grid over the widest problem's tiles, whose other workgroups left at
  // once, gave the XCD with the classifier's head 1.7 times the others' work.)
  const int total = gridDim.x, xcd = blockIdx.x % 8;
  const int lid = xcd * (total / 8) + min(xcd, total % 8) + int(blockIdx.x) / 8;
  // problem 0 has an input width of its own, the others N = M
  const int nx = wb.M / WG_TILE, t0 = nx * (wb.p[0].N / WG_TILE), t1 = nx * nx;
  const int rest = lid - t0 * wb.S;
  const int prob = rest < 0 ? 0 : 1 + rest / (t1 * wb.S);
  const int at = rest < 0 ? lid : rest % (t1 * wb.S), tiles = rest < 0 ? t0 : t1;
  const int split = at / tiles, bx = (at % tiles) % nx, by = (at % tiles) / nx;
  const WgradProb& p = wb.p[prob];
  __shared__ __attribute__((aligned(16))) uint8_t lds[WG_SLOTS * WG_SLOT];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 1, wn = wave & 1;
  const int m0 = bx * WG_TILE, n0 = by * WG_TILE;
  const int n = wb.B / wb.S / 32;  // stages, an even number
  // a stage's copies: wave w takes tile w of either operand, in two halves of
  // 16 samples; sample 8 c + j is row c + 4 j of the tile in memory
  const size_t a_step = size_t(32) * wb.M, b_step = size_t(32) * p.ldx;
  const uint16_t* Ab = p.G + size_t(split) * n * a_step + (m0 / 32 + wave) * 1024;
  const uint16_t* Bb = p.X + size_t(split) * n * b_step + (n0 / 32 + wave) * 1024;
  const uint32_t copy_off = uint32_t(nedf_train_tile_row(lane >> 2)) * 64u + 16u * (lane & 3);
  auto copy = [&](int st, int slot) __attribute__((always_inline)) {
    const int sc = min(st, n - 1);  // the last stage again past the end, into a free slot
    const eng::gbyte* ga = (const eng::gbyte*)(Ab + sc * a_step);
    const eng::gbyte* gb = (const eng::gbyte*)(Bb + sc * b_step);
    uint32_t off = copy_off;
    asm volatile("" : "+s"(ga), "+s"(gb), "+v"(off));
    uint8_t* d = lds + slot * WG_SLOT + wave * 2048;
    __builtin_amdgcn_global_load_lds((const void*)(ga + off), d, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)(ga + (off + 128u)), d + 1024, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)(gb + off), d + WG_SLOT / 2, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)(gb + (off + 128u)), d + WG_SLOT / 2 + 1024, 16, 0, 0);
  };
  // fragment reads: lane l takes value l % 32 at samples 8 (l / 32) .. + 7 of
  // a K-step, in two reads of four samples
  const uint32_t rd = eng::lds_offset(lds) + uint32_t(8 * (lane >> 5) + ((lane >> 2) & 3)) * 64u +
                      uint32_t(16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2u;
  const uint32_t rdA = rd + wm * 4096, rdB = rd + WG_SLOT / 2 + wn * 4096;
  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16_t{};
  // column sums (the first n tile's workgroups): wave (wm, wn) adds block wn
  // of its 64 rows; a lane's eight samples of each of four K-steps apart
  const bool sums = by == 0;
  float cs[4] = {0.f, 0.f, 0.f, 0.f};
  copy(0, 0);
  copy(1, 1);
  int cur = 0;
#pragma unroll 1
  for (int s0 = 0; s0 < n; s0 += 2) {
    eng::static_for<2>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      // stage s0 + q has landed (the next one may be in flight), and every
      // wave has read the stage before, whose slot the new copies take
      eng::dma_wait_barrier_n<4>();
      copy(s0 + q + 2, cur == 0 ? 2 : cur - 1);
      const uint32_t atA = rdA + cur * WG_SLOT, atB = rdB + cur * WG_SLOT;
      cur = cur == 2 ? 0 : cur + 1;
      u32x2 f[2][4][2];  // [K-step][A 0, A 1, B 0, B 1][samples 0..3, 4..7]
      eng::static_for<2>([&](auto kc) __attribute__((always_inline)) {
        constexpr int ks = decltype(kc)::value;
        eng::static_for<2>([&](auto ic) __attribute__((always_inline)) {
          constexpr int i = decltype(ic)::value;
          constexpr int at = i * 2048 + ks * 1024;
          f[ks][i][0] = lds_read_tr<at>(atA);
          f[ks][i][1] = lds_read_tr<at + 256>(atA);
          f[ks][2 + i][0] = lds_read_tr<at>(atB);
          f[ks][2 + i][1] = lds_read_tr<at + 256>(atB);
        });
      });
      eng::static_for<2>([&](auto kc) __attribute__((always_inline)) {
        constexpr int ks = decltype(kc)::value;
        u32x2(&w)[4][2] = f[ks];
        asm volatile("s_waitcnt lgkmcnt(%8)"
                     : "+v"(w[0][0]), "+v"(w[0][1]), "+v"(w[1][0]), "+v"(w[1][1]), "+v"(w[2][0]), "+v"(w[2][1]),
                       "+v"(w[3][0]), "+v"(w[3][1])
                     : "n"(ks == 0 ? 8 : 0));
        bf16x8_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          o[i] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(w[i][0], w[i][1], 0, 1, 2, 3));
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            // B first: lane l's accumulators hold row m = l % 32 of the block
            // and, per group of four, four consecutive columns
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o[2 + j], o[i], acc[i][j], 0, 0, 0);
        if (sums) {
          float s = 0.f;
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const uint32_t v = wn ? w[1][h][e] : w[0][h][e];
              s += __uint_as_float(v << 16) + __uint_as_float(v & 0xFFFF0000u);
            }
          cs[2 * q + ks] += s;
        }
      });
    });
  }
  // the copies past the end must land before the workgroup gives up its LDS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // accumulator r of block (i, j): row 64 wm + 32 i + lane % 32, column
  // 64 wn + 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = m0 + wm * 64 + 32 * i + (lane & 31);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = n0 + wn * 64 + 32 * j + 8 * q + 4 * (lane >> 5);
        *reinterpret_cast<float4*>(p.part + (size_t(split) * wb.M + row) * p.N + col) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      }
  }
  // the eight sums of a row (sample groups 0..7 of 64) in order
  if (sums) {
    float(&s_cs)[WG_TILE][8] = *reinterpret_cast<float(*)[WG_TILE][8]>(lds);
    __syncthreads();  // the ring is free
#pragma unroll
    for (int k = 0; k < 4; ++k) s_cs[wm * 64 + 32 * wn + (lane & 31)][2 * k + (lane >> 5)] = cs[k];
    __syncthreads();
    if (t < WG_TILE) {
      float s_ = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) s_ += s_cs[t][q];
      p.colsum[size_t(split) * wb.M + m0 + t] = s_;
    }
  }
}

// Weight and bias gradients of every hidden layer from the split partials,
// summed over the splits in order (deterministic): gW[m][k] for k < K, gb[m].
// The slice blockIdx.y = n_layers sums the chain's partials: one wave per
// output (regression form: 512 head weight gradients, 2 bias gradients, 3
// loss terms; classifier form: 3 loss terms), lane l adding workgroups l, l +
// 64, ... in order, then a fixed butterfly.  The first thread also counts the update in the Adam
// step counter, which the Adam launch after this one reads.
struct ReduceLayer {
  const float* part;   // [S][M][N]
  const float* csum;   // [S][M]
  float* gW;           // [M][K]
  float* gb;           // [M]
  int M, N, K;
};
struct ReduceArgs {
  ReduceLayer L[NEDF_TRAIN_MAX_LAYERS];
  int n_layers, S;
  int64_t* step;
  // regression form: head partials [h_blocks][HEAD_PART]; classifier form:
  // loss sums [h_blocks][3] (gWh null), over B samples
  const float* hpart;
  int h_blocks, B;
  float *gWh, *gbh, *loss;
};
__global__ void k_reduce_grads(ReduceArgs r) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *r.step += 1;
  if (int(blockIdx.y) == r.n_layers) {
    const int j = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int row = r.gWh ? HEAD_PART : 3;
    if (j >= (r.gWh ? 517 : 3)) return;
    float s = 0.f;
    for (int q = lane; q < r.h_blocks; q += 64) s += r.hpart[size_t(q) * row + j];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane != 0) return;
    if (!r.gWh) r.loss[j] = s / float(r.B);
    else if (j < 512) r.gWh[j] = s;
    else if (j < 514) r.gbh[j - 512] = s;
    else r.loss[j - 514] = s;
    return;
  }
  const ReduceLayer& L = r.L[blockIdx.y];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int MN = L.M * L.N;
  if (i < MN) {
    const int m = i / L.N, n = i % L.N;
    if (n < L.K) {
      float s = 0.f;
      for (int q = 0; q < r.S; ++q) s += L.part[size_t(q) * MN + i];
      L.gW[size_t(m) * L.K + n] = s;
    }
  } else if (i < MN + L.M) {
    const int m = i - MN;
    float s = 0.f;
    for (int q = 0; q < r.S; ++q) s += L.csum[size_t(q) * L.M + m];
    L.gb[m] = s;
  }
}

__global__ void k_zero_f32(float* p, size_t n) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// Adam (Kingma & Ba 2015) with bias correction, step t = *step (counted by
// the gradient reduction just before), over every
// parameter array of the network in one launch (segments listed in AdamArgs;
// a block never spans two segments); the bfloat16 copy of weight matrices is
// refreshed in the same pass.
struct AdamSeg {
  float *p, *m, *v;
  const float* g;
  uint16_t* w16;  // or null: packed copy (train_layout.h)
  uint16_t* w16t; // or null: packed transpose
  int n, K, Kpad, N;
  int k_outer;    // K-steps of the packed copy outermost
  int block0;     // first block of this segment
};
struct AdamArgs {
  AdamSeg seg[2 * (NEDF_MAX_LAYERS + 1)];
  int n_seg;
  const int64_t* step;
  float lr, b1, b2, eps;
};
__global__ void k_adam(AdamArgs a) {
  int si = 0;
  while (si + 1 < a.n_seg && int(blockIdx.x) >= a.seg[si + 1].block0) ++si;
  const AdamSeg& S = a.seg[si];
  const int i = (int(blockIdx.x) - S.block0) * blockDim.x + threadIdx.x;
  if (i >= S.n) return;
  const float t = float(*a.step);
  const float bc1 = 1.0f - powf(a.b1, t), bc2 = 1.0f - powf(a.b2, t);
  const float gi = S.g[i];
  const float mi = a.b1 * S.m[i] + (1.0f - a.b1) * gi;
  const float vi = a.b2 * S.v[i] + (1.0f - a.b2) * gi * gi;
  S.m[i] = mi;
  S.v[i] = vi;
  const float pi = S.p[i] - a.lr * (mi / bc1) / (sqrtf(vi / bc2) + a.eps);
  S.p[i] = pi;
  if (!S.w16) return;
  const int r = i / S.K, c = i % S.K;
  S.w16[nedf_train_frag(r, c, S.Kpad / 16, S.k_outer)] = bf16_bits(pi);
  if (S.w16t) S.w16t[nedf_train_frag(c, r, S.N / 16, 0)] = bf16_bits(pi);
}

// Initial state: master weights from float32 arrays, moments and gradients
// zero, bfloat16 copies (zero padded): row-major (packed = 0, the calibration
// pass), or packed as fragments (1; 2: K-steps outermost) with their transpose.
__global__ void k_copy_w(const float* src, float* dst, uint16_t* w16, uint16_t* w16t, int N, int K, int Kpad,
                         int Nsrc, int packed) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N * Kpad) return;
  const int r = i / Kpad, c = i % Kpad;
  const float v = (c < K && r < Nsrc) ? src[r * K + c] : 0.0f;
  if (c < K && dst) dst[r * K + c] = v;
  if (w16) w16[packed ? nedf_train_frag(r, c, Kpad / 16, packed == 2) : size_t(i)] = bf16_bits(v);
  if (w16t) w16t[nedf_train_frag(c, r, N / 16, 0)] = bf16_bits(v);
}

unsigned blocks(size_t n, int b = 256) { return unsigned((n + b - 1) / b); }

void launch_encode_rows(const nedf_mlp_shape& sh, const float* o_l, const float* d_l, int B, int K0p, uint16_t* H,
                        hipStream_t s) {
  const dim3 grid(blocks(size_t(B) * (K0p / 8)));
  if (sh.in_kind == NEDF_IN_PLUECKER)
    hipLaunchKernelGGL(k_encode_rows<6>, grid, dim3(256), 0, s, o_l, d_l, B, sh.enc_L, K0p, H);
  else
    hipLaunchKernelGGL(k_encode_rows<3>, grid, dim3(256), 0, s, o_l, d_l, B, sh.enc_L, K0p, H);
}

// ---- classifier-form network (NEDF_IN_POINTS16) ---------------------------------
// Encoded input of the 16 line points (natural order: point-major, each
// [x, sin(2^0 pi x), cos(2^0 pi x), ...], 63 values) zero padded to Kpad, and
// labels mu* = (t_perp - D) / l, alpha = hit.  The points come from the
// compensated frame of the inference kernel, applied to the local ray.
template <int L>
__global__ void k_train_encode_points(const float* o_l, const float* d_l, const float* depth, const uint8_t* hit,
                                      int B, int Kpad, float bound, uint16_t* H, float* mu, float* alpha) {
  constexpr int per = 3 * (1 + 2 * L);  // features per point
  const int groups = Kpad / 8;
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int s = tid / groups, grp = tid % groups;
  if (s >= B) return;
  const float o[3] = {o_l[3 * s], o_l[3 * s + 1], o_l[3 * s + 2]};
  const float d[3] = {d_l[3 * s], d_l[3 * s + 1], d_l[3 * s + 2]};
  const float zero[3] = {0.f, 0.f, 0.f};
  W2L id{};
  id.rt[0] = id.rt[4] = id.rt[8] = 1.0f;
  id.s = id.inv_s = 1.0f;
  f2 q[3], dv[3];
  float tperp, ol[3];
  local_points_frame(id, o, d, zero, bound, q, dv, tperp, ol);
  // point p of the line (compensated: value and low part), for the at most
  // two points this thread's 8 features belong to
  auto point = [&](int p, float (&x)[3], float (&xlo)[3]) {
    const float cp = float(2 * p + 1) * 0.0625f - 1.0f;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma clang fp contract(off)
      const f2 pp = two_prod(cp, dv[r].hi);
      const f2 sm = two_sum(q[r].hi, pp.hi);
      x[r] = sm.hi;
      xlo[r] = sm.lo + ((pp.lo + q[r].lo) + cp * dv[r].lo);
    }
  };
  const int pa = (8 * grp) / per;
  float xa[3], xla[3], xb[3], xlb[3];
  point(pa, xa, xla);
  point(pa + 1, xb, xlb);
  uint32_t packed[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    float v2[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int f = 8 * grp + e + u;
      float v = 0.0f;
      if (f < NEDF_CLS_POINTS * per) {
        const bool second = f >= (pa + 1) * per;
        const int e2 = f - (second ? pa + 1 : pa) * per;
        float x[3], xlo[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          x[r] = second ? xb[r] : xa[r];
          xlo[r] = second ? xlb[r] : xla[r];
        }
        if (e2 < 3) {
          v = e2 == 0 ? x[0] : e2 == 1 ? x[1] : x[2];
        } else {
          const int qq = e2 - 3, level = qq / 6, w = qq % 6, c = w % 3;
          const float xc = c == 0 ? x[0] : c == 1 ? x[1] : x[2];
          const float xlc = c == 0 ? xlo[0] : c == 1 ? xlo[1] : xlo[2];
          v = sinpi_hw(float(1 << level) * xc, float(1 << level) * xlc, w >= 3 ? 1 : 0);
        }
      }
      v2[u] = v;
    }
    packed[e / 2] = uint32_t(bf16_bits(v2[0])) | (uint32_t(bf16_bits(v2[1])) << 16);
  }
  // in tiles of 32 samples x 32 features
  uint16_t* dst = H + size_t(s / 32) * (32 * size_t(Kpad)) + (grp / 4) * 1024 + nedf_train_tile_row(s % 32) * 32 +
                  8 * (grp % 4);
  *reinterpret_cast<uint4*>(dst) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
  if (grp != 0) return;
  const bool h = hit[s] != 0;
  alpha[s] = h ? 1.0f : 0.0f;
  mu[s] = h ? (tperp - depth[s]) / bound : 0.0f;
}

}  // namespace

// Split count of a batched weight-gradient launch over `tiles` 128 x 128
// output tiles: a power of two up to 64 giving at most 640 workgroups, one
// round (three share a compute unit, 768 in all; a second round would be part
// empty, and every split's partial sums are written and read back), with the
// batch a multiple of 128 per split (the batch is a multiple of 256).
int wgrad_batch_splits(int B, int tiles) {
  int S = 1;
  while (S < 64 && tiles * S * 2 <= 640 && B % (S * 2 * 128) == 0) S *= 2;
  return S;
}

// 128 x 128 output tiles of the regression form's hidden-layer weight gradients.
int regression_wgrad_tiles(const nedf_mlp_shape& sh, const nedf_train_layout& tl) {
  int t = 0;
  for (int l = 0; l < sh.n_hidden; ++l) t += (sh.width / 128) * (tl.L[l].Kpad / 128);
  return t;
}

size_t train_ws_bytes_cls(const nedf_mlp_shape& sh, int B);

size_t train_ws_bytes(const nedf_mlp_shape& sh, int B) {
  if (sh.in_kind == NEDF_IN_POINTS16) return train_ws_bytes_cls(sh, B);
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  const int S = wgrad_batch_splits(B, regression_wgrad_tiles(sh, tl));
  size_t off = 0;
  off = nedf_tl_align(off + size_t(B) * tl.L[0].Kpad * 2);           // H_in
  off = nedf_tl_align(off + size_t(B) * sh.width * 2 * sh.n_hidden);  // H_0..H_{n-1}
  off = nedf_tl_align(off + size_t(B) * sh.width * 2 * sh.n_hidden);  // G_0..G_{n-1}
  off = nedf_tl_align(off + size_t(B) * (sh.width / 8) * sh.n_hidden);  // ReLU mask bits of H_0..H_{n-1}
  for (int l = 0; l < sh.n_hidden; ++l)                                // weight-gradient partials
    off = nedf_tl_align(off + size_t(S) * sh.width * (tl.L[l].Kpad + 1) * 4);
  off = nedf_tl_align(off + size_t(B / GT_BM) * HEAD_PART * 4);  // head partials, per 128-row tile
  return off;
}

namespace {
// packed: bfloat16 copies as matrix-core fragments (training), or row-major
// (the calibration pass)
hipError_t init_state(const nedf_mlp_shape& sh, const float* const* W, const float* const* b, uint8_t* st,
                      bool packed, hipStream_t s) {
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  hipLaunchKernelGGL(k_zero_f32, dim3(blocks(tl.total / 4)), dim3(256), 0, s, reinterpret_cast<float*>(st),
                     tl.total / 4);
  for (int i = 0; i < tl.n_layers; ++i) {
    const nedf_train_layer& l = tl.L[i];
    // the regression form's head has no copies, first layers no transpose
    const bool copies = l.N % 32 == 0;
    const bool cls = sh.in_kind == NEDF_IN_POINTS16;
    hipLaunchKernelGGL(k_copy_w, dim3(blocks(size_t(l.N) * l.Kpad)), dim3(256), 0, s, W[i],
                       reinterpret_cast<float*>(st + l.W), copies ? reinterpret_cast<uint16_t*>(st + l.W16) : nullptr,
                       copies && packed && i > 0 ? reinterpret_cast<uint16_t*>(st + l.W16T) : nullptr, l.N, l.K, l.Kpad,
                       l.Nsrc, !packed ? 0 : cls && i == 0 ? 2 : 1);
    // the bias as one row of N values, of which the caller's array holds Nsrc
    hipLaunchKernelGGL(k_copy_w, dim3(blocks(size_t(l.N))), dim3(256), 0, s, b[i],
                       reinterpret_cast<float*>(st + l.b), static_cast<uint16_t*>(nullptr),
                       static_cast<uint16_t*>(nullptr), 1, l.Nsrc, l.N, 1, 0);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_train_init(const nedf_mlp_shape& sh, const float* const* W, const float* const* b, uint8_t* st,
                             hipStream_t s) {
  return init_state(sh, W, b, st, true, s);
}

hipError_t launch_train_step_cls(const nedf_mlp_shape& sh, uint8_t* st, const float* o_l, const float* d_l,
                                 const float* depth, const uint8_t* hit, int B, float lr, float b1, float b2,
                                 float eps, float w_hit, float bound, float* loss, uint8_t* ws, hipStream_t s);

hipError_t launch_train_step(const nedf_mlp_shape& sh, uint8_t* st, const float* o_l, const float* d_l,
                             const float* depth, const uint8_t* hit, int B, float lr, float b1, float b2, float eps,
                             float w_hit, float bound, float* loss, uint8_t* ws, hipStream_t s) {
  if (sh.in_kind == NEDF_IN_POINTS16)
    return launch_train_step_cls(sh, st, o_l, d_l, depth, hit, B, lr, b1, b2, eps, w_hit, bound, loss, ws, s);
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  const int W = sh.width, NH = sh.n_hidden;
  const int K0p = tl.L[0].Kpad;
  const int S = wgrad_batch_splits(B, regression_wgrad_tiles(sh, tl));
  size_t off = 0;
  uint16_t* Hin = reinterpret_cast<uint16_t*>(ws + off);
  off = nedf_tl_align(off + size_t(B) * K0p * 2);
  uint16_t* Hs = reinterpret_cast<uint16_t*>(ws + off);
  off = nedf_tl_align(off + size_t(B) * W * 2 * NH);
  uint16_t* Gs = reinterpret_cast<uint16_t*>(ws + off);
  off = nedf_tl_align(off + size_t(B) * W * 2 * NH);
  uint8_t* bits = ws + off;
  off = nedf_tl_align(off + size_t(B) * (W / 8) * NH);
  float* wpart[NEDF_MAX_LAYERS];
  for (int l = 0; l < NH; ++l) {
    wpart[l] = reinterpret_cast<float*>(ws + off);
    off = nedf_tl_align(off + size_t(S) * W * (tl.L[l].Kpad + 1) * 4);
  }
  float* hpart = reinterpret_cast<float*>(ws + off);
  const int waves = chain_line_waves(B, cu_count());
  const int hblocks = B / GT_BM;
  auto Hl = [&](int l) { return Hs + size_t(l) * B * W; };
  auto Gl = [&](int l) { return Gs + size_t(l) * B * W; };  // gradient at layer l's pre-activation
  auto F = [&](size_t o) { return reinterpret_cast<float*>(st + o); };
  auto U = [&](size_t o) { return reinterpret_cast<uint16_t*>(st + o); };

  prof_mark("train.step", s, true);
  // encoding, forward pass, head, loss and data gradients in one kernel
  const nedf_train_layer& hd = tl.L[NH];
  {
    ChainLineArgs c{};
    c.o_l = o_l; c.d_l = d_l; c.depth = depth; c.hit = hit;
    c.B = B; c.enc_L = sh.enc_L; c.n_hidden = NH;
    c.bound = bound; c.w_hit = w_hit;
    for (int l = 0; l < NH; ++l) {
      c.w[l] = st + tl.L[l].W16;
      c.wt[l] = st + tl.L[l].W16T;
      c.bias[l] = F(tl.L[l].b);
    }
    c.head_w = F(hd.W); c.head_b = F(hd.b);
    c.Hin = Hin; c.H = Hs; c.G = Gs; c.bits = bits; c.hpart = hpart;
    launch_chain_line(c, sh.in_kind == NEDF_IN_PLUECKER ? 6 : 3, K0p / 16, waves, s);
  }
  // weight-gradient partials dW_l = G_l^T H_{l-1} of every layer in one
  // launch, then their sums over the splits in order
  {
    WgradBatch wb{};
    wb.S = S; wb.M = W; wb.B = B;
    ReduceArgs ra{};
    ra.n_layers = NH;
    ra.S = S;
    ra.step = reinterpret_cast<int64_t*>(st);
    ra.hpart = hpart; ra.h_blocks = hblocks;
    ra.gWh = F(hd.gW); ra.gbh = F(hd.gb); ra.loss = loss;
    int maxmn = 517 * 64;  // the head slice: one wave per output
    for (int l = 0; l < NH; ++l) {
      const nedf_train_layer& L = tl.L[l];
      wb.p[l] = WgradProb{Gl(l), l == 0 ? Hin : Hl(l - 1), wpart[l], wpart[l] + size_t(S) * W * L.Kpad,
                          l == 0 ? K0p : W, L.Kpad};
      ra.L[l] = ReduceLayer{wb.p[l].part, wb.p[l].colsum, F(L.gW), F(L.gb), W, L.Kpad, L.K};
      maxmn = std::max(maxmn, W * L.Kpad + W);
    }
    hipLaunchKernelGGL(k_wgrad, dim3(regression_wgrad_tiles(sh, tl) * S), dim3(256), 0, s, wb);
    hipLaunchKernelGGL(k_reduce_grads, dim3(blocks(maxmn), NH + 1), dim3(256), 0, s, ra);
  }
  // Adam on every parameter array, one launch
  AdamArgs aa{};
  aa.step = reinterpret_cast<const int64_t*>(st);
  aa.lr = lr; aa.b1 = b1; aa.b2 = b2; aa.eps = eps;
  int nb = 0;
  for (int i = 0; i < tl.n_layers; ++i) {
    const nedf_train_layer& L = tl.L[i];
    const bool copies = i < NH;
    aa.seg[aa.n_seg++] = AdamSeg{F(L.W), F(L.mW), F(L.vW), F(L.gW), copies ? U(L.W16) : nullptr,
                                 copies && i > 0 ? U(L.W16T) : nullptr, L.N * L.K, L.K, L.Kpad, L.N, 0, nb};
    nb += int(blocks(size_t(L.N) * L.K));
    aa.seg[aa.n_seg++] = AdamSeg{F(L.b), F(L.mb), F(L.vb), F(L.gb), nullptr, nullptr, L.N, 1, 1, 1, 0, nb};
    nb += int(blocks(size_t(L.N)));
  }
  hipLaunchKernelGGL(k_adam, dim3(nb), dim3(256), 0, s, aa);
  prof_mark("train.step", s, false);
  return hipGetLastError();
}

// ---- classifier-form training step ----------------------------------------------
namespace {
// 128 x 128 output tiles of every layer's weight gradient (the tail's N
// padded to the width).
int cls_wgrad_tiles(const nedf_train_layout& tl, int W) {
  int t = 0;
  for (int i = 0; i < tl.n_layers; ++i) t += (W / 128) * (tl.L[i].Kpad / 128);
  return t;
}
struct ClsTrainWs {
  uint16_t *X, *H, *A, *G;
  uint8_t* bits;
  float *mu, *alpha, *wpart, *lpart;
  size_t part_off[NEDF_TRAIN_MAX_LAYERS];  // each layer's split partials, floats from wpart
  size_t end;
};
ClsTrainWs cls_train_ws(const nedf_mlp_shape& sh, int B, uint8_t* base) {
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  const int W = sh.width, NB = sh.n_hidden, K0p = tl.L[0].Kpad;
  const int S = wgrad_batch_splits(B, cls_wgrad_tiles(tl, W));
  ClsTrainWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    uint8_t* p = base ? base + off : nullptr;
    off = nedf_tl_align(off + bytes);
    return p;
  };
  w.X = reinterpret_cast<uint16_t*>(take(size_t(B) * K0p * 2));
  w.H = reinterpret_cast<uint16_t*>(take(size_t(B) * W * 2 * (NB + 1)));
  w.A = reinterpret_cast<uint16_t*>(take(size_t(B) * W * 2 * NB));
  // the bfloat16 gradient at every layer's pre-activation
  w.G = reinterpret_cast<uint16_t*>(take(size_t(B) * W * 2 * tl.n_layers));
  // signs of the head's output and of each block's two layers
  w.bits = take(size_t(B) * (W / 8) * (2 * NB + 1));
  w.mu = reinterpret_cast<float*>(take(size_t(B) * 4));
  w.alpha = reinterpret_cast<float*>(take(size_t(B) * 4));
  size_t nf = 0;
  for (int i = 0; i < tl.n_layers; ++i) {
    w.part_off[i] = nf;
    nf += size_t(S) * W * (tl.L[i].Kpad + 1);
    nf = (nf + 63) & ~size_t(63);
  }
  w.wpart = reinterpret_cast<float*>(take(nf * 4));
  w.lpart = reinterpret_cast<float*>(take(size_t(B / 64) * 3 * 4));
  w.end = off;
  return w;
}
}  // namespace

size_t train_ws_bytes_cls(const nedf_mlp_shape& sh, int B) { return cls_train_ws(sh, B, nullptr).end; }

// One Adam step of a classifier-form network (Eq. 6): encoding, the forward
// and backward chain, the weight gradients by split-K products reduced in
// order, Adam.
hipError_t launch_train_step_cls(const nedf_mlp_shape& sh, uint8_t* st, const float* o_l, const float* d_l,
                                 const float* depth, const uint8_t* hit, int B, float lr, float b1, float b2,
                                 float eps, float w_hit, float bound, float* loss, uint8_t* ws, hipStream_t s) {
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  const int W = sh.width, NB = sh.n_hidden;
  const int K0p = tl.L[0].Kpad;
  const int S = wgrad_batch_splits(B, cls_wgrad_tiles(tl, W));
  const ClsTrainWs w = cls_train_ws(sh, B, ws);
  auto F = [&](size_t o) { return reinterpret_cast<float*>(st + o); };
  auto U = [&](size_t o) { return reinterpret_cast<uint16_t*>(st + o); };
  auto Hk = [&](int k) { return w.H + size_t(k) * B * W; };
  auto Ak = [&](int k) { return w.A + size_t(k) * B * W; };
  auto Gi = [&](int i) { return w.G + size_t(i) * B * W; };  // gradient at layer i's pre-activation
  const int tail = tl.n_layers - 1;
  const int waves = chain_points_waves(B, cu_count());
  prof_mark("train.step", s, true);
  // gamma_10 (the only classifier encoding training accepts)
  hipLaunchKernelGGL(k_train_encode_points<10>, dim3(blocks(size_t(B) * (K0p / 8))), dim3(256), 0, s, o_l, d_l, depth,
                     hit, B, K0p, bound, w.X, w.mu, w.alpha);
  {
    ChainPointsArgs c{};
    c.B = B; c.n_blocks = NB; c.w_hit = w_hit;
    for (int i = 0; i < tl.n_layers; ++i) {
      c.w[i] = st + tl.L[i].W16;
      c.wt[i] = st + tl.L[i].W16T;
      c.bias[i] = F(tl.L[i].b);
    }
    c.X = w.X; c.mu = w.mu; c.alpha = w.alpha;
    c.H = w.H; c.A = w.A; c.G = w.G; c.bits = w.bits; c.lpart = w.lpart;
    launch_chain_points(c, waves, s);
  }
  // weight gradients of every layer from its pre-activation gradient and its
  // input, in one launch, then their sums over the splits in order
  {
    WgradBatch wb{};
    wb.S = S; wb.M = W; wb.B = B;
    ReduceArgs ra{};
    ra.n_layers = tl.n_layers;
    ra.S = S;
    ra.step = reinterpret_cast<int64_t*>(st);
    ra.hpart = w.lpart; ra.h_blocks = B / (32 * waves); ra.B = B;
    ra.loss = loss;
    int maxmn = 0;
    for (int i = 0; i < tl.n_layers; ++i) {
      const nedf_train_layer& L = tl.L[i];
      const uint16_t* X = i == 0 ? w.X : i == tail ? Hk(NB) : (i % 2 == 1 ? Hk((i - 1) / 2) : Ak((i - 2) / 2));
      float* part = w.wpart + w.part_off[i];
      wb.p[i] = WgradProb{Gi(i), X, part, part + size_t(S) * W * L.Kpad, i == 0 ? K0p : W, L.Kpad};
      ra.L[i] = ReduceLayer{part, part + size_t(S) * W * L.Kpad, F(L.gW), F(L.gb), W, L.Kpad, L.K};
      maxmn = std::max(maxmn, W * L.Kpad + W);
    }
    hipLaunchKernelGGL(k_wgrad, dim3(cls_wgrad_tiles(tl, W) * S), dim3(256), 0, s, wb);
    hipLaunchKernelGGL(k_reduce_grads, dim3(blocks(maxmn), tl.n_layers + 1), dim3(256), 0, s, ra);
  }
  // Adam, in launches of at most one argument block of segments
  AdamArgs aa{};
  aa.step = reinterpret_cast<const int64_t*>(st);
  aa.lr = lr; aa.b1 = b1; aa.b2 = b2; aa.eps = eps;
  int nb = 0;
  auto flush = [&]() {
    if (aa.n_seg) hipLaunchKernelGGL(k_adam, dim3(nb), dim3(256), 0, s, aa);
    aa.n_seg = 0;
    nb = 0;
  };
  constexpr int MAXSEG = int(sizeof(aa.seg) / sizeof(aa.seg[0]));
  for (int i = 0; i < tl.n_layers; ++i) {
    if (aa.n_seg + 2 > MAXSEG) flush();
    const nedf_train_layer& L = tl.L[i];
    aa.seg[aa.n_seg++] = AdamSeg{F(L.W), F(L.mW), F(L.vW), F(L.gW), U(L.W16), i > 0 ? U(L.W16T) : nullptr, L.N * L.K,
                                 L.K, L.Kpad, L.N, i == 0, nb};
    nb += int(blocks(size_t(L.N) * L.K));
    aa.seg[aa.n_seg++] = AdamSeg{F(L.b), F(L.mb), F(L.vb), F(L.gb), nullptr, nullptr, L.N, 1, 1, 1, 0, nb};
    nb += int(blocks(size_t(L.N)));
  }
  flush();
  prof_mark("train.step", s, false);
  return hipGetLastError();
}

// Per-layer E4M3 scales of a network from a calibration batch: the bfloat16
// forward pass of the training path records amax of every hidden layer's
// input; weight scales from the float32 weights.  ws holds a temporary
// training state followed by the forward workspace.
hipError_t launch_fp8_calibrate(const nedf_mlp_shape& sh, const float* const* W, const float* const* b,
                                const float* o_l, const float* d_l, int B, float* scales, uint8_t* ws,
                                hipStream_t s) {
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  uint8_t* st = ws;
  uint8_t* fw = ws + nedf_tl_align(tl.total);
  uint32_t* amax = reinterpret_cast<uint32_t*>(fw + train_ws_bytes(sh, B));
  const int W_ = sh.width, NH = sh.n_hidden;
  hipError_t e = init_state(sh, W, b, st, false, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_zero_f32, dim3(1), dim3(64), 0, s, reinterpret_cast<float*>(amax), size_t(2 * NEDF_MAX_LAYERS));
  const int K0p = tl.L[0].Kpad;
  uint16_t* Hin = reinterpret_cast<uint16_t*>(fw);
  uint16_t* Hs = reinterpret_cast<uint16_t*>(fw + nedf_tl_align(size_t(B) * K0p * 2));
  launch_encode_rows(sh, o_l, d_l, B, K0p, Hin, s);
  hipLaunchKernelGGL(k_amax16, dim3(256), dim3(256), 0, s, Hin, size_t(B) * K0p, amax + NEDF_MAX_LAYERS);
  for (int l = 0; l < NH; ++l) {
    GemmArgs g{};
    g.A = l == 0 ? Hin : Hs + size_t(l - 1) * B * W_;
    g.lda = l == 0 ? K0p : W_;
    g.B = reinterpret_cast<const uint16_t*>(st + tl.L[l].W16);
    g.ldb = tl.L[l].Kpad;
    g.M = B; g.N = W_; g.K = tl.L[l].Kpad;
    g.bias = reinterpret_cast<const float*>(st + tl.L[l].b);
    g.out16 = Hs + size_t(l) * B * W_;
    g.ldo = W_;
    hipLaunchKernelGGL(k_gemm, dim3(B / GT_BM, W_ / GT_BN), dim3(512), 0, s, g);
    if (l + 1 < NH) hipLaunchKernelGGL(k_amax16, dim3(256), dim3(256), 0, s, g.out16, size_t(B) * W_, amax + NEDF_MAX_LAYERS + l + 1);
    hipLaunchKernelGGL(k_amax32, dim3(64), dim3(256), 0, s, reinterpret_cast<const float*>(st + tl.L[l].W),
                       size_t(tl.L[l].N) * tl.L[l].K, amax + l);
  }
  hipLaunchKernelGGL(k_fp8_scales, dim3(1), dim3(64), 0, s, amax, amax + NEDF_MAX_LAYERS, NH, scales);
  return hipGetLastError();
}

size_t fp8_calibrate_ws_bytes(const nedf_mlp_shape& sh, int B) {
  return nedf_tl_align(nedf_train_layout_of(sh).total) + train_ws_bytes(sh, B) + 2 * NEDF_MAX_LAYERS * 4 + 256;
}

hipError_t launch_train_export(const nedf_mlp_shape& sh, const uint8_t* st, float* const* W, float* const* b,
                               bool grads, hipStream_t s) {
  const nedf_train_layout tl = nedf_train_layout_of(sh);
  for (int i = 0; i < tl.n_layers; ++i) {
    const nedf_train_layer& l = tl.L[i];
    const size_t ow = grads ? l.gW : l.W, ob = grads ? l.gb : l.b;
    hipError_t e = hipMemcpyAsync(W[i], st + ow, size_t(l.Nsrc) * l.K * 4, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(b[i], st + ob, size_t(l.Nsrc) * 4, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace nedf
