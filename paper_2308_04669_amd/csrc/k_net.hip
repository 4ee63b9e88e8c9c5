// The NeDF intersection network (Eq. 1, 2, 7) in its regression form, with
// routing of uncertain pairs to the marcher (short BF16 and FP32 lists run on
// the feature-split kernel).
#include "pipeline.h"
#include "runtime.h"

namespace nedf {
namespace {

// NeDF stage: a workgroup takes items of 128 NB pairs (32 NB per wave) of
// one object; each lane pair evaluates the intersection network on its pairs'
// line coordinates (NB blocks of 32 pairs share every weight read from LDS).
// Confident hits go to the key buffer, uncertain pairs (and origins inside
// the bounding sphere) to list B for the marcher.
template <int DT, int WIDTH, int NHID, int L, int SBX, int OCC, int NB, int NW>
__global__ __launch_bounds__(64 * NW, OCC) void k_nedf(KArgs a) {
  using T = eng::Tr<DT>;
  constexpr int PPW = 32 * NB;  // pairs per wave and item
  constexpr int KS0 = eng::ks_for_slots<DT>(6 * L + 3);
  constexpr int KSH = WIDTH / T::KPS;
  constexpr int CHUNK = eng::cmax(eng::chunk_bytes<DT>(KS0, 0), eng::chunk_bytes<DT>(KSH, 2));
  __shared__ __attribute__((aligned(16))) uint8_t lds[eng::NBUF * eng::slot_bytes(CHUNK, SBX)];
  // per-lane pair state parked across the network (keeps registers free)
  constexpr int NT = 64 * NW;
  __shared__ __attribute__((aligned(16))) uint8_t s_stash[16 * NB * NT];
  __shared__ int s_item;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const uint32_t stash = eng::lds_offset(s_stash) + 16u * threadIdx.x;
  __shared__ ItemTable s_tab;  // the current depth slab
  if (!build_items(a, s_tab, PPW * NW)) return;
  const int total = s_tab.total;
  if (threadIdx.x == 0) s_item = atomicAdd(a.lwork, 1);
  __syncthreads();
  int item = s_item;
  int slot = 0;
  bool primed = false;
  // routing counts, per wave, flushed once at the end
  int n_route[3] = {0, 0, 0};
  while (item < total) {
    // claim the next item now so that its weights stream in behind this pass
    __syncthreads();
    if (threadIdx.x == 0) s_item = atomicAdd(a.lwork, 1);
    __syncthreads();
    const int next = s_item;
    const int obj = item_object(s_tab, a.n_obj, item);
    const int first = (item - s_tab.start[obj]) * (PPW * NW) + wave * PPW + (lane & 31);
    const ObjDesc& od = a.obj[obj];
    const uint8_t* blob = od.nedf_blob;
    const uint8_t* next_blob = next < total ? a.obj[item_object(s_tab, a.n_obj, next)].nedf_blob : nullptr;
    const nedf_blob_header* hb = reinterpret_cast<const nedf_blob_header*>(blob);
    const float* hbias_p = reinterpret_cast<const float*>(blob + uniform_load_u64(&hb->off_head_b));
    const float hbias[2] = {uniform_load_f32(hbias_p), uniform_load_f32(hbias_p + 1)};
    const float l = od.bound;
    typename T::frag Benc[NB][KS0];
    const float in_scale = DT == 2 ? uniform_load_f32(blob + uniform_load_u64(&hb->off_scales)) : 1.0f;
    // lane-half-dependent encoding constants are recomputed per pass rather
    // than hoisted out of the loop (where they would stay live, and spill,
    // across the network)
    int half_v = half;
    asm volatile("" : "+v"(half_v));
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int local = first + 32 * nb;
      const bool valid = local < s_tab.cnt[obj];
      const uint2 pr = a.pairs[s_tab.off[obj] + (valid ? local : 0)];
      const W2L g = load_w2l(a.w2l, int(pr.y));
      float o[3], d[3], dlo[3], ol[3], pl[6], pllo[6], tperp;
      make_ray(a.rays, pr.x, o, d, dlo);
      local_line(g, o, d, dlo, pl, pllo, tperp, ol);
      const bool inside = sum_sq(ol[0], ol[1], ol[2]) < l * l;
      eng::encode_input<DT, 6, L, KS0>(pl, pllo, half_v, Benc[nb], in_scale);
      // ray and instance ids (< 2^31, flags in bit 31), t_perp and s
      eng::lds_write16(stash + uint32_t(nb) * (16u * NT),
                       eng::u32x4{pr.x | (valid ? 0x80000000u : 0u), pr.y | (inside ? 0x80000000u : 0u),
                                  __float_as_uint(tperp), __float_as_uint(g.s)});
    }
    float partial[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) partial[nb][0] = partial[nb][1] = 0.f;
    typename T::frag Blast[NB][KSH];
    eng::trunk<DT, WIDTH, KS0, NHID, 2, CHUNK, false, 0, WIDTH / 32, SBX, NB, NW>(hb, blob, Benc, lds, partial, Blast,
                                                                             nullptr, &slot, next_blob, primed);
    primed = next_blob != nullptr;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      eng::u32x4 st = eng::lds_read16<0>(stash + uint32_t(nb) * (16u * NT));
      eng::lds_wait1<0>(st);
      const uint2 prs = make_uint2(st.x & 0x7FFFFFFFu, st.y & 0x7FFFFFFFu);
      const bool valid_s = (st.x >> 31) != 0, inside_s = (st.y >> 31) != 0;
      const float mu_hat = partial[nb][0] + __shfl_xor(partial[nb][0], 32) + hbias[0];
      const float z = partial[nb][1] + __shfl_xor(partial[nb][1], 32) + hbias[1];
      const float p = sigmoidf_(z);
      const float D = __uint_as_float(st.w) * (__uint_as_float(st.z) - l * fminf(fmaxf(mu_hat, -1.0f), 1.0f));
      route_pairs(a, obj, s_tab.off[obj], prs, valid_s && half == 0, inside_s, p, D, lane, n_route);
    }
    item = next;
  }
  flush_routing(a, lane, n_route);
}

template <int DT>
void launch_nedf_net(const KArgs& k, hipStream_t s, int v) {
  const dim3 b4(256), b8(512), g1(cu_count()), g2(2 * cu_count());
  if constexpr (DT == 2) {
    switch (v) {
      case 11: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 1, 1, 4>), g1, b4, 0, s, k); return;
      case 12: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 2, 1, 1, 4>), g1, b4, 0, s, k); return;
      case 21: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 2, 1, 4>), g2, b4, 0, s, k); return;
      case 22: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 2, 2, 1, 4>), g2, b4, 0, s, k); return;
      case 1011: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 1, 1, 8>), g1, b8, 0, s, k); return;
      case 1012: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 2, 1, 1, 8>), g1, b8, 0, s, k); return;
      case 1014: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 4, 1, 1, 8>), g1, b8, 0, s, k); return;
      default: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 4, 1, 1, 4>), g1, b4, 0, s, k); return;
    }
  } else if constexpr (DT == 1) {
    switch (v) {
      case 11: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 1, 1, 4>), g1, b4, 0, s, k); return;
      case 21: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 2, 1, 4>), g2, b4, 0, s, k); return;
      case 111: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 1, 2, 4>), g1, b4, 0, s, k); return;
      case 112: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 2, 1, 2, 4>), g1, b4, 0, s, k); return;
      case 1011: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 1, 1, 8>), g1, b8, 0, s, k); return;
      case 1012: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 2, 1, 1, 8>), g1, b8, 0, s, k); return;
      default: hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 2, 1, 1, 4>), g1, b4, 0, s, k); return;
    }
  } else if constexpr (DT == 3) {
    // MX: superchunks of four blocks; eight waves (items of 256 pairs) or four
    if (v >= 1000) hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 4, 1, 1, 8>), g1, b8, 0, s, k);
    else hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 4, 1, 1, 4>), g1, b4, 0, s, k);
  } else {
    hipLaunchKernelGGL((k_nedf<DT, 256, 8, 8, 1, 1, 1, 4>), g1, b4, 0, s, k);
  }
}

}  // namespace

void launch_nedf(const KArgs& k, hipStream_t s, int dtype, int v) {
  if (dtype == NEDF_FP8) launch_nedf_net<2>(k, s, v);
  else if (dtype == NEDF_FP8_MX) launch_nedf_net<3>(k, s, v);
  else if (dtype == NEDF_BF16) launch_nedf_net<1>(k, s, v);
  else launch_nedf_net<0>(k, s, v);
}

}  // namespace nedf
