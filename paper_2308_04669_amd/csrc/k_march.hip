// The plain volume-rendering marcher (Eq. 5) on MLP density fields (short BF16
// lists and most FP32 lists of 256-wide networks run on the feature-split
// kernel).
#include "pipeline.h"
#include "runtime.h"

namespace nedf {
namespace {

// Matrix-core marcher: a workgroup takes items of NW pairs (one per wave) of
// one object of the list; each wave marches its pair in chunks of 32 NB
// samples through the register-resident density network (NB blocks of 32
// share every weight read from LDS), then scans each block's optical depths
// across the wave in sample order, so that the sums are the same for any NB.
template <int DT, int WIDTH, int NHID, int L, int SBX, int OCC, int NB, int NW>
__global__ __launch_bounds__(64 * NW, OCC) void k_march_mlp(KArgs a) {
  using T = eng::Tr<DT>;
  constexpr int KS0 = eng::ks_for_slots<DT>(3 * L + 2);
  constexpr int KSH = WIDTH / T::KPS;
  constexpr int CHUNK = eng::cmax(eng::chunk_bytes<DT>(KS0, 0), eng::chunk_bytes<DT>(KSH, 1));
  constexpr int SPC = 32 * NB;  // samples per wave per chunk
  __shared__ __attribute__((aligned(16))) uint8_t lds[eng::NBUF * eng::slot_bytes(CHUNK, SBX)];
  __shared__ int s_item;
  __shared__ ItemTable s_tab;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const int N = a.n_samples;
  const int n_chunks = (N + SPC - 1) / SPC;
  if (!build_items(a, s_tab, NW)) return;
  const int total = s_tab.total;
  // one item of lookahead: the next item is claimed during the current
  // item's last pass so that its weights stream in behind this one's
  if (threadIdx.x == 0) s_item = atomicAdd(a.lwork, 1);
  __syncthreads();
  int item = s_item;
  int slot = 0;
  bool primed = false;
  while (item < total) {
    const int obj = item_object(s_tab, a.n_obj, item);
    const int local = (item - s_tab.start[obj]) * NW + wave;
    const bool valid = local < s_tab.cnt[obj];
    const uint2 pr = a.pairs[s_tab.off[obj] + (valid ? local : 0)];
    const ObjDesc& od = a.obj[obj];
    const uint8_t* blob = od.blob;
    const nedf_blob_header* hb = reinterpret_cast<const nedf_blob_header*>(blob);
    const float head_b = uniform_load_f32(blob + uniform_load_u64(&hb->off_head_b));
    const W2L g = load_w2l(a.w2l, int(pr.y));
    float o[3], d[3], ol[3], dl[3];
    make_ray(a.rays, pr.x, o, d);
    to_local(g, o, d, ol, dl);
    float ta = 0.f, tb = 0.f;
    bool seg = true;
    if (a.clip) {
      seg = sphere_chord(ol, dl, od.bound, ta, tb);
      if (!seg) { ta = 0.f; tb = 0.f; }
    } else {
      ta = a.t_near * g.inv_s;
      tb = a.t_far * g.inv_s;
    }
    const float delta = (tb - ta) / float(N);
    const float pa[3] = {fmaf(ta, dl[0], ol[0]), fmaf(ta, dl[1], ol[1]), fmaf(ta, dl[2], ol[2])};
    MarchSum sum;
    int next = total;
    for (int c = 0; c < n_chunks; ++c) {
      const bool last = c + 1 == n_chunks;
      if (last) {
        __syncthreads();  // every wave has read s_item
        if (threadIdx.x == 0) s_item = atomicAdd(a.lwork, 1);
        __syncthreads();
        next = s_item;
      }
      const uint8_t* next_blob = !last ? blob : (next < total ? a.obj[item_object(s_tab, a.n_obj, next)].blob : nullptr);
      typename T::frag Benc[NB][KS0];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float tr = (float(c * SPC + 32 * nb + (lane & 31)) + 0.5f) * delta;
        float p[3] = {fmaf(tr, dl[0], pa[0]), fmaf(tr, dl[1], pa[1]), fmaf(tr, dl[2], pa[2])};
        eng::encode_input<DT, 3, L, KS0>(p, half, Benc[nb]);
      }
      float partial[NB][1];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) partial[nb][0] = 0.f;
      typename T::frag Blast[NB][KSH];
      eng::trunk<DT, WIDTH, KS0, NHID, 1, CHUNK, false, 0, WIDTH / 32, SBX, NB, NW>(hb, blob, Benc, lds, partial,
                                                                               Blast, nullptr, &slot, next_blob,
                                                                               primed);
      primed = next_blob != nullptr;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int si = c * SPC + 32 * nb + (lane & 31);
        const float tr = (float(si) + 0.5f) * delta;
        const float p[3] = {fmaf(tr, dl[0], pa[0]), fmaf(tr, dl[1], pa[1]), fmaf(tr, dl[2], pa[2])};
        const float u = partial[nb][0] + __shfl_xor(partial[nb][0], 32) + head_b;
        float v = mlp_sigma<true>(od, u, p[0], p[1], p[2]) * delta;
        if (lane >= 32 || si >= N || !seg) v = 0.f;
        sum.add(v, ta + tr, lane);
      }
    }
    if (lane == 0 && valid && seg) sum.emit(a, pr, g.s);
    item = next;
  }
}

template <int DT, int WIDTH, int NHID, int L>
void launch_march_mlp(const KArgs& k, hipStream_t s) {
  const dim3 b4(256), b8(512), g1(cu_count()), g2(2 * cu_count());
  if constexpr (DT == 1 && WIDTH == 256) {
    switch (tune_value(NEDF_TUNE_MARCH, DT)) {
      case 11: hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, 1, 1, 1, 4>), g1, b4, 0, s, k); return;
      case 21: hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, 1, 2, 1, 4>), g2, b4, 0, s, k); return;
      case 111: hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, 1, 1, 2, 4>), g1, b4, 0, s, k); return;
      case 112: hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, 2, 1, 2, 4>), g1, b4, 0, s, k); return;
      case 1011: hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, 1, 1, 1, 8>), g1, b8, 0, s, k); return;
      case 1012: hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, 2, 1, 1, 8>), g1, b8, 0, s, k); return;
      default: break;
    }
  }
  hipLaunchKernelGGL((k_march_mlp<DT, WIDTH, NHID, L, eng::sb_default<DT>(), 1, 1, 4>), g1, b4, 0, s, k);
}

}  // namespace

int march_waves(int dtype, int width) {
  if (dtype != NEDF_BF16 || width != 256) return 4;
  return tune_waves(tune_value(NEDF_TUNE_MARCH, dtype));
}

void launch_march(const KArgs& k, hipStream_t s, int dtype, int W) {
  if (dtype == NEDF_BF16) {
    if (W == 256) launch_march_mlp<1, 256, 8, 10>(k, s);
    else launch_march_mlp<1, 64, 3, 6>(k, s);
  } else {
    if (W == 256) launch_march_mlp<0, 256, 8, 10>(k, s);
    else launch_march_mlp<0, 64, 3, 6>(k, s);
  }
}

}  // namespace nedf
