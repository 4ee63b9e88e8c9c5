// The network stages on the feature-split engine: the intersection network,
// the MLP marcher and the secant refinement of 256-wide, eight-layer
// networks, for BF16 lists that leave the register-resident kernels short of
// work, the network's FP32 lists up to 36 rounds, and every marched or refined
// FP32 list.  One workgroup of eight waves evaluates 32 (or, per pass, 64)
// samples.
//
// BF16: a pass is bound by the 1 MB of weights a compute unit reads from L2
// (about 7 us at 64 bytes a clock); 32 pairs take 9-10 us against 31 us for
// the 256 of a register-resident workgroup, so short lists end sooner and
// long ones do not.  FP32: a pass is bound by the matrix cores in both forms (69
// us for 32 pairs, 261 us for the 128 of a register-resident workgroup of four
// waves): the split form has four times finer items, and per 64 samples, two
// blocks to a weight read, the higher rate too.  Measured, before and after:
// 64 x 64 frame, 8 instances, BF16: march 155 -> 43 us, refinement 157 -> 46
// us, network 31 -> 23 us; 20,011 FP32 rays, 24 instances: network 514 -> 366
// us, march 992 -> 249 us, refinement 1,053 -> 522 us; FP32 marcher, 160 x
// 160, 16 objects, 192 samples: 21.4 -> 20.5 ms.
#include "coop_engine.h"
#include "pipeline.h"
#include "runtime.h"

namespace nedf {
namespace {

// Intersection network: a workgroup takes 32 pairs of one object at a time.
template <int DT>
__global__ __launch_bounds__(coop::THREADS, 1) void k_nedf_small(KArgs a) {
  constexpr int L = 8, KS0 = eng::ks_for_slots<DT>(6 * L + 3);
  __shared__ __attribute__((aligned(16))) uint8_t lds[coop::Lds<DT, 1, 2>::BYTES];
  __shared__ ItemTable s_tab;
  if (!build_items<ROUTE_SMALL>(a, s_tab, 32)) return;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  int n_route[3] = {0, 0, 0};
  for (int item = blockIdx.x; item < s_tab.total; item += gridDim.x) {
    const int obj = item_object(s_tab, a.n_obj, item);
    const int local = (item - s_tab.start[obj]) * 32 + (lane & 31);
    const bool valid = local < s_tab.cnt[obj];
    const uint2 pr = a.pairs[s_tab.off[obj] + (valid ? local : 0)];
    const ObjDesc& od = a.obj[obj];
    const uint8_t* blob = od.nedf_blob;
    const nedf_blob_header* hb = reinterpret_cast<const nedf_blob_header*>(blob);
    const float* hbias = reinterpret_cast<const float*>(blob + uniform_load_u64(&hb->off_head_b));
    const float l = od.bound;
    const W2L g = load_w2l(a.w2l, int(pr.y));
    float o[3], d[3], dlo[3], ol[3], pl[6], pllo[6], tperp;
    make_ray(a.rays, pr.x, o, d, dlo);
    local_line(g, o, d, dlo, pl, pllo, tperp, ol);
    const bool inside = sum_sq(ol[0], ol[1], ol[2]) < l * l;
    float y[1][2];
    coop::network<DT, KS0, 8, 2, 1>(
        hb, blob, lds, [&](int, auto rc) { return coop::encode_read<DT, 6, L>(pl, pllo, half, rc); }, y);
    if (threadIdx.x < 64) {
      const float mu_hat = y[0][0] + uniform_load_f32(hbias);
      const float z = y[0][1] + uniform_load_f32(hbias + 1);
      const float p = sigmoidf_(z);
      const float D = g.s * (tperp - l * fminf(fmaxf(mu_hat, -1.0f), 1.0f));
      route_pairs(a, obj, s_tab.off[obj], pr, valid && half == 0, inside, p, D, lane, n_route);
    }
  }
  if (threadIdx.x < 64) flush_routing(a, lane, n_route);
}

// Marcher: a workgroup takes one pair at a time, 64 samples per pass; with
// TAIL the last 32 or fewer take a pass of their own (FP32, 160 x 160 rays, 16
// objects, 32 samples: 6.3 ms with half of every pass empty, 3.6 without).  An
// instantiation of its own, since its code costs the others 1 %.
template <int DT, bool TAIL>
__global__ __launch_bounds__(coop::THREADS, 1) void k_march_small(KArgs a) {
  constexpr int L = 10, KS0 = eng::ks_for_slots<DT>(3 * L + 2);
  __shared__ __attribute__((aligned(16))) uint8_t lds[coop::Lds<DT, 2, 1>::BYTES];
  __shared__ ItemTable s_tab;
  if (!build_items<ROUTE_SMALL>(a, s_tab, 1)) return;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int N = a.n_samples;
  for (int item = blockIdx.x; item < s_tab.total; item += gridDim.x) {
    const int obj = item_object(s_tab, a.n_obj, item);
    const uint2 pr = a.pairs[s_tab.off[obj] + item - s_tab.start[obj]];
    const ObjDesc& od = a.obj[obj];
    const uint8_t* blob = od.blob;
    const nedf_blob_header* hb = reinterpret_cast<const nedf_blob_header*>(blob);
    const float head_b = uniform_load_f32(blob + uniform_load_u64(&hb->off_head_b));
    const W2L g = load_w2l(a.w2l, int(pr.y));
    float o[3], d[3], ol[3], dl[3];
    make_ray(a.rays, pr.x, o, d);
    to_local(g, o, d, ol, dl);
    float ta = 0.f, tb = 0.f;
    if (a.clip) {
      if (!sphere_chord(ol, dl, od.bound, ta, tb)) continue;  // the workgroup's one pair: uniform
    } else {
      ta = a.t_near * g.inv_s;
      tb = a.t_far * g.inv_s;
    }
    const float delta = (tb - ta) / float(N);
    const float pa[3] = {fmaf(ta, dl[0], ol[0]), fmaf(ta, dl[1], ol[1]), fmaf(ta, dl[2], ol[2])};
    MarchSum sum;
    auto pass = [&](auto nbc, int s0) __attribute__((always_inline)) {
      constexpr int NB = decltype(nbc)::value;
      float tr[NB], p[NB][3];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        tr[nb] = (float(s0 + 32 * nb + (lane & 31)) + 0.5f) * delta;
#pragma unroll
        for (int c = 0; c < 3; ++c) p[nb][c] = fmaf(tr[nb], dl[c], pa[c]);
      }
      const float zero[3] = {0.f, 0.f, 0.f};
      float y[NB][1];
      coop::network<DT, KS0, 8, 1, NB>(
          hb, blob, lds, [&](int nb, auto rc) { return coop::encode_read<DT, 3, L>(p[nb], zero, half, rc); }, y);
      if (threadIdx.x < 64) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          float v = mlp_sigma<true>(od, y[nb][0] + head_b, p[nb][0], p[nb][1], p[nb][2]) * delta;
          if (lane >= 32 || s0 + 32 * nb + (lane & 31) >= N) v = 0.f;
          sum.add(v, ta + tr[nb], lane);
        }
      }
    };
    int s0 = 0;
    for (; N - s0 > (TAIL ? 32 : 0); s0 += 64) pass(std::integral_constant<int, 2>{}, s0);
    if constexpr (TAIL) pass(std::integral_constant<int, 1>{}, s0);
    if (threadIdx.x == 0) sum.emit(a, pr, g.s);
  }
}

// Secant refinement: a workgroup takes 32 pixels of one object at a time; the
// two seeds' evaluations share a pass.
template <int DT>
__global__ __launch_bounds__(coop::THREADS, 1) void k_refine_small(KArgs a) {
  constexpr int L = 10, KS0 = eng::ks_for_slots<DT>(3 * L + 2);
  __shared__ __attribute__((aligned(16))) uint8_t lds[coop::Lds<DT, 2, 1>::BYTES];
  __shared__ ItemTable s_tab;
  if (!build_items<ROUTE_SMALL>(a, s_tab, 32)) return;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  for (int item = blockIdx.x; item < s_tab.total; item += gridDim.x) {
    const int obj = item_object(s_tab, a.n_obj, item);
    const int local = (item - s_tab.start[obj]) * 32 + (lane & 31);
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
    auto eval = [&](auto nbc, const float* t, float* f) __attribute__((always_inline)) {
      constexpr int NB = decltype(nbc)::value;
      float p[NB][3], y[NB][1];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float tl = t[nb] * g.inv_s;
#pragma unroll
        for (int c = 0; c < 3; ++c) p[nb][c] = fmaf(tl, dl[c], ol[c]);
      }
      const float zero[3] = {0.f, 0.f, 0.f};
      coop::network<DT, KS0, 8, 1, NB>(
          hb, blob, lds, [&](int nb, auto rc) { return coop::encode_read<DT, 3, L>(p[nb], zero, half, rc); }, y);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) f[nb] = mlp_surface(od, y[nb][0] + head_b, p[nb][0], p[nb][1], p[nb][2]);
    };
    Secant s;
    s.start<DT == 1>(a.depth[pr.x], a.refine_h, g.s);
    {
      const float t[2] = {s.t0, s.t1};
      float f[2];
      eval(std::integral_constant<int, 2>{}, t, f);
      s.f0 = f[0];
      s.f1 = f[1];
    }
    s.active = s.f0 < 0.0f && s.f1 >= 0.0f;
    for (int it = 0; it < a.refine_steps; ++it) {
      const float tn = s.update();
      if (it + 1 < a.refine_steps) {
        float fn;
        eval(std::integral_constant<int, 1>{}, &tn, &fn);
        s.shift(tn, fn);
      }
    }
    if (valid && threadIdx.x < 32) a.depth[pr.x] = s.out;
  }
}

}  // namespace

void launch_nedf_small(const KArgs& k, hipStream_t s, int dtype, unsigned grid) {
  if (dtype == NEDF_BF16) hipLaunchKernelGGL(k_nedf_small<1>, dim3(grid), dim3(coop::THREADS), 0, s, k);
  else hipLaunchKernelGGL(k_nedf_small<0>, dim3(grid), dim3(coop::THREADS), 0, s, k);
}

void launch_march_small(const KArgs& k, hipStream_t s, int dtype, unsigned grid) {
  const dim3 g(grid), b(coop::THREADS);
  const bool tail = (k.n_samples - 1) % 64 < 32;  // 1 to 32 samples beyond whole passes
  if (dtype == NEDF_BF16) {
    if (tail) hipLaunchKernelGGL((k_march_small<1, true>), g, b, 0, s, k);
    else hipLaunchKernelGGL((k_march_small<1, false>), g, b, 0, s, k);
  } else {
    if (tail) hipLaunchKernelGGL((k_march_small<0, true>), g, b, 0, s, k);
    else hipLaunchKernelGGL((k_march_small<0, false>), g, b, 0, s, k);
  }
}

void launch_refine_small(const KArgs& k, hipStream_t s, int dtype, unsigned grid) {
  if (dtype == NEDF_BF16) hipLaunchKernelGGL(k_refine_small<1>, dim3(grid), dim3(coop::THREADS), 0, s, k);
  else hipLaunchKernelGGL(k_refine_small<0>, dim3(grid), dim3(coop::THREADS), 0, s, k);
}

}  // namespace nedf
