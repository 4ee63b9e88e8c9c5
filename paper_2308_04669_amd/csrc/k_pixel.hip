// Per-pixel stages after the depth buffer: binning hit pixels by object,
// secant refinement of the winning depth, deferred shading (Eq. 8, Alg. 1
// step 2), shadow rays and the shadow multiplier (Alg. 2), composite.
#include <algorithm>
#include <cstring>

#include "pipeline.h"
#include "runtime.h"

namespace nedf {
namespace {

// Start of the shading call: the status word, list R and (for the outliers)
// the counts of list B (its fill counters are the depth call's).
__global__ void k_begin_pixels(KArgs a, int resample) {
  const int t = threadIdx.x;
  constexpr int words = int(sizeof(PairList) / 4);
  if (t == 0) *a.status = 0;
  for (int i = t; i < words; i += blockDim.x) reinterpret_cast<int32_t*>(&a.C->R)[i] = 0;
  if (resample && t < NEDF_MAX_OBJECTS) a.C->B.cnt[t] = 0;
  if (t == 0 && resample) a.C->B.work_counter = a.C->stats[1] = 0;
}

// Pairs of list R: pixels with a valid ID whose object is in `mask`, as
// (pixel, instance), after their counts per object (k_finalize or
// k_clear_rgb): the workgroup counts its own pixels, reserves one range per
// object and writes.  The first workgroup records the segments and the work
// items over item_mask.  Objects outside `mask` keep their counts and get no
// segment.
__global__ __launch_bounds__(256) void k_bin_write(KArgs a, const int32_t* ids, uint32_t mask) {
  __shared__ int s_cnt[NEDF_MAX_OBJECTS], s_base[NEDF_MAX_OBJECTS], s_seg[NEDF_MAX_OBJECTS], s_lim[NEDF_MAX_OBJECTS];
  const int t = threadIdx.x, lane = t & 63;
  const int64_t per = bin_span(a.n_rays, gridDim.x);
  const int64_t p0 = int64_t(blockIdx.x) * per;
  const int64_t p1 = p0 + per < a.n_rays ? p0 + per : a.n_rays;
  PairList* L = &a.C->R;
  if (t < 64) {
    const bool listed = t < a.n_obj && ((mask >> t) & 1u);
    const int64_t c = listed ? L->cnt[t] : 0;
    int64_t total;
    const int64_t off = wave_prefix(c, t, total);
    const int64_t o0 = min(off, a.capacity), lim = min(off + c, a.capacity) - o0;
    if (t < NEDF_MAX_OBJECTS) {
      s_seg[t] = int(o0);
      s_lim[t] = int(lim);
      s_cnt[t] = 0;
    }
    if (blockIdx.x == 0) {
      const bool counted = t < a.n_obj && ((a.item_mask >> t) & 1u);
      int items, pairs;
      wave_prefix(counted ? int((lim + a.item_pairs - 1) / a.item_pairs) : 0, t, items);
      wave_prefix(counted ? int(lim) : 0, t, pairs);
      if (t <= a.n_obj) L->off[t] = int(o0);
      if (listed) L->cnt[t] = int(lim);
      if (t == 0) {
        a.C->last_pairs = pairs;
        a.C->last_items = items;
        if (total > a.capacity) set_status(a.status, NEDF_ERR_CAPACITY);
      }
    }
  }
  __syncthreads();
  for (int64_t pb = p0; pb < p1; pb += 256) {
    const int64_t p = pb + t;
    bin_groups(a, p < p1 ? ids[p] : -1, mask, lane, [&](int o, uint64_t match, bool) {
      if (lane == __ffsll((unsigned long long)match) - 1) atomicAdd(&s_cnt[o], __popcll(match));
    });
  }
  __syncthreads();
  if (t < a.n_obj) {
    s_base[t] = s_cnt[t] ? atomicAdd(&L->fill[t], s_cnt[t]) : 0;
    s_cnt[t] = 0;
  }
  __syncthreads();
  for (int64_t pb = p0; pb < p1; pb += 256) {
    const int64_t p = pb + t;
    const int inst = p < p1 ? ids[p] : -1;
    bin_groups(a, inst, mask, lane, [&](int o, uint64_t match, bool mine) {
      const int leader = __ffsll((unsigned long long)match) - 1;
      int off = 0;
      if (lane == leader) off = atomicAdd(&s_cnt[o], __popcll(match));
      off = __shfl(off, leader);
      const int pos = s_base[o] + off + __popcll(match & ((1ull << lane) - 1ull));
      if (mine && pos < s_lim[o]) a.pairs[s_seg[o] + pos] = make_uint2(uint32_t(p), uint32_t(inst));
    });
  }
}

__global__ void k_refine_analytic(KArgs a, uint32_t mask) {
  const PairList* L = &a.C->R;
  for (int m = 0; m < a.n_obj; ++m) {
    if (!((mask >> m) & 1u)) continue;
    const ObjDesc od = a.obj[m];
    const int cnt = L->cnt[m], off = L->off[m];
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < cnt; q += gridDim.x * blockDim.x) {
      const uint2 pr = a.pairs[off + q];
      const W2L g = load_w2l(a.w2l, int(pr.y));
      float o[3], d[3], ol[3], dl[3];
      make_ray(a.rays, pr.x, o, d);
      to_local(g, o, d, ol, dl);
      auto f = [&](float t) {
        const float tl = t * g.inv_s;
        const float x = fmaf(tl, dl[0], ol[0]), y = fmaf(tl, dl[1], ol[1]), z = fmaf(tl, dl[2], ol[2]);
        return (od.param[1] - sqrtf(x * x + y * y + z * z)) / od.param[2];
      };
      Secant s;
      s.start(a.depth[pr.x], a.refine_h, g.s);
      s.f0 = f(s.t0);
      s.f1 = f(s.t1);
      s.active = s.f0 < 0.0f && s.f1 >= 0.0f;
      for (int it = 0; it < a.refine_steps; ++it) {
        const float tn = s.update();
        if (it + 1 < a.refine_steps) s.shift(tn, f(tn));
      }
      a.depth[pr.x] = s.out;
    }
  }
}

// Density-network refinement: items of 128 pixels (32 per wave) of one
// SDF-mode object; each evaluation of f is one pass of the trunk.
template <int DT, int WIDTH, int NHID, int L, int SBX, int OCC, int NW>
__global__ __launch_bounds__(64 * NW, OCC) void k_refine_mlp(KArgs a) {
  using T = eng::Tr<DT>;
  constexpr int NB = T::NB;
  constexpr int KS0 = eng::ks_for_slots<DT>(3 * L + 2);
  constexpr int KSH = WIDTH / T::KPS;
  constexpr int CHUNK = eng::cmax(eng::chunk_bytes<DT>(KS0, 0), eng::chunk_bytes<DT>(KSH, 1));
  __shared__ __attribute__((aligned(16))) uint8_t lds[eng::NBUF * eng::slot_bytes(CHUNK, SBX)];
  __shared__ int s_item;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  __shared__ ItemTable s_tab;
  if (!build_items(a, s_tab, 32 * NW)) return;
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.lwork, 1);
    __syncthreads();
    const int item = s_item;
    __syncthreads();
    if (item >= s_tab.total) break;
    const int obj = item_object(s_tab, a.n_obj, item);
    const int local = (item - s_tab.start[obj]) * (32 * NW) + wave * 32 + (lane & 31);
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
    // the item's field evaluations run back to back on one blob: each pass
    // but the last prefetches the next pass's first chunks
    const int n_eval = 2 + (a.refine_steps > 1 ? a.refine_steps - 1 : 0);
    int eval_i = 0, slot = 0;
    bool primed = false;
    auto f = [&](float t) {
      const float tl = t * g.inv_s;
      float p[3] = {fmaf(tl, dl[0], ol[0]), fmaf(tl, dl[1], ol[1]), fmaf(tl, dl[2], ol[2])};
      typename T::frag Benc[NB][KS0];
      eng::encode_input<DT, 3, L, KS0>(p, half, Benc[0]);
      float partial[NB][1] = {{0.f}};
      typename T::frag Blast[NB][KSH];
      const uint8_t* nb_ = ++eval_i < n_eval ? blob : nullptr;
      eng::trunk<DT, WIDTH, KS0, NHID, 1, CHUNK, false, 0, WIDTH / 32, SBX, NB, NW>(hb, blob, Benc, lds, partial,
                                                                                   Blast, nullptr, &slot, nb_, primed);
      primed = nb_ != nullptr;
      const float u = partial[0][0] + __shfl_xor(partial[0][0], 32) + head_b;
      return mlp_surface(od, u, p[0], p[1], p[2]);
    };
    Secant s;
    s.start<DT == 1>(a.depth[pr.x], a.refine_h, g.s);
    s.f0 = f(s.t0);
    s.f1 = f(s.t1);
    s.active = s.f0 < 0.0f && s.f1 >= 0.0f;
    for (int it = 0; it < a.refine_steps; ++it) {
      const float tn = s.update();
      if (it + 1 < a.refine_steps) {
        const float fn = f(tn);
        s.shift(tn, fn);
      }
    }
    if (valid && half == 0) a.depth[pr.x] = s.out;
  }
}

// ---- deferred shading ---------------------------------------------------------
// Clear colour (or an analytic object's own colour) of every pixel; with BIN
// the hit pixels per object of `mask` are counted for k_bin_write.
template <bool BIN>
__global__ __launch_bounds__(256) void k_clear_rgb(KArgs a, const int32_t* ids, uint32_t mask) {
  __shared__ int s_cnt[NEDF_MAX_OBJECTS];
  const int t = threadIdx.x, lane = t & 63;
  if (BIN && t < NEDF_MAX_OBJECTS) s_cnt[t] = 0;
  if (BIN) __syncthreads();
  const int64_t per = bin_span(a.n_rays, gridDim.x);
  const int64_t p0 = int64_t(blockIdx.x) * per;
  const int64_t p1 = p0 + per < a.n_rays ? p0 + per : a.n_rays;
  for (int64_t pb = p0; pb < p1; pb += 256) {
    const int64_t p = pb + t;
    const int inst = p < p1 ? ids[p] : -1;
    if (p < p1) {
      float c[3] = {a.clear_rgb[0], a.clear_rgb[1], a.clear_rgb[2]};
      if (inst >= 0 && inst < a.n_inst) {
        const ObjDesc& od = a.obj[a.inst_object[inst]];
        if (od.field != NEDF_FIELD_MLP) { c[0] = od.param[3]; c[1] = od.param[4]; c[2] = od.param[5]; }
      }
      a.rgb[3 * p + 0] = c[0];
      a.rgb[3 * p + 1] = c[1];
      a.rgb[3 * p + 2] = c[2];
    }
    if constexpr (BIN) bin_groups(a, inst, mask, lane, [&](int o, uint64_t match, bool) {
      if (lane == __ffsll((unsigned long long)match) - 1) atomicAdd(&s_cnt[o], __popcll(match));
    });
  }
  if constexpr (BIN) {
    __syncthreads();
    if (t < a.n_obj && s_cnt[t]) atomicAdd(&a.C->R.cnt[t], s_cnt[t]);
  }
}

// NeRF shading: a wave shades 32 / K pixels with K samples each; trunk with
// the sigma head, then the colour layer on [h_last, gamma_dirL(d)], then
// local compositing across each pixel's K lanes.
template <int DT, int WIDTH, int NHID, int L, int DIRL, int RGBW, int SBX, int OCC, int NW>
__global__ __launch_bounds__(64 * NW, OCC) void k_shade(KArgs a) {
  using T = eng::Tr<DT>;
  constexpr int NB = T::NB;
  constexpr int KS0 = eng::ks_for_slots<DT>(3 * L + 2);
  constexpr int KSH = WIDTH / T::KPS;
  constexpr int KSD = eng::ks_for_slots<DT>(3 * DIRL + 2);
  constexpr int KSR = KSH + KSD;
  constexpr int CBR = eng::chunk_bytes<DT>(KSR, 3);
  constexpr int CHUNK = eng::cmax(eng::cmax(eng::chunk_bytes<DT>(KS0, 0), eng::chunk_bytes<DT>(KSH, 1)), CBR);
  __shared__ __attribute__((aligned(16))) uint8_t lds[eng::NBUF * eng::slot_bytes(CHUNK, SBX)];
  __shared__ int s_item;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
  const int K = a.shade_K;  // 1, 2, 4, 8, 16 or 32
  const int ppw = 32 / K;
  const int slot = lane & 31, q = slot / K, j = slot % K;
  // first pass: the binned pixels (list R), outliers pushed to the same
  // segments of list B; second pass (chord mode): list B
  const bool chord = a.shade_chord != 0;
  const uint2* prs_list = chord ? a.pairsB : a.pairs;
  PairList* RS = &a.C->B;
  __shared__ ItemTable s_tab;
  build_items(a, s_tab, ppw * NW);
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.lwork, 1);
    __syncthreads();
    const int item = s_item;
    __syncthreads();
    if (item >= s_tab.total) break;
    const int obj = item_object(s_tab, a.n_obj, item);
    const int local = (item - s_tab.start[obj]) * (ppw * NW) + wave * ppw + q;
    const bool valid = local < s_tab.cnt[obj];
    const uint2 pr = prs_list[s_tab.off[obj] + (valid ? local : 0)];
    const ObjDesc& od = a.obj[obj];
    const uint8_t* blob = od.blob;
    const nedf_blob_header* hb = reinterpret_cast<const nedf_blob_header*>(blob);
    const float head_b = uniform_load_f32(blob + uniform_load_u64(&hb->off_head_b));
    const float* rgb_bp = reinterpret_cast<const float*>(blob + uniform_load_u64(&hb->off_rgbh_b));
    const float rgb_b[3] = {uniform_load_f32(rgb_bp), uniform_load_f32(rgb_bp + 1), uniform_load_f32(rgb_bp + 2)};
    const W2L g = load_w2l(a.w2l, int(pr.y));
    float o[3], d[3], ol[3], dl[3];
    make_ray(a.rays, pr.x, o, d);
    to_local(g, o, d, ol, dl);
    // sample window in world units: [D - h, D + h], or (chord mode) the
    // chord of the bounding sphere
    float t_lo, step;
    {
      float ca = 0.0f, cb = 0.0f;
      if (chord && sphere_chord(ol, dl, od.bound, ca, cb)) {
        t_lo = g.s * ca;
        step = g.s * (cb - ca) / float(K);
      } else {
        const float D = a.depth[pr.x];
        t_lo = D - a.shade_h;
        step = 2.0f * a.shade_h / float(K);
      }
    }
    const float t = t_lo + (float(j) + 0.5f) * step;
    const float tl = t * g.inv_s;
    float p[3] = {fmaf(tl, dl[0], ol[0]), fmaf(tl, dl[1], ol[1]), fmaf(tl, dl[2], ol[2])};
    typename T::frag Benc[NB][KS0];
    eng::encode_input<DT, 3, L, KS0>(p, half, Benc[0]);
    float partial[NB][1] = {{0.f}};
    typename T::frag Blast[NB][KSH];
    int cur = 0;
    eng::trunk<DT, WIDTH, KS0, NHID, 1, CHUNK, true, CBR, RGBW / 32, SBX, NB, NW>(
        hb, blob, Benc, lds, partial, Blast, blob + uniform_load_u64(&hb->off_rgb), &cur);
    const float u = partial[0][0] + __shfl_xor(partial[0][0], 32) + head_b;
    const float sig = mlp_sigma(od, u, p[0], p[1], p[2]);
    // colour layer input: [h_last, gamma_dirL(d_l)]
    typename T::frag Bc[NB][KSR];
#pragma unroll
    for (int k = 0; k < KSH; ++k) Bc[0][k] = Blast[0][k];
    {
      typename T::frag Bd[KSD];
      eng::encode_input<DT, 3, DIRL, KSD>(dl, half, Bd);
#pragma unroll
      for (int k = 0; k < KSD; ++k) Bc[0][KSH + k] = Bd[k];
    }
    float prgb[NB][3] = {{0.f, 0.f, 0.f}};
    typename T::frag dummy[NB][1];
    eng::layer<DT, NB, KSR, RGBW / 32, CBR, 0, 1, 3, 1, CHUNK, RGBW / 32, SBX, NW>(
        Bc, dummy, blob + uniform_load_u64(&hb->off_rgb), nullptr, lds, cur, prgb);
    float c[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) c[ch] = sigmoidf_(prgb[0][ch] + __shfl_xor(prgb[0][ch], 32) + rgb_b[ch]);
    // local compositing over the K lanes of this pixel
    const float v = sig * (step * g.inv_s);
    float incl = v;
    for (int off = 1; off < K; off <<= 1) {
      const float y = __shfl_up(incl, off);
      if (j >= off) incl += y;
    }
    const float w = expf(-(incl - v)) * one_minus_exp_neg(v);
    float sw = w, sc0 = w * c[0], sc1 = w * c[1], sc2 = w * c[2];
    for (int off = 1; off < K; off <<= 1) {
      sw += __shfl_xor(sw, off);
      sc0 += __shfl_xor(sc0, off);
      sc1 += __shfl_xor(sc1, off);
      sc2 += __shfl_xor(sc2, off);
    }
    const int near = (K - 1) / 2;
    const int src = (lane & ~(K - 1)) + near;
    const float n0 = __shfl(c[0], src), n1 = __shfl(c[1], src), n2 = __shfl(c[2], src);
    if (!chord && a.rs_sigma > 0.0f) {
      // outlier (Sec. "Deferred Shading"): density below the threshold at
      // every sample of the pixel; pushed to the object's segment of list B
      float smax = sig;
      for (int off = 1; off < K; off <<= 1) smax = fmaxf(smax, __shfl_xor(smax, off));
      const bool outlier = valid && half == 0 && j == 0 && smax < a.rs_sigma;
      const uint64_t m = __ballot(outlier);
      if (m) {
        const int leader = __ffsll((unsigned long long)m) - 1;
        int base = 0;
        if (lane == leader) {
          base = atomicAdd(&RS->cnt[obj], __popcll(m));
          atomicAdd(&a.C->stats[1], __popcll(m));
        }
        base = __shfl(base, leader);
        if (outlier) a.pairsB[s_tab.off[obj] + base + __popcll(m & ((1ull << lane) - 1ull))] = pr;
      }
    }
    if (valid && half == 0 && j == 0) {
      float* out = a.rgb + 3 * size_t(pr.x);
      if (sw < 1e-6f) {
        out[0] = n0; out[1] = n1; out[2] = n2;
      } else {
        out[0] = sc0 / sw; out[1] = sc1 / sw; out[2] = sc2 / sw;
      }
    }
  }
}

// ---- shadows --------------------------------------------------------------------
// Shadow ray of pixel p for light Lm: origin Lm, direction towards
// x = o + D d; pixels without an ID get a NaN ray (culled everywhere).
// Shadow rays of one light (Alg. 2) for the hit pixels: from a point light
// at (lx, ly, lz) towards x = o + D d, or (dir_dist > 0) for a directional
// light of unit direction of travel (lx, ly, lz), from x - dir_dist l along
// l (parallel, orthographic rays); dist gets the distance from the origin to
// x.  Pixels without a hit get a NaN direction (culled as no candidate).
__global__ void k_shadow_rays(KArgs a, const int32_t* ids, float lx, float ly, float lz, float dir_dist, float* so,
                              float* sd, float* dist) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= a.n_rays) return;
  float o[3], d[3];
  make_ray(a.rays, p, o, d);
  const float D = a.depth[p];
  const bool hit = ids[p] >= 0;
  const float nan = __int_as_float(0x7fc00000);
  const float px = fmaf(D, d[0], o[0]), py = fmaf(D, d[1], o[1]), pz = fmaf(D, d[2], o[2]);
  if (dir_dist > 0.0f) {
    so[3 * p + 0] = fmaf(-dir_dist, lx, px);
    so[3 * p + 1] = fmaf(-dir_dist, ly, py);
    so[3 * p + 2] = fmaf(-dir_dist, lz, pz);
    sd[3 * p + 0] = hit ? lx : nan; sd[3 * p + 1] = hit ? ly : nan; sd[3 * p + 2] = hit ? lz : nan;
    dist[p] = hit ? dir_dist : 0.f;
    return;
  }
  const float x = px - lx, y = py - ly, z = pz - lz;
  const float r = sqrtf(x * x + y * y + z * z);
  const float inv = hit && r > 0.f ? 1.0f / r : nan;
  so[3 * p + 0] = lx; so[3 * p + 1] = ly; so[3 * p + 2] = lz;
  sd[3 * p + 0] = x * inv; sd[3 * p + 1] = y * inv; sd[3 * p + 2] = z * inv;
  dist[p] = hit ? r : 0.f;
}

__global__ void k_shadow_init(KArgs a, float* shadow) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p < a.n_rays) shadow[p] = 1.0f;
}

// Occlusion test of Alg. 2 for one light: D_L + eps < |L - x| multiplies by beta.
__global__ void k_shadow_apply(KArgs a, const int32_t* ids, const float* depth_l, const float* dist, float eps,
                               float beta, float* shadow) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= a.n_rays || ids[p] < 0) return;
  if (depth_l[p] + eps < dist[p]) shadow[p] *= beta;
}

__global__ void k_composite(KArgs a, const float* shadow, float* rgb) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= a.n_rays) return;
  const float f = shadow[p];
  rgb[3 * p + 0] *= f;
  rgb[3 * p + 1] *= f;
  rgb[3 * p + 2] *= f;
}

unsigned grid_n(int64_t n) {
  const int64_t g = (n + 255) / 256;
  return unsigned(g > 0 ? g : 1);
}

}  // namespace

void stage_bin_write(const KArgs& k0, hipStream_t s, const int32_t* ids, uint32_t mask, uint32_t item_mask, int per) {
  KArgs k = k0;
  k.item_mask = item_mask;
  k.item_pairs = per;
  hipLaunchKernelGGL(k_bin_write, dim3(bin_blocks(k.n_rays)), dim3(256), 0, s, k, ids, mask);
}

void stage_refine(const KArgs& k0, hipStream_t s, const int32_t* ids, uint32_t mlp_mask, uint32_t sphere_mask,
                  int dtype) {
  prof_mark("infer.refine", s, true);
  KArgs k = k0;
  k.lcnt = k.C->R.cnt;
  k.loff = k.C->R.off;
  k.lwork = &k.C->R.work_counter;
  k.item_mask = mlp_mask;
  // long BF16 lists: one workgroup of 8 waves per CU, which streams each
  // weight chunk into LDS once for 256 samples (two workgroups of 4 waves
  // stream it twice; the refinement is bound by that L2 -> LDS stream, and the
  // 8-wave form measured 8 % faster on the 1080p frame)
  const int nw = dtype == NEDF_BF16 ? 8 : 4;
  // both kinds in one binning, unless the list may not hold the pixels of both
  // (a composition's workspace may be as small as one kind needs); the
  // counters report the networks' items
  const int per = mlp_mask ? 32 * nw : 1;
  if (mlp_mask && sphere_mask && k.capacity < k.n_rays) {
    stage_bin_write(k, s, ids, sphere_mask, sphere_mask, 1);
    hipLaunchKernelGGL(k_refine_analytic, dim3(256), dim3(256), 0, s, k, sphere_mask);
    stage_bin_write(k, s, ids, mlp_mask, mlp_mask, per);
  } else {
    stage_bin_write(k, s, ids, mlp_mask | sphere_mask, mlp_mask ? mlp_mask : sphere_mask, per);
    if (sphere_mask) hipLaunchKernelGGL(k_refine_analytic, dim3(256), dim3(256), 0, s, k, sphere_mask);
  }
  if (mlp_mask) {
    Kernels kn{true, false};
    if (dtype == NEDF_BF16) kn = choose_kernels(k, 32, 3 * cu_count(), std::min<int64_t>(k.capacity, k.n_rays));
    if (kn.small) launch_refine_small(k, s, dtype, cu_count());
    if (kn.large)
      hipLaunchKernelGGL((k_refine_mlp<1, 256, 8, 10, 2, 1, 8>), dim3(cu_count()), dim3(512), 0, s, k);
  }
  prof_mark("infer.refine", s, false);
}

namespace {
void launch_shade(const KArgs& k, hipStream_t s, int dtype) {
  if (dtype == NEDF_BF16)
    hipLaunchKernelGGL((k_shade<1, 256, 8, 10, 4, 128, 2, 1, 8>), dim3(cu_count()), dim3(512), 0, s, k);
  else
    hipLaunchKernelGGL((k_shade<0, 256, 8, 10, 4, 128, eng::sb_default<0>(), 1, 4>), dim3(cu_count()), dim3(256),
                       0, s, k);
}
}  // namespace

void stage_shade(const KArgs& k0, hipStream_t s, const int32_t* ids, uint32_t nerf_mask, int dtype, int rs_samples) {
  prof_mark("shade", s, true);
  KArgs k = k0;
  const dim3 g(bin_blocks(k.n_rays));
  // list R takes the hit pixels; list B the outliers of the first pass in
  // the segments of list R (an object's outliers are a subset of its pixels)
  hipLaunchKernelGGL(k_begin_pixels, dim3(1), dim3(64), 0, s, k, nerf_mask && rs_samples > 0 ? 1 : 0);
  if (nerf_mask) hipLaunchKernelGGL(k_clear_rgb<true>, g, dim3(256), 0, s, k, ids, nerf_mask);
  else hipLaunchKernelGGL(k_clear_rgb<false>, g, dim3(256), 0, s, k, ids, nerf_mask);
  if (nerf_mask) {
    // BF16: one workgroup of 8 waves per CU sharing each weight copy; FP32: 4 waves
    const int nw = dtype == NEDF_BF16 ? 8 : 4;
    stage_bin_write(k, s, ids, nerf_mask, nerf_mask, (32 / k.shade_K) * nw);
    k.item_mask = nerf_mask;
    k.loff = k.C->R.off;
    k.lcnt = k.C->R.cnt;
    k.lwork = &k.C->R.work_counter;
    KArgs k1 = k;
    k1.shade_chord = 0;
    if (rs_samples <= 0) k1.rs_sigma = 0.0f;
    launch_shade(k1, s, dtype);
    if (rs_samples > 0) {
      // second pass: the outliers, volume-rendered over the bounding chord
      prof_mark("shade.resample", s, true);
      KArgs k2 = k;
      k2.shade_chord = 1;
      k2.shade_K = rs_samples;
      k2.lcnt = k.C->B.cnt;
      k2.lwork = &k.C->B.work_counter;
      launch_shade(k2, s, dtype);
      prof_mark("shade.resample", s, false);
    }
  }
  prof_mark("shade", s, false);
}

void stage_shadow_rays(const KArgs& k, hipStream_t s, const int32_t* ids, const float L[3], float dir_dist, float* so,
                       float* sd, float* dist) {
  hipLaunchKernelGGL(k_shadow_rays, dim3(grid_n(k.n_rays)), dim3(256), 0, s, k, ids, L[0], L[1], L[2], dir_dist, so,
                     sd, dist);
}

void stage_shadow_init(const KArgs& k, hipStream_t s, float* shadow) {
  hipLaunchKernelGGL(k_shadow_init, dim3(grid_n(k.n_rays)), dim3(256), 0, s, k, shadow);
}

void stage_shadow_apply(const KArgs& k, hipStream_t s, const int32_t* ids, const float* depth_l, const float* dist,
                        float eps, float beta, float* shadow) {
  hipLaunchKernelGGL(k_shadow_apply, dim3(grid_n(k.n_rays)), dim3(256), 0, s, k, ids, depth_l, dist, eps, beta,
                     shadow);
}

void stage_composite(const KArgs& k, hipStream_t s, const float* shadow, float* rgb) {
  hipLaunchKernelGGL(k_composite, dim3(grid_n(k.n_rays)), dim3(256), 0, s, k, shadow, rgb);
}

}  // namespace nedf
