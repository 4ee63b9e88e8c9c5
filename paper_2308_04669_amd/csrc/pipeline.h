// Shared device-side state of the depth / shading / shadow pipeline: pair
// lists in the workspace, kernel arguments and small epilogue helpers.
#pragma once
#include "device_common.h"
#include "launch.h"
#include "mlp_engine.h"

namespace nedf {

// Kernel arguments shared by the stages (passed by value).
struct KArgs {
  RaySrc rays;
  int64_t n_rays;
  int32_t n_obj, n_inst;
  ObjDesc obj[NEDF_MAX_OBJECTS];
  const int32_t* inst_object;
  const float* w2l;
  // instance index written into the depth keys (null: the scene's own
  // index); lets keys of a subset of a scene carry the full scene's indices
  const int32_t* inst_gid;
  int32_t n_samples, clip;
  float t_near, t_far, hit_thr;
  uint32_t item_mask;    // objects whose pairs the matrix-core stage takes
  int32_t item_pairs;    // pairs per work item of that stage
  int* status;
  WsCounters* C;
  // list the current stage reads: counts and segment offsets per object, the
  // counter its work items are claimed from, and its pair array
  const int32_t* lcnt;
  const int32_t* loff;
  int32_t* lwork;
  uint2* pairs;
  int32_t split_per, split_max;  // choice between a stage's two kernels (build_items)
  uint2* pairsB;         // fallback list
  uint2* pairsS;         // depth-slab list of the network stage
  float* pair_dm;        // per pair of list A: lowest depth it can report (world units)
  uint8_t* pair_slab;    // per pair of list A: its depth slab (network stage)
  uint32_t* slab_mask;   // per SLAB_BLOCK pairs of list A: bit s set if slab s occurs
  // shadow-ray queries: only whether some hit lies closer than
  // ray_tmax[ray] - tmax_eps matters (null for depth queries)
  const float* ray_tmax;
  float tmax_eps;
  // ray arrays laid out as an image of this width (shadow rays, one per
  // pixel): culled in 16 x 16 tiles; 0 for unstructured arrays
  int32_t ray_grid_w;
  int64_t capacity;
  uint64_t* keys;
  uint32_t* opac;
  float* depth;
  int32_t* id;
  float* opacity;
  // NeDF inference
  float p_lo, p_hi;
  // refinement / shading / shadow
  float refine_h;
  int32_t refine_steps;
  int32_t shade_K;
  float shade_h;
  float rs_sigma;       // outlier threshold of deferred shading (0: off)
  int32_t shade_chord;  // second pass: samples over the bounding chord of list B's pixels
  float clear_rgb[3];
  float* rgb;
};

// Depth beyond which a pair of `ray` can no longer change the result: the
// pixel's nearest hit so far; for shadow queries the occlusion distance, or
// -inf once the ray is already known to be occluded.
__device__ __forceinline__ float depth_limit(const KArgs& a, uint32_t ray) {
  const float best = __uint_as_float(uint32_t(a.keys[ray] >> 32));
  if (!a.ray_tmax) return best;
  const float cut = a.ray_tmax[ray] - a.tmax_eps;
  return best < cut ? -INFINITY : cut;
}

__device__ __forceinline__ void neu_add(float& s, float& c, float x) {
  const float t = s + x;
  c += fabsf(s) >= fabsf(x) ? (s - t) + x : (x - t) + s;
  s = t;
}

__device__ __forceinline__ float analytic_sigma(const ObjDesc& od, float x, float y, float z) {
  if (od.field == NEDF_FIELD_SPHERE) {
    const float r = sqrtf(x * x + y * y + z * z);
    return od.param[0] * sigmoidf_((od.param[1] - r) / od.param[2]);
  }
  return (z >= od.param[1] && z <= od.param[2]) ? od.param[0] : 0.0f;
}

// Density of an MLP field from the raw head output u at local point x (MARCH:
// as a marcher's sample, see sdf_shape).
template <bool MARCH = false>
__device__ __forceinline__ float mlp_sigma(const ObjDesc& od, float u, float x, float y, float z) {
  if (od.sigma_mode == NEDF_SIGMA_SDF)
    return od.param[0] * sigmoidf_(u - sdf_shape<MARCH>(int(od.param[2]), x, y, z) / od.param[1]);
  const float s = softplusf_(u);
  if (od.sigma_mode == NEDF_SIGMA_SOFTPLUS_MASKED)
    return sum_sq(x, y, z) <= od.bound * od.bound ? s : 0.0f;
  return s;
}

// Surface function (logit of sigma / sigma_max) of an SDF-mode MLP field.
__device__ __forceinline__ float mlp_surface(const ObjDesc& od, float u, float x, float y, float z) {
  return u - sdf_shape(int(od.param[2]), x, y, z) / od.param[1];
}

__device__ __forceinline__ void emit_key(const KArgs& a, uint32_t ray, uint32_t inst, float D) {
  const int gid = a.inst_gid ? a.inst_gid[inst] : int(inst);
  atomicMin(reinterpret_cast<unsigned long long*>(&a.keys[ray]), (unsigned long long)pack_key(D, gid));
}

// Work items of the list a stage reads, formed by every workgroup for itself
// from the counts in the workspace (one wave, one scan over the at most 32
// objects): a launch of its own for this prefix would cost more than all
// workgroups repeating it, since each launch waits for the one before
// (4-5 us each; the depth pass of a 64 x 64 frame was mostly such launches).
struct ItemTable {
  int32_t start[NEDF_MAX_OBJECTS + 1];  // first work item of each object
  int32_t cnt[NEDF_MAX_OBJECTS];
  int32_t off[NEDF_MAX_OBJECTS];
  int32_t total, mine;
};

// Exclusive prefix of v over the lanes of a wave (lanes 0..63) and its total.
template <class I>
__device__ __forceinline__ I wave_prefix(I v, int lane, I& total) {
  I incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const I y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  total = __shfl(incl, 63);
  return incl - v;
}

// Which of a stage's two kernels takes the list: the register-resident one
// (ROUTE_LARGE) or the feature-split one (ROUTE_SMALL), by the number of
// split_per-pair units in the list against split_max, on the device, where
// the counts are; 0 (no split_per): the stage has launched one kernel only.
enum { ROUTE_LARGE = 0, ROUTE_SMALL = 1 };

// Called by the whole workgroup; ends with a barrier.  False if the list is
// the other kernel's (uniform over the grid).
template <int ROUTE = ROUTE_LARGE>
__device__ __forceinline__ bool build_items(const KArgs& a, ItemTable& t, int per) {
  if (threadIdx.x < 64) {
    const int m = threadIdx.x;
    const int c = m < a.n_obj ? a.lcnt[m] : 0;
    const int items = m < a.n_obj && ((a.item_mask >> m) & 1u) ? (c + per - 1) / per : 0;
    int total;
    const int start = wave_prefix(items, m, total);
    if (m <= NEDF_MAX_OBJECTS) t.start[m] = start;
    if (m < NEDF_MAX_OBJECTS) {
      t.cnt[m] = c;
      t.off[m] = m < a.n_obj ? a.loff[m] : 0;
    }
    if (m == 0) t.total = total;
    int units = 0;
    if (a.split_per) wave_prefix(items ? (c + a.split_per - 1) / a.split_per : 0, m, units);
    if (m == 0) t.mine = !a.split_per || (units <= a.split_max) == (ROUTE == ROUTE_SMALL);
  }
  __syncthreads();
  return t.mine != 0;
}

// Object of work item `item`.
__device__ __forceinline__ int item_object(const ItemTable& t, int n_obj, int item) {
  int obj = 0;
  while (obj + 1 < n_obj && t.start[obj + 1] <= item) ++obj;
  return obj;
}

// Optical depth and weights of one pair, 32 samples at a time in order, one
// per lane (lanes 32..63 pass v = 0): the scan runs across the wave, the sums
// over chunks are Neumaier-compensated.
struct MarchSum {
  float carry = 0.f, carry_c = 0.f, sw = 0.f, sw_c = 0.f, swt = 0.f, swt_c = 0.f;
  // v: optical depth of this lane's sample, t: its local depth
  __device__ __forceinline__ void add(float v, float t, int lane) {
    // inclusive scan of optical depth over the wave (sample order = lane order)
    float incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    const float tau = (carry + carry_c) + (incl - v);
    const float w = expf(-tau) * one_minus_exp_neg(v);
    float ws = w, wts = w * t;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      ws += __shfl_xor(ws, off);
      wts += __shfl_xor(wts, off);
    }
    // a block wholly past the last sample adds exact zeros
    neu_add(sw, sw_c, ws);
    neu_add(swt, swt_c, wts);
    neu_add(carry, carry_c, __shfl(incl, 63));
  }
  // One lane of the pair's wave.
  __device__ __forceinline__ void emit(const KArgs& a, uint2 pr, float s) const {
    const float A = sw + sw_c;
    if (A >= a.hit_thr && A > 0.0f) emit_key(a, pr.x, pr.y, s * ((swt + swt_c) / A));
    atomicMax(&a.opac[pr.x], __float_as_uint(fmaxf(A, 0.0f)));
  }
};

// Routing of the intersection network's pairs (one per lane of a half wave;
// `mine` selects the lanes that hold one): confident hits to the key buffer,
// uncertain pairs and origins inside the bounding sphere to the object's
// segment of list B; n counts hits, fallbacks and misses.  Whole wave active.
__device__ __forceinline__ void route_pairs(const KArgs& a, int obj, int seg_off, uint2 pr, bool mine, bool inside,
                                            float p, float D, int lane, int (&n)[3]) {
  const bool to_fb = mine && (inside || (p >= a.p_lo && p <= a.p_hi));
  const bool hit = mine && !to_fb && p > a.p_hi && D > 0.0f;
  if (hit) emit_key(a, pr.x, pr.y, D);
  // wave-aggregated push into the object's segment of list B
  const uint64_t m = __ballot(to_fb);
  if (m) {
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(&a.C->B.cnt[obj], __popcll(m));
    base = __shfl(base, leader);
    if (to_fb) a.pairsB[seg_off + base + __popcll(m & ((1ull << lane) - 1ull))] = pr;
  }
  const uint64_t mh = __ballot(hit), mv = __ballot(mine);
  n[0] += __popcll(mh);
  n[1] += __popcll(m);
  n[2] += __popcll(mv) - __popcll(mh) - __popcll(m);
}
__device__ __forceinline__ void flush_routing(const KArgs& a, int lane, const int (&n)[3]) {
  if (lane == 0 && (n[0] | n[1] | n[2]))
    for (int i = 0; i < 3; ++i) atomicAdd(&a.C->stats[i], n[i]);
}

// ---- secant refinement --------------------------------------------------------
// f(t) = surface function at the local point of world depth t; seeds D -/+ h,
// `steps` secant updates with a [D - 2h, D + 2h] guard (needs steps + 1
// evaluations; the last iterate is not evaluated).
struct Secant {
  float t0, t1, f0, f1, out, lo, hi;
  bool active;
  // Seeds around D at h = rh * s.  Left to the compiler, whether a seed's
  // product is rounded before the sum depends on where in the kernel the seed
  // is used, and two kernels would start from neighbouring values.  The upper
  // seed has two roundings (ROUNDED: that of the BF16 networks), each kept so
  // that refined depths stay what they were.
  template <bool ROUNDED = false>
  __device__ void start(float D, float rh, float s) {
#pragma clang fp contract(off)
    const float h = rh * s;
    t0 = fmaf(-rh, s, D);
    t1 = ROUNDED ? D + h : fmaf(rh, s, D);
    out = D;
    lo = fmaf(-2.f, h, D);
    hi = fmaf(2.f, h, D);
  }
  __device__ float update() {  // returns the new iterate (evaluation point)
    const float den = f1 - f0;
    bool ok = active && den != 0.0f;
    const float tn = ok ? t1 - f1 * (t1 - t0) / den : t1;
    ok = ok && tn >= lo && tn <= hi;
    if (ok) out = tn;
    active = ok;
    return tn;
  }
  __device__ void shift(float tn, float fn) {
    if (active) { t0 = t1; f0 = f1; t1 = tn; f1 = fn; }
  }
};

// ---- binning of pixels by object --------------------------------------------
// A workgroup takes a contiguous range of pixels and aggregates its counts
// per object in LDS (lanes of a wave grouped by object, one LDS atomic per
// group), so global atomics are one per (workgroup, object): per-wave global
// atomics on the few counters of a list serialise across the whole chip.
constexpr unsigned BIN_BLOCKS = 1024;

inline unsigned bin_blocks(int64_t n_rays) {
  const int64_t g = (n_rays + 255) / 256;
  return unsigned(g < 1 ? 1 : g > int64_t(BIN_BLOCKS) ? int64_t(BIN_BLOCKS) : g);
}

// Pixels of each workgroup.
__device__ __forceinline__ int64_t bin_span(int64_t n_rays, unsigned blocks) {
  return ((n_rays + blocks - 1) / blocks + 255) / 256 * 256;
}

// Calls f(object, lanes, whether this lane is one of them) for every object
// of `mask` among the wave's instances (inst < 0: none); whole wave active.
template <class F>
__device__ __forceinline__ void bin_groups(const KArgs& a, int inst, uint32_t mask, int lane, F&& f) {
  const int obj = inst >= 0 && inst < a.n_inst ? a.inst_object[inst] : -1;
  const bool want = obj >= 0 && obj < a.n_obj && ((mask >> obj) & 1u);
  uint64_t pending = __ballot(want);
  while (pending) {
    const int o = __shfl(obj, __ffsll((unsigned long long)pending) - 1);
    const bool mine = want && obj == o;
    const uint64_t match = __ballot(mine);
    f(o, match, mine);
    pending &= ~match;
  }
}

}  // namespace nedf
