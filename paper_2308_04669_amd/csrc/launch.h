// Host-side launch interface between the C-ABI layer and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nedf.h"

namespace nedf {

// Per-object description passed to kernels by value.
struct ObjDesc {
  int32_t field, sigma_mode;
  float bound;
  float param[6];
  const uint8_t* blob;      // density network blob (device) or NULL
  const uint8_t* nedf_blob; // intersection network blob (device) or NULL
};

struct RaySrcHost {
  int32_t kind, width, height;
  float eye[3], fwd[3], right[3], up[3];
  const float* o;
  const float* d;
  int64_t n;
};

// A per-object list of (ray or pixel, instance) pairs in the workspace:
// object m owns pairs[off[m] .. off[m] + cnt[m]).
struct PairList {
  int32_t cnt[NEDF_MAX_OBJECTS];
  int32_t fill[NEDF_MAX_OBJECTS];
  int32_t off[NEDF_MAX_OBJECTS + 1];
  int32_t work_counter;
};

// Device counters in the workspace (after the 256-byte status block).
struct WsCounters {
  PairList A;       // primary pairs (culling result)
  PairList B;       // fallback pairs (NeDF uncertain rays); fill: those left after the depth test (marched)
  PairList R;       // pixels binned by object (refinement, shading)
  // pairs of the current depth slab of the network stage, in the segments of
  // list A: slab k counts in set k % 2 while its filter clears the other set
  int32_t slab_cnt[2][NEDF_MAX_OBJECTS];
  int32_t slab_work[2];
  int32_t last_pairs, last_items;  // of the list binned last
  int32_t stats[8]; // [0] pairs decided by the network, [1] sent to the marcher, [2] network misses,
                    // [4] pairs after culling
  uint32_t dmin_bits, dmax_bits;  // range of the pairs' lowest possible depths (float bits, >= 0)
};

// Workspace layout: status | counters | keys | opacity bits | extra (shadow
// rays) | pairs A | pairs B | pairs S | depth bounds of list A | depth slabs
// of list A | per 1024 pairs of list A, the set of slabs present (one bit per
// slab).  Capacity is per pair list (a multiple of SLAB_BLOCK).
constexpr size_t WS_BYTES_PER_PAIR = 3 * 8 + 4 + 1;
constexpr int SLAB_BLOCK = 1024;
struct WsLayout {
  size_t counters, keys, opac, pairs, pairsB, pairsS, pairsD, pairsSlab, slabMask, extra, end;
  int64_t capacity;
};

WsLayout ws_layout(int64_t n_rays, size_t extra_bytes, size_t ws_bytes);
size_t ws_fixed_bytes(int64_t n_rays, size_t extra_bytes);

hipError_t launch_compose_transforms(const double* G, int32_t n, float* w2l, hipStream_t s);

bool march_mlp_supported(int dtype, int width, int n_hidden, int L);
// Waves per workgroup of the marcher launch the tuning table selects (the
// pairs per work item of a list it marches).
int march_waves(int dtype, int width);
bool nedf_net_supported(int dtype, int width, int n_hidden, int L);
bool shade_supported(int dtype, const nedf_mlp_shape& s);
bool refine_supported(int dtype, const nedf_mlp_shape& s);

struct KArgs;

// Initial value of NEDF_TUNE_SLABS (not a number of slabs): it is chosen by
// the size of the call.
constexpr int NEDF_SLABS_AUTO = 0;

int cu_count();

// Launch shape of the 256-wide BF16/FP8 kernels from the tuning table: value
// 100 * (32-row blocks per wave - 1) + 10 * occupancy + superchunk (blocks
// sharing each weight read, workgroups per CU, chunks per copy); other shapes
// use one block, one workgroup per CU and the default superchunk.  The grid
// is persistent: one workgroup per CU and occupancy level.
// Tuning value of the matrix-core kernels: 1000 * (workgroup waves / 4 - 1) +
// 100 * (row blocks per wave - 1) + 10 * workgroups per CU + chunks per
// superchunk.

inline int tune_waves(int v) { return v >= 1000 ? 8 : 4; }

// The same stages for short lists (k_small.hip): 256-wide, eight-layer
// networks in F32 or BF16 with `grid` workgroups.
void launch_nedf_small(const KArgs& k, hipStream_t s, int dtype, unsigned grid);
void launch_march_small(const KArgs& k, hipStream_t s, int dtype, unsigned grid);
void launch_refine_small(const KArgs& k, hipStream_t s, int dtype, unsigned grid);

// Sets up k for the choice between a stage's two kernels and says which to
// launch: lists of at most `most` units of `per` pairs go to the small one.
// `most` is where the two take equal time: three rounds of 32-pair units on the
// chip (3 x 10 us against 31 us for the one round of the large kernel), four
// rounds of marched pairs (4 x 40 us against its 4 serial passes of 38 us).  In
// FP32 a round of 32-pair units takes 69 us and one of the large network
// kernel, four times the pairs, 261 us: it makes up for a part-empty last
// round after some 36 rounds of the small one (2.17 M pairs: 18.3 ms on the
// small kernel, 17.4 ms on the large one), and so does the marcher with pairs
// of at most 32 samples (25,600 rays, 16 objects: 3.6 and 3.4 ms).  With more
// samples, and in the refinement, the small FP32 kernels take 64 samples to a
// weight read and are the faster at every length.
// `bound` is the host's bound on the pairs; if it does not decide, both are
// launched and the device's counts decide (the other ends at once, about
// 4 us).  That holds for large calls too: a small object in a frame of 1.1 M
// rays leaves 756 marched pairs and 300 refined pixels, 174 and 149 us on the
// large kernels and 130 and 55 us on these.
struct Kernels {
  bool small, large;
};
Kernels choose_kernels(KArgs& k, int per, int most, int64_t bound);

// Matrix-core marcher over the list in k (objects in its item_mask).
void launch_march(const KArgs& k, hipStream_t s, int dtype, int W);
// Regression-form intersection networks over the list in k; v: launch shape.
void launch_nedf(const KArgs& k, hipStream_t s, int dtype, int v);

// Stages (kernels enqueued on s, no host synchronisation).
void stage_init_cull(const KArgs& k, hipStream_t s, uint32_t item_mask, int item_pairs);
void stage_march(const KArgs& k, hipStream_t s, bool list_b, uint32_t analytic_mask, int dtype, int W, int H,
                 int L);
// Intersection-network stage over list A, front to back in up to slabs.n depth
// slabs (objects in nedf_mask).
struct SlabPlan {
  int n;         // slabs launched
  int per_slab;  // culled pairs that make a slab worth using (0: all n are used)
};
void stage_nedf(const KArgs& k, hipStream_t s, int dtype, uint32_t nedf_mask, SlabPlan slabs,
                bool classifier = false);
// Classifier-form networks (NEDF_IN_POINTS16) over the current slab list; the
// BF16 lists of one round of four-wave items go to that kernel, longer ones to
// the eight-wave one (a round of it takes 1.4 times as long and holds twice
// the pairs).  `bound`: the host's bound on the pairs.
void launch_nedf_cls(const KArgs& k, hipStream_t s, int dtype, int64_t bound);
bool nedf_cls_supported(int dtype, const nedf_mlp_shape& s);
// Keys -> depth / id; with a nonzero bin_mask the hit pixels of those objects
// are counted for the binning that follows (stage_bin_write).
void stage_finalize(const KArgs& k, hipStream_t s, uint32_t bin_mask = 0);
constexpr int MAX_KEY_SETS = 8;
struct KeySets {
  const uint64_t* p[MAX_KEY_SETS];
  int32_t n;
};
void stage_merge_keys(const KArgs& k, hipStream_t s, const KeySets& ks);
// Second half of the binning of hit pixels into list R: the pairs, after
// their counts per object; item_mask and per describe the work items that
// the counters report.
void stage_bin_write(const KArgs& k, hipStream_t s, const int32_t* ids, uint32_t mask, uint32_t item_mask, int per);
void stage_refine(const KArgs& k, hipStream_t s, const int32_t* ids, uint32_t mlp_mask, uint32_t sphere_mask,
                  int dtype);
// rs_samples > 0: pixels whose density stays below k.rs_sigma at every one of
// their K samples are shaded again by volume rendering over the bounding
// chord with rs_samples samples.
void stage_shade(const KArgs& k, hipStream_t s, const int32_t* ids, uint32_t nerf_mask, int dtype,
                 int rs_samples = 0);
void stage_shadow_rays(const KArgs& k, hipStream_t s, const int32_t* ids, const float L[3], float dir_dist, float* so,
                       float* sd, float* dist);
void stage_shadow_init(const KArgs& k, hipStream_t s, float* shadow);
void stage_shadow_apply(const KArgs& k, hipStream_t s, const int32_t* ids, const float* depth_l, const float* dist,
                        float eps, float beta, float* shadow);
void stage_composite(const KArgs& k, hipStream_t s, const float* shadow, float* rgb);

size_t train_ws_bytes(const nedf_mlp_shape& sh, int B);
hipError_t launch_train_init(const nedf_mlp_shape& sh, const float* const* W, const float* const* b, uint8_t* st,
                             hipStream_t s);
hipError_t launch_train_step(const nedf_mlp_shape& sh, uint8_t* st, const float* o_l, const float* d_l,
                             const float* depth, const uint8_t* hit, int B, float lr, float b1, float b2, float eps,
                             float w_hit, float bound, float* loss, uint8_t* ws, hipStream_t s);
hipError_t launch_fp8_calibrate(const nedf_mlp_shape& sh, const float* const* W, const float* const* b,
                                const float* o_l, const float* d_l, int B, float* scales, uint8_t* ws,
                                hipStream_t s);
size_t fp8_calibrate_ws_bytes(const nedf_mlp_shape& sh, int B);
hipError_t launch_train_export(const nedf_mlp_shape& sh, const uint8_t* st, float* const* W, float* const* b,
                               bool grads, hipStream_t s);

}  // namespace nedf
