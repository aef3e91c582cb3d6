// Internal data layout shared by the host API (ht_api.cpp) and the kernels (ht_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "handtrack.h"

namespace ht {

constexpr int kTile = 8;            // 8x8 pixel tile = one wavefront of 64 lanes
constexpr int kTilePx = kTile * kTile;
constexpr int kWave = 64;
constexpr int kBlock = 256;         // 4 wavefronts per workgroup
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kRec = 20;            // floats per primitive record
constexpr int kNumTypes = 5;        // HT_SPHERE .. HT_ECYLINDER
constexpr int kQueues = 8;          // work queues of the ray cast: a grid has as many workgroups
constexpr int kQueueStride = 256;   // at least; ints between two queues' counters (1 KB)
constexpr int kCounterInts = kQueues * kQueueStride;
constexpr float kDMatch = 10.0f;    // d_m, mm
constexpr float kDClamp = 40.0f;    // d_M, mm
constexpr double kLambda = 20.0;
constexpr double kLambdaK = 10.0;

// Observation word: bits 0..15 depth (mm, 0 = undefined), bit 16 skin, bit 17 pixel inside
// the ROI (tiles over-hang the ROI on its right and bottom edges).
constexpr uint32_t kSkinBit = 1u << 16;
constexpr uint32_t kValidBit = 1u << 17;

// Hand model as laid out in device memory.
struct DevModel {
  int n_dof, n_seg, n_prim, n_kc;
  int n_roots;                           // independent kinematic trees (hands), <= kMaxRects
  int seg_depth[HT_MAX_SEG];             // segments above it (root: 0)
  int seg_wrist[HT_MAX_SEG];             // first wrist dof of its tree
  uint8_t seg_path[HT_MAX_SEG][HT_MAX_SEG];   // root .. the segment itself (seg_depth + 1)
  int seg_dof[HT_MAX_SEG][2];
  double seg_off[HT_MAX_SEG][12];        // row-major 3x4
  double seg_axis[HT_MAX_SEG][2][3];
  // primitives in type order (so that neighbouring lanes take the same set-up path), each with
  // its index in the model, segment, type and tree, so that a lane's loads depend on nothing
  int4 prim_id[HT_MAX_PRIM];             // index, segment, type, tree
  double prim_frame[HT_MAX_PRIM][12];
  double prim_size[HT_MAX_PRIM][3];
  double prim_inv2[HT_MAX_PRIM][3];      // 1 / size^2 (ellipsoid semi-axes)
  float lo[HT_MAX_DOF], hi[HT_MAX_DOF];
  int mutate[HT_MAX_DOF];
  int kc_a[HT_MAX_KC], kc_b[HT_MAX_KC];
  uint32_t dof_desc[HT_MAX_DOF];         // segments moved by each pose parameter
  int dof_trans[HT_MAX_DOF];             // 1 for the wrist translations (mm), else angle
};

constexpr int kMaxRects = 4;             // tile rectangles per particle (one per tree)

// Primitive index masks per type (bits for primitives 0..63 and 64..127).
struct TypeMasks {
  uint64_t m[kNumTypes][2];
};

// One observation slot.
struct FrameSlot {
  int W, H, TW, TH;          // ROI size and tile grid
  float sx, sy, sz;          // ray d = ((u-cx)*sx, (v-cy)*sy, sz); depth = t * sz
  float cx, cy, fx, fy;
  float bg;                  // background plane depth B (<= 0: none)
  int set;
  const uint32_t* words;     // [TH*TW][64] tile-major observation words
  const float* tile_td;      // [TH*TW] sum of min(|o_d - r_bg|, d_M) over the tile
  const int* tile_skin;      // [TH*TW] skin pixels of the tile
  const double* totals;      // [2]: the same two sums over the whole ROI
  const uint8_t* grad_mask;  // [H][W] gradient pixel mask of the slot, NULL: every pixel
};

// Per-particle header written by the kinematics kernel.  The tiles to visit are the union of
// up to kMaxRects disjoint rectangles (one per kinematic tree, overlapping ones merged), each
// covering its primitives' screen boxes; tile t of the particle is found by walking them.  It
// also carries what the ray cast needs of the frame's slot, so that one read of the header
// (scalar loads) starts a particle without a dependent slot lookup.
struct alignas(16) PInfo {
  int4 rect[kMaxRects];       // tx0, ty0, tw, th (tiles)
  int n_rects;
  int n_tiles;                // sum of the rectangles' tiles
  int slot;                   // observation slot (-1: unset slot)
  float kc;                   // collision term of Eq. 5
  int valid;                  // 0: non-finite pose or unset slot
  int skip;                   // 1: not evaluated (its frame has stopped, or it is a candidate
                              // of a refined particle that has stopped): nothing is written
  int kc_mask;                // collision pairs with a positive term (bit i: pair i)
  int TW;                     // the slot's tile columns and ROI width
  int W;
  float bg;                   // the slot's background plane depth, ray scales and centre
  float sx, sy, sz, cx, cy;
  const uint32_t* words;      // the slot's observation words, tile sums and gradient mask
  const float* tile_td;
  const int* tile_skin;
  const uint8_t* grad_mask;
  double bg_td, bg_or;        // the observation's ROI-wide background sums
};

struct Partial {
  double td;  // clamped depth sum minus the background sum of the processed tiles
  int a;      // sum(o_s and r_m)
  int o;      // sum(o_s or r_m) minus the background skin count of the processed tiles
};

// A particle's primitive tables as the ray cast stages them in LDS, one contiguous run of
// 16-byte words per particle: the records ([n_prim][kRec] floats), the pixel boxes ([n_prim]
// float4 (cx, hx, cy, hy): a tile overlaps when its corner pixel (x, y) has |x - cx| <= hx and
// |y - cy| <= hy; negative halves: empty), the image segments of the bounding capsules
// ([n_prim] float4 (x0, y0, dx, dy): the centres of the end spheres' image discs, pixels) and
// their reaches ([n_prim] float2 (1 / |(dx, dy)|^2 or 0, reach^2): a tile whose centre lies
// farther than reach from the segment sees none of the primitive).
struct Tables {
  int box, cap, capr, words;  // offsets of the three later pieces and the total, 16-byte words
  __host__ __device__ explicit Tables(int n_prim)
      : box(n_prim * (kRec / 4)), cap(box + n_prim), capr(cap + n_prim),
        words(capr + (n_prim + 1) / 2) {}
};

// Workspace of one evaluation call (device pointers, owned by the context).
struct Workspace {
  float4* tables;        // [n_total][Tables(n_prim).words]
  PInfo* pinfo;          // [n_total]
  float* dof_frame;      // [n_total][n_dof][8]: kind, axis xyz, point xyz (camera frame)
  float* seg_org;        // [n_total][n_seg][4]
  int* tiles;            // [n_total] tiles of each particle (a compact copy for the work list),
                         // -1 for a particle that is not evaluated (skipped)
  int* item_off;         // [n_total + 1] work list of a gradient launch: items per particle
  int* item_map;         // [items] particle of each item (launches of more than kSelfSchedMax)
  int* list;             // [4] items, tiles per item, 1: interleaved tiles (as item_map)
  Partial* partial;      // [items] forward: part q of particle r at r * parts + q
  float* wrench;         // [items][n_seg][6] (gradient only)
  int* counters;         // [2][kCounterInts] work queue counters, cleared by the kinematics
                         // kernel: for its own evaluation, and for one that reuses its tables
};

struct EvalArgs {
  const DevModel* model;
  const FrameSlot* slots;
  const int* frame_slots;
  int n_frames, n_particles;
  const float* poses;
  float* cost;
  float* grad;                 // NULL for forward only
  const uint8_t* pixel_mask;   // gradient mask of frame 0, may be NULL
  const int* frame_stop;       // [n_frames] stop flags of a swarm, may be NULL
  // NULL, or per group of active_div consecutive particles a flag: 0 = the group is not
  // evaluated (the candidates of a refined particle that has stopped refining)
  const int* active;
  int active_div;
  // evaluations performed (not skipped), kCountSlots forward sums, then as many gradient ones
  // (a workgroup adds to the sum of its index, so that they do not meet on one address)
  unsigned long long* eval_count;
  unsigned int* dev_errors;    // HT_DEVERR_* flags raised on the device, may be NULL
  // NULL, or per evaluated particle r its source s = src[r]: the particle reuses the kinematics
  // of workspace particle (r / n_particles) * src_stride + s from the previous evaluation
  // (same poses; the kinematics stage is skipped)
  const int* src;
  int src_stride;
  ht_debug dbg;                // pointers may be NULL
  int dbg_W, dbg_H;
  float dbg_bg;
  TypeMasks type_masks;
  int cull;                    // 1: screen boxes clipped to the bounding capsule's image extent
  int adjoint;                 // 1: the kinematics also writes dof_frame and seg_org
  int grid;                    // persistent workgroups
  int parts;                   // work items per particle: parts * particles <= grid, or 1
  int tiles_per_item;          // gradient work list: most tiles per item, and the nominal grid
  int list_grid;               // that its items are sized for
  int direct;                  // 1 (forward, whole particles): the ray cast writes the costs
  int finish;                  // 1: a small launch writes the costs, the last part of a particle
  int* done;                   // to finish, counted in done [n_total] where there are several;
  int* done_next;              // the launch clears a later one's counters, done_ints of them
  int done_ints;
  int n_prim, n_seg, n_dof;
};

// Tiles of a part: part q of a particle split into n parts takes tiles t with
// (t / kWavesPerBlock) mod n = q, wavefront w of its workgroup those with t mod kWavesPerBlock
// = w, so every part samples the whole hand and carries about equal work.  Parts past the
// particle's tiles do nothing; the others' partials are read by the kernel that assembles the
// evaluation.
__device__ __forceinline__ int active_parts(int n_tiles, int parts) {
  return min(parts, max((n_tiles + kWavesPerBlock - 1) / kWavesPerBlock, 1));
}

// Eq. 4-5 from the sums (FP64).
__device__ inline float cost_from_sums(double S_d, long long S_and, long long S_or, float kc) {
  double D;
  if (S_or == 0) {
    D = kLambda;
  } else {
    D = S_d / (double)S_or + kLambda * (1.0 - 2.0 * (double)S_and / (double)(S_and + S_or));
  }
  return (float)(D + kLambdaK * (double)kc);
}

// The cost of a particle that has none: of an unset slot, or of a pose that is not finite.
__device__ __forceinline__ float no_cost(int slot) { return slot < 0 ? NAN : INFINITY; }

// A particle's cost from its parts' sums (pi: its header).
template <class Ptr>
__device__ __forceinline__ float particle_cost(Ptr pi, double td, int sa, int so) {
  return pi->valid ? cost_from_sums(pi->bg_td + td, sa, (long long)pi->bg_or + so, pi->kc)
                   : no_cost(pi->slot);
}

// Sums over lanes on the vector unit: DPP moves within each 16-lane row (quad permutations, then
// row rotations by 4 and 8), on every lane of the row; for a wavefront the four row sums read from
// lanes 0, 16, 32, 48 and added in a fixed order.  Deterministic; a wavefront's total is
// wave-uniform.  (__shfl_xor lowers to ds_bpermute, an LDS round trip per step: with it the wavefront
// totals at the end of every item, of finalize and of the gradient's list cost 1 to 2 us a launch;
// gradients of 256 poses of a 64x64 hand 54.4 us, 52.5 with DPP.)  Every lane must be active, of a
// row or of the wavefront.
template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(dpp<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = dpp<CTRL>((int)b), hi = dpp<CTRL>((int)(b >> 32));
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ T row_sum(T v) {
  v += dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp<0x124>(v);   // row_ror:4
  v += dpp<0x128>(v);   // row_ror:8
  return v;
}
__device__ __forceinline__ int read_lane(int v, int lane) {
  return __builtin_amdgcn_readlane(v, lane);
}
__device__ __forceinline__ double read_lane(double v, int lane) {
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ T wave_sum(T v) {
  v = row_sum(v);
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Launch helpers implemented in ht_kernels.hip.
hipError_t launch_pack_observation(const uint16_t* depth, const uint8_t* skin, int W, int H,
                                   int TW, int TH, uint32_t* words, float* tile_td,
                                   int* tile_skin, double* totals, float bg, hipStream_t s);
enum { kStageFk = 0, kStageSched = 1, kStageRaycast = 2, kStageFinalize = 3, kNumStages = 4,
       kStageSmall = 4 };   // small forward launches: kinematics and ray cast in one
constexpr int kSelfSchedMax = 256;   // gradient launches of at most this many particles build
                                     // their own work list
constexpr int kMinTilesPerItem = 4;  // lower bound of the configured tiles_per_item
constexpr int kCountSlots = 64;
hipError_t launch_eval_stage(int stage, const EvalArgs& a, const Workspace& ws, hipStream_t s);
int raycast_groups_per_cu(bool grad, bool dbg, bool all_types, bool self, int n_prim, int n_seg);
hipError_t launch_pso_init(const DevModel* model, const ht_swarm& sw, int n_dof, hipStream_t s);
int preprocess_partials(int W, int H);
hipError_t launch_preprocess(int W, int H, const uint8_t* rgb, const uint16_t* depth,
                             const ht_seg_params& p, int* partial, uint16_t* depth_out,
                             uint8_t* skin_out, hipStream_t s);
hipError_t launch_box_around(const DevModel* model, int n_frames, int n_dof, const float* center,
                             const float* halfwidth, float* lo, float* hi, hipStream_t s);
hipError_t launch_pso_update(const DevModel* model, const ht_swarm& sw, const ht_pso_params& p,
                             int n_dof, int* flags, hipStream_t s);
// The generation update of a small swarm in one launch, which also assembles the evaluation
// before it (its arguments and workspace) into the costs.
bool pso_update_is_small(const ht_swarm& sw, int n_dof);
hipError_t launch_pso_update_small(const DevModel* model, const ht_swarm& sw,
                                   const ht_pso_params& p, int n_dof, const EvalArgs& a,
                                   const Workspace& ws, hipStream_t s);
hipError_t launch_refine_select(const ht_swarm& sw, int K, int n_dof, int* sel, float* rx,
                                float* rcost, int* active, hipStream_t s);
// One refinement update (ht_kernels.hip), fused with the assembly of the evaluation before
// it (whose arguments and workspace it reads): the gradient evaluation of the selected
// particles (propose only) or the evaluation of their candidates, four per particle.
struct RefineOp {
  int accept, propose, gather;
};
struct RefineArgs {
  int n_ref, K, n_dof;
  float eta_rot, eta_trans;
  RefineOp op;
  int eval_grad;             // the preceding evaluation computed gradients
  ht_swarm sw;
  const int* sel;            // [n_ref] swarm index of each refined particle
  float* rx;                 // [n_ref][n_dof] positions
  float* rcost;              // [n_ref] costs
  int* active;               // [n_ref] 1 while refining
  float* cand;               // [4 n_ref][n_dof] candidates
  float* grad;               // [n_ref][n_dof] gradients at rx
};
hipError_t launch_refine_update(const EvalArgs& a, const Workspace& ws, const RefineArgs& ra,
                                hipStream_t s);

}  // namespace ht
