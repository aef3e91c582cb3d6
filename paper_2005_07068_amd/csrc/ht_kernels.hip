// Evaluation kernels: observation packing, forward kinematics prologue,
// persistent ray cast + Eq. 4 cost terms + reduction (with the optional adjoint), finalize.
//
// Work decomposition: an 8x8 pixel tile is one wavefront (64 lanes, one pixel each).  The
// primitives of a particle are culled per tile by their conservative screen boxes with a
// ballot; tiles that no primitive touches render the background, whose cost terms are
// summed once per observation, so only touched tiles are visited.  A work item is a particle or
// one of the equal parts it is split into; persistent workgroups of four wavefronts stage the
// particle's primitive tables in LDS and write its cost, or one partial per part, which the
// finalize kernel combines in part order (deterministic).  The clamped depth sum is accumulated
// in FP64: its FP32 per-pixel terms are multiples of 2^-15 mm (depths of at least 256 mm), so
// the sum is exact and the cost does not depend on how the tiles were split.
#include <float.h>
#include <math.h>

#include "ht_device.h"

namespace ht {

// ------------------------------------------------------------------------------------
// small helpers

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// A pointer read from memory (a FrameSlot field) is generic to the compiler, and generic
// loads count against the LDS counter too, so every LDS wait would also wait for them; these
// buffers are device memory, so their loads are issued as global loads.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* global_ptr(const T* p) {
  return (const __attribute__((address_space(1))) T*)p;
}

// A wave-uniform address of memory that this kernel does not write: read with scalar loads
// into scalar registers.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* scalar_ptr(const T* p) {
  return (const __attribute__((address_space(4))) T*)p;
}

// C = A * B for 3x4 affine transforms (row-major, implicit last row 0 0 0 1).
__device__ inline void mul34(const double* A, const double* B, double* C) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double v = A[i * 4 + 0] * B[0 * 4 + j] + A[i * 4 + 1] * B[1 * 4 + j] +
                 A[i * 4 + 2] * B[2 * 4 + j];
      if (j == 3) v += A[i * 4 + 3];
      C[i * 4 + j] = v;
    }
  }
}

__device__ __forceinline__ void split(double x, float& hi, float& lo) {
  hi = (float)x;
  lo = (float)(x - (double)hi);
}

// ------------------------------------------------------------------------------------
// observation packing: one wavefront per tile

__global__ __launch_bounds__(kBlock) void pack_kernel(const uint16_t* __restrict__ depth,
                                                      const uint8_t* __restrict__ skin, int W,
                                                      int H, int TW, int TH,
                                                      uint32_t* __restrict__ words,
                                                      float* __restrict__ tile_td,
                                                      int* __restrict__ tile_skin, float bg) {
  const int lane = threadIdx.x & (kWave - 1);
  const int tile = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (tile >= TW * TH) return;
  const int tx = tile % TW, ty = tile / TW;
  const int u = tx * kTile + (lane & 7), v = ty * kTile + (lane >> 3);
  uint32_t w = 0;
  float td = 0.0f;
  int sk = 0;
  if (u < W && v < H) {
    const uint32_t d = depth[(size_t)v * W + u];
    const int s = skin[(size_t)v * W + u] != 0;
    w = d | (s ? kSkinBit : 0u) | kValidBit;
    const float rbg = bg > 0.0f ? bg : 0.0f;
    td = fminf(fabsf((float)d - rbg), kDClamp);
    sk = s;
  }
  words[(size_t)tile * kTilePx + lane] = w;
  // (FP32: a background that is no whole number makes this sum round, so its order is part of
  // the result)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) td += __shfl_xor(td, o);
  sk = wave_sum(sk);
  if (lane == 0) {
    tile_td[tile] = td;
    tile_skin[tile] = sk;
  }
}

// Whole-ROI background sums in a fixed order (one workgroup, a chain of latencies: 16 wavefronts
// with four tiles a load take a 640x480 frame's 4800 tiles in two rounds, 4 wavefronts with one
// tile a load in 19: 6.8 to 2.2 us, a frame's ingest 56 to 51.4 us).
constexpr int kTotalBlock = 1024;
__global__ __launch_bounds__(kTotalBlock) void total_kernel(const float* __restrict__ tile_td,
                                                            const int* __restrict__ tile_skin,
                                                            int n_tiles, double* __restrict__ out) {
  __shared__ double s_td[kTotalBlock / kWave];
  __shared__ double s_sk[kTotalBlock / kWave];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t >> 6;
  double td = 0.0, sk = 0.0;
  // (both arrays start an allocation, so their quads are aligned)
  const float4* td4 = reinterpret_cast<const float4*>(tile_td);
  const int4* sk4 = reinterpret_cast<const int4*>(tile_skin);
  const int quads = n_tiles >> 2;
  for (int i = t; i < quads; i += kTotalBlock) {
    const float4 a = td4[i];
    const int4 b = sk4[i];
    td += ((double)a.x + (double)a.y) + ((double)a.z + (double)a.w);
    sk += ((double)b.x + (double)b.y) + ((double)b.z + (double)b.w);
  }
  if (t < (n_tiles & 3)) {
    td += (double)tile_td[4 * quads + t];
    sk += (double)tile_skin[4 * quads + t];
  }
  td = wave_sum(td);
  sk = wave_sum(sk);
  if (lane == 0) {
    s_td[wave] = td;
    s_sk[wave] = sk;
  }
  __syncthreads();
  if (wave == 0) {
    td = wave_sum(lane < kTotalBlock / kWave ? s_td[lane] : 0.0);
    sk = wave_sum(lane < kTotalBlock / kWave ? s_sk[lane] : 0.0);
    if (lane == 0) {
      out[0] = td;
      out[1] = sk;
    }
  }
}

hipError_t launch_pack_observation(const uint16_t* depth, const uint8_t* skin, int W, int H,
                                   int TW, int TH, uint32_t* words, float* tile_td,
                                   int* tile_skin, double* totals, float bg, hipStream_t s) {
  const int n_tiles = TW * TH;
  hipLaunchKernelGGL(pack_kernel, dim3((n_tiles + kWavesPerBlock - 1) / kWavesPerBlock),
                     dim3(kBlock), 0, s, depth, skin, W, H, TW, TH, words, tile_td, tile_skin,
                     bg);
  hipLaunchKernelGGL(total_kernel, dim3(1), dim3(kTotalBlock), 0, s, tile_td, tile_skin, n_tiles,
                     totals);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// work list of a gradient launch of more than kSelfSched particles, built by one workgroup.
// Which tiles a wrench sum takes together is part of a gradient's bits (the rows are FP32
// sums), and the accept decisions of the refinement hang on them, so the items of a gradient
// launch are fixed by its particles and a nominal grid (a.list_grid), whatever executes them:
// about one item per nominal workgroup, a multiple of the wavefronts per workgroup, at least
// kFloorTiles tiles and at most the configured tiles_per_item (itself >= kMinTilesPerItem, which
// sizes the workspace).  An exclusive scan of the per-particle item counts then gives the
// item -> particle map.

constexpr int kFloorTiles = 8;       // (a refined generation of 64 poses of a 128x128 frame 120.5
                                     // us, 126.6 us with 16)

// Tiles per item of a list of total_tiles tiles.
__device__ __forceinline__ int tiles_per_item(const EvalArgs& a, int total_tiles) {
  int tq = (total_tiles + a.list_grid - 1) / a.list_grid;
  tq = (tq + kWavesPerBlock - 1) / kWavesPerBlock * kWavesPerBlock;
  return max(min(kFloorTiles, a.tiles_per_item), min(tq, a.tiles_per_item));
}

// Items of about equal work: a list of at most two items per nominal workgroup has nothing to
// even out its items' different costs, so each particle's items take interleaved tiles.
__device__ __forceinline__ bool interleaved(const EvalArgs& a, int total_items) {
  return total_items <= 2 * a.list_grid;
}

// Inclusive scan over the workgroup; every thread gets its own prefix and the total: a scan
// within each wavefront by lane shifts, then the wavefront totals through LDS (two barriers
// instead of two per doubling step).
// The same for a pair: v is scanned, w only totalled, through the same two barriers.
template <int NW>
__device__ int block_scan2(int2* s_sum, int v, int w, int* total_v, int* total_w) {
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
    w += __shfl_xor(w, o);
  }
  if (lane == kWave - 1) s_sum[wv] = make_int2(v, w);
  __syncthreads();
  int before = 0, all = 0, all_w = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int2 t = s_sum[q];
    before += q < wv ? t.x : 0;
    all += t.x;
    all_w += t.y;
  }
  __syncthreads();
  *total_v = all;
  *total_w = all_w;
  return v + before;
}

template <int NW>
__device__ int block_scan(int* s_sum, int v, int* total) {
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  if (lane == kWave - 1) s_sum[wv] = v;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int w = s_sum[q];
    before += q < wv ? w : 0;
    all += w;
  }
  __syncthreads();
  *total = all;
  return v + before;
}

// Each thread of the work-list kernel loads kSchedBatch tile counts at a time, so that their
// latencies overlap (the counts were written by every XCD, so each load misses this L2).
constexpr int kSchedBatch = 8;
constexpr int kSchedBlock = 1024;    // threads of the work-list kernel (its only workgroup)
constexpr int kSchedWindow = 8192;   // items staged in LDS per round (32 KB)

// Workspace particle holding the kinematics of evaluated particle r (itself, or its source
// from the previous evaluation).
__device__ __forceinline__ int src_of(const EvalArgs& a, int r) {
  return a.src ? (r / a.n_particles) * a.src_stride + a.src[r] : r;
}

// Tile counts of particles i0 .. i0 + kSchedBatch - 1 (zero from e on).  The loads are
// unconditional, their indices clamped to the last particle, so all of them are in flight at
// once (a guarded load per particle compiled into a wait per particle).
__device__ __forceinline__ void load_tiles(const EvalArgs& a, const Workspace& ws, int i0, int e,
                                           int (&v)[kSchedBatch]) {
  const int last = a.n_frames * a.n_particles - 1;
  int r[kSchedBatch];
#pragma unroll
  for (int j = 0; j < kSchedBatch; ++j) r[j] = min(i0 + j, last);
  if (a.src) {   // one branch for the batch (src_of per particle branched per load)
    int q[kSchedBatch];
#pragma unroll
    for (int j = 0; j < kSchedBatch; ++j) q[j] = a.src[r[j]];
#pragma unroll
    for (int j = 0; j < kSchedBatch; ++j) r[j] = (r[j] / a.n_particles) * a.src_stride + q[j];
  }
#pragma unroll
  for (int j = 0; j < kSchedBatch; ++j) v[j] = ws.tiles[r[j]];
  // past the chunk: not counted and no tiles (-1, as a skipped particle)
#pragma unroll
  for (int j = 0; j < kSchedBatch; ++j) v[j] = i0 + j < e ? v[j] : -1;
}

// The tile counts of batch i0 of a thread whose particles start at b: the first batch (every
// batch of launches up to BLOCK * kSchedBatch particles) is kept in registers from the
// first pass, later ones are loaded again.
__device__ __forceinline__ void batch_tiles(const EvalArgs& a, const Workspace& ws, int i0, int b,
                                            int e, const int (&v0)[kSchedBatch],
                                            int (&v)[kSchedBatch]) {
  if (i0 == b) {
#pragma unroll
    for (int j = 0; j < kSchedBatch; ++j) v[j] = v0[j];
  } else {
    load_tiles(a, ws, i0, e, v);
  }
}

__global__ __launch_bounds__(kSchedBlock) void sched_kernel(EvalArgs a, Workspace ws) {
  constexpr int BLOCK = kSchedBlock, kNW = BLOCK / kWave;
  const int n_total = a.n_frames * a.n_particles;
  __shared__ int s_sum[kNW];
  const int t = threadIdx.x;
  const int chunk = (n_total + BLOCK - 1) / BLOCK;
  const int b = min(t * chunk, n_total), e = min(b + chunk, n_total);
  int v0[kSchedBatch];
  load_tiles(a, ws, b, e, v0);
  // tiles to visit, and particles evaluated (not skipped), of this thread's chunk; a skipped
  // particle has tile count -1 and no work items
  int tiles = 0, evaluated = 0;
  for (int i0 = b; i0 < e; i0 += kSchedBatch) {
    int v[kSchedBatch];
    batch_tiles(a, ws, i0, b, e, v0, v);
#pragma unroll
    for (int j = 0; j < kSchedBatch; ++j) {
      tiles += max(v[j], 0);
      evaluated += v[j] >= 0 ? 1 : 0;
    }
  }
  __shared__ int2 s_sum2[kNW];
  int total_tiles, total_evaluated;
  block_scan2<kNW>(s_sum2, tiles, evaluated, &total_tiles, &total_evaluated);
  const int tpi = tiles_per_item(a, total_tiles);

  int local = 0;
  for (int i0 = b; i0 < e; i0 += kSchedBatch) {
    int v[kSchedBatch];
    batch_tiles(a, ws, i0, b, e, v0, v);
#pragma unroll
    for (int j = 0; j < kSchedBatch; ++j) local += (max(v[j], 0) + tpi - 1) / tpi;
  }
  int total_items;
  const int incl = block_scan<kNW>(s_sum, local, &total_items);
  const int my_b = incl - local, my_e = incl;   // this thread's items, contiguous
  // item offsets: staged in LDS (then stored coalesced) when they fit
  __shared__ int s_map[kSchedWindow];
  const bool staged = n_total <= kSchedWindow;
  int off = my_b;
  for (int i0 = b; i0 < e; i0 += kSchedBatch) {
    int v[kSchedBatch];
    batch_tiles(a, ws, i0, b, e, v0, v);
#pragma unroll
    for (int j = 0; j < kSchedBatch; ++j) {
      if (i0 + j >= e) break;
      if (staged) s_map[i0 + j] = off;
      else ws.item_off[i0 + j] = off;
      off += (max(v[j], 0) + tpi - 1) / tpi;
    }
  }
  if (staged) {
    __syncthreads();
    for (int i = t; i < n_total; i += BLOCK) ws.item_off[i] = s_map[i];
    __syncthreads();
  }
  // the item -> particle map, staged in LDS one window at a time so that the global stores
  // are coalesced (each thread's items are contiguous, so its own stores would touch one
  // cache line per lane)
  for (int w0 = 0; w0 < total_items; w0 += kSchedWindow) {
    const int w1 = min(w0 + kSchedWindow, total_items);
    if (my_b < w1 && my_e > w0) {
      int o = my_b;
      for (int i0 = b; i0 < e && o < w1; i0 += kSchedBatch) {
        int v[kSchedBatch];
        batch_tiles(a, ws, i0, b, e, v0, v);
#pragma unroll
        for (int j = 0; j < kSchedBatch; ++j) {
          if (i0 + j >= e) break;
          const int n = (max(v[j], 0) + tpi - 1) / tpi;
          const int q0 = max(o, w0), q1 = min(o + n, w1);
          for (int q = q0; q < q1; ++q) s_map[q - w0] = i0 + j;
          o += n;
        }
      }
    }
    __syncthreads();
    for (int q = w0 + t; q < w1; q += BLOCK) ws.item_map[q] = s_map[q - w0];
    __syncthreads();
  }
  if (t == 0) {
    if (a.eval_count)
      atomicAdd(&a.eval_count[kCountSlots], (unsigned long long)total_evaluated);
    ws.item_off[n_total] = total_items;
    ws.list[0] = total_items;
    ws.list[1] = tpi;
    ws.list[2] = interleaved(a, total_items) ? 1 : 0;
  }
}

// Image extent of a capsule (segment q0-q1, radius r) as the hull of its two end spheres'
// extents: the planes x = a z through the camera that touch a sphere with centre (X, Y, Z),
// Z > r, have a = (X Z -/+ r sqrt(X^2 + Z^2 - r^2)) / (Z^2 - r^2), and likewise in y.  The
// capsule's support along a plane normal is the larger of its end spheres', so no interior
// point lies outside.  Writes pixel coordinates (u0, u1, v0, v1), padded by a quarter pixel
// for the FP32 rounding; returns false when a sphere reaches the camera plane.  The culling
// geometry takes the hardware reciprocal and square root (errors of about 1e-7 relative,
// 1e-4 pixel at most, far inside the pads; the quotients' range-safe sequences made the
// primitive set-up a long chain of latencies).
using FrameSlotRef = const __attribute__((address_space(4))) FrameSlot&;
__device__ __forceinline__ bool capsule_extent(const float* q0, const float* q1, float rr,
                                               FrameSlotRef fs, float* e) {
  float amin = INFINITY, amax = -INFINITY, bmin = INFINITY, bmax = -INFINITY;
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float* q = j ? q1 : q0;
    const float X = q[0], Y = q[1], Z = q[2];
    ok &= Z > 1.001f * rr + 1.0f;
    const float den = (Z - rr) * (Z + rr);
    const float inv = fast_rcp(den);
    const float hx = rr * fast_sqrt(fmaf(X, X, den)), hy = rr * fast_sqrt(fmaf(Y, Y, den));
    const float xz = X * Z, yz = Y * Z;
    amin = fminf(amin, (xz - hx) * inv);
    amax = fmaxf(amax, (xz + hx) * inv);
    bmin = fminf(bmin, (yz - hy) * inv);
    bmax = fmaxf(bmax, (yz + hy) * inv);
  }
  e[0] = fmaf(fs.fx, amin, fs.cx) - 0.25f;
  e[1] = fmaf(fs.fx, amax, fs.cx) + 0.25f;
  e[2] = fmaf(fs.fy, bmin, fs.cy) - 0.25f;
  e[3] = fmaf(fs.fy, bmax, fs.cy) + 0.25f;
  return ok;
}

// Bounding disc of the image of a sphere (centre q, radius r, q.z > r): the image is an
// ellipse whose major axis points away from the principal point and spans the normalised
// radii tan(theta - alpha) .. tan(theta + alpha), theta being the angle of q from the optical
// axis and sin(alpha) = r / |q|.  Its centre and semi-major axis, in pixels (the larger focal
// length for the radius), give a disc that contains it.
__device__ __forceinline__ void sphere_image_disc(const float* q, float R, FrameSlotRef fs, float* D,
                                                  float& rho) {
  const float X = q[0], Y = q[1], Z = q[2];
  const float rad = fast_sqrt(fmaf(X, X, Y * Y));
  const float inv_n = __builtin_amdgcn_rsqf(fmaf(rad, rad, Z * Z));
  const float st = rad * inv_n, ct = Z * inv_n, sa = R * inv_n;
  const float ca = fast_sqrt(fmaxf(0.0f, 1.0f - sa * sa));
  const float tp = fmaf(st, ca, ct * sa) * fast_rcp(fmaf(ct, ca, -st * sa));   // tan(theta + alpha)
  const float tm = fmaf(st, ca, -ct * sa) * fast_rcp(fmaf(ct, ca, st * sa));   // tan(theta - alpha)
  const float m = 0.5f * (tp + tm), h = 0.5f * (tp - tm);
  const float ir = fast_rcp(rad);
  const float ex = rad > 0.0f ? X * ir : 1.0f, ey = rad > 0.0f ? Y * ir : 0.0f;
  D[0] = fmaf(fs.fx, m * ex, fs.cx);
  D[1] = fmaf(fs.fy, m * ey, fs.cy);
  rho = h * fmaxf(fs.fx, fs.fy);
}

// Farthest pixel centre of an 8x8 tile from the tile's centre: 3.5 sqrt(2) pixels.
constexpr float kTileHalfDiag = 4.9498f;
// The pad of a primitive's reach in pixels.  What FP32 and the hardware's reciprocals (1 ulp) take
// away is covered by the factor 1.0001 and the capsule's own margin: over images of 4096 pixels,
// principal points up to 100 000 px outside them, focal lengths of 5 to 20 000 px and hands at 30
// mm to 20 m, the silhouettes stayed 0.126 px inside the reach, and 0.24 px inside the boxes (pad
// 0.25).  (With 0.5 px 1024 two-hand poses take 116.0 us, 115.0 with 0.125; 65536 poses 2384 and
// 2367 us.)
constexpr float kReachPad = 0.125f;

// ------------------------------------------------------------------------------------
// forward kinematics prologue: one wavefront per particle (FP64 inside)

// One primitive's model data.
struct PrimIn {
  int k, seg, type, root;
  double frame[12];
  double size[3];
  double inv2[3];
};

__device__ __forceinline__ void load_prim(const DevModel* __restrict__ G, int o, PrimIn& q) {
  const int4 id = G->prim_id[o];
  q.k = id.x;
  q.seg = id.y;
  q.type = id.z;
  q.root = id.w;
  for (int i = 0; i < 12; ++i) q.frame[i] = G->prim_frame[o][i];
  for (int i = 0; i < 3; ++i) {
    q.size[i] = G->prim_size[o][i];
    q.inv2[i] = G->prim_inv2[o][i];
  }
}

// The kinematic tables of the model (everything before the primitive tables).
constexpr int kSegBytes = ((int)offsetof(DevModel, prim_id) + 15) / 16 * 16;
static_assert(kSegBytes <= (int)sizeof(DevModel), "copy stays inside the model");

// LDS of the kinematics of PPB particles.
struct FkParticle {
  double T[HT_MAX_SEG][12], L[HT_MAX_SEG][12];
  double h[HT_MAX_DOF], sin[HT_MAX_DOF], cos[HT_MAX_DOF];
  int rect[kMaxRects][4];
  int fin;
};
template <int PPB>
struct FkShared {
  FkParticle p[PPB];
  alignas(16) unsigned char model[kSegBytes];
};

// Kinematics of particle p0 + pb by wavefront h of its WPP ones (every thread of the BLOCK-thread
// workgroup calls this, for its kPpb particles): the primitive tables go to tab, the header to
// header(PInfo, lane), called by the first wavefront after the last barrier, and with a.adjoint the
// joint frames and segment origins to the workspace.  Returns false where every particle of the
// workgroup is skipped.  The rows of the transforms and the primitives are spread over the
// particle's wavefronts.
template <int BLOCK, int WPP, class Header>
__device__ __forceinline__ bool fk_particle(const EvalArgs& a, const Workspace& ws,
                                            FkShared<BLOCK / kWave / WPP>& sh, int p0, int pb,
                                            int h, int lane, int n_total, float4* tab,
                                            Header&& header) {
  constexpr int kPpb = BLOCK / kWave / WPP;      // particles per workgroup
  const int p = p0 + pb;
  const bool active = p < n_total;
  const int n_dof = a.n_dof, n_seg = a.n_seg, n_prim = a.n_prim;
  const DevModel* __restrict__ G = a.model;
  // Every load that depends on the particle alone is issued first, together and with clamped
  // indices (a load behind a branch, or issued after another whose result is awaited, adds a
  // memory latency to this latency-bound kernel): this lane's pose parameter, the frame's
  // slot and stop flag, the candidate's active flag and this lane's collision pair.
  const int pc = min(p, n_total - 1);
  const int f = pc / a.n_particles;
  const float x_lane = a.poses[(size_t)pc * n_dof + min(lane, n_dof - 1)];
  const int slot_raw = scalar_ptr(a.frame_slots)[f];
  const int stop_raw = a.frame_stop ? scalar_ptr(a.frame_stop)[f] : 0;
  const int act_raw = a.active ? scalar_ptr(a.active)[pc / a.active_div] : 1;
  const int kc_i = min(lane, HT_MAX_KC - 1);
  const int kc_a = G->kc_a[kc_i], kc_b = G->kc_b[kc_i];
  // the kinematic tables (everything before the primitive tables), staged by one coalesced
  // copy with all its loads in flight at once: the tree walk would otherwise wait on long
  // chains of dependent global loads.  The primitive tables are read from global memory by the
  // lane that sets a primitive up, issued here so that their latency overlaps the
  // trigonometry and the tree walk.
  constexpr int kN = kSegBytes / 16;
  static_assert(kN <= 2 * BLOCK, "two 16-byte words per thread");
  const uint4* model4 = reinterpret_cast<const uint4*>(a.model);
  const int tid = threadIdx.x;
  const uint4 stage0 = model4[min(tid, kN - 1)];
  uint4 stage1{};
  if constexpr (kN > BLOCK) stage1 = model4[min(tid + BLOCK, kN - 1)];
  const int slot = active ? slot_raw : -1;
  const bool in_range = slot >= 0 && slot < HT_MAX_SLOTS;
  FrameSlotRef fs = scalar_ptr(a.slots)[in_range ? slot : 0];
  const bool slot_ok = in_range && fs.set;
  if (active && !slot_ok && h == 0 && lane == 0 && a.dev_errors)
    atomicOr(a.dev_errors, HT_DEVERR_UNSET_SLOT);
  // a particle of a stopped frame (tracking stop rule), or a candidate of a refined particle
  // that has stopped refining, is neither cast nor written
  const bool skip = active && (stop_raw != 0 || act_raw == 0);

  // A workgroup whose particles are all skipped writes their headers and is done (a frozen
  // swarm's generation 1.6 us here, 3.5 us with the rest of the kernel).
  if (a.frame_stop || a.active) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < kPpb; ++j) {
      const int q = min(p0 + j, n_total - 1);
      all &= (a.frame_stop && scalar_ptr(a.frame_stop)[q / a.n_particles] != 0) ||
             (a.active && scalar_ptr(a.active)[q / a.active_div] == 0);
    }
    if (all) {
      if (active && h == 0) {
        PInfo pi{};
        pi.slot = slot_ok ? slot : -1;
        pi.skip = 1;
        header(pi, lane);
      }
      return false;
    }
  }

  {
    uint4* dst = reinterpret_cast<uint4*>(sh.model);
    if (tid < kN) dst[tid] = stage0;
    if constexpr (kN > BLOCK)
      if (tid + BLOCK < kN) dst[tid + BLOCK] = stage1;
  }
  // only the members before prim_id may be read through M
  const DevModel& M = *reinterpret_cast<const DevModel*>(sh.model);
  // this wavefront's primitives (slots of the type order): its share, in a row, so that its
  // lanes take few of the set-up paths
  const int o_per = (n_prim + WPP - 1) / WPP;
  const int o_end = min((h + 1) * o_per, n_prim);
  // every angle's sine and cosine at once (one lane per pose parameter, n_dof <= 64), so the
  // tree walk below is trigonometry-free
  static_assert(HT_MAX_DOF <= kWave, "one lane per pose parameter");
  bool finite = true;
  if (active && !skip && h == 0 && lane < n_dof) {
    const float x = x_lane;
    sh.p[pb].h[lane] = (double)x;
    finite = isfinite(x);
    double sv = 0.0, cv = 1.0;
    if (finite) sincos((double)x, &sv, &cv);
    sh.p[pb].sin[lane] = sv;
    sh.p[pb].cos[lane] = cv;
  }
  finite = __ballot(!finite) == 0ull;
  if (h == 0 && lane == 0) sh.p[pb].fin = finite ? 1 : 0;
  __syncthreads();
  // the first wavefront's finiteness test, for every wavefront of the particle
  if (WPP > 1) finite = __builtin_amdgcn_readfirstlane(sh.p[pb].fin) != 0;
  const bool valid = slot_ok && finite && !skip;
  // the slot's background sums, needed only by the record written at the end (scalar loads, two
  // dependent latencies under the tree walk)
  double bg_td = 0.0, bg_or = 0.0;
  if (slot_ok && h == 0) {
    const double* tot = fs.totals;
    bg_td = scalar_ptr(tot)[0];
    bg_or = scalar_ptr(tot)[1];
  }

  // Segment transforms, T_s = W L_root ... L_parent(s) L_s with L_s = Off_s Rot(a1, q1)
  // Rot(a2, q2) and W the wrist of s's tree, one lane per row of a transform: a row of a product
  // needs that row of the left factor alone, so a lane forms its row of L_s (a row vector times
  // a rotation is c v + (1 - c)(v.a) a + s (v x a): 21 operations a joint, where the 3x3
  // product takes 60), stages it in LDS, and after one barrier carries its row of the wrist
  // down the path from the root (12 multiply-adds a segment).  48 of a hand's lanes work where
  // one lane per segment kept 16 busy with three times the operations each.
  const int n_rows = valid ? 3 * n_seg : 0;
#pragma unroll 1
  for (int q = lane + h * kWave; q < n_rows; q += kWave * WPP) {
    const int s = q / 3, i = q - 3 * s;
    const double* off = M.seg_off[s] + 4 * i;
    double v[3] = {off[0], off[1], off[2]};
    const double t = off[3];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int dof = M.seg_dof[s][j];
      if (dof < 0) continue;
      const double* x = M.seg_axis[s][j];
      const double sn = sh.p[pb].sin[dof], cs = sh.p[pb].cos[dof];
      const double d = (1.0 - cs) * (v[0] * x[0] + v[1] * x[1] + v[2] * x[2]);
      const double c0 = v[1] * x[2] - v[2] * x[1], c1 = v[2] * x[0] - v[0] * x[2],
                   c2 = v[0] * x[1] - v[1] * x[0];
      v[0] = cs * v[0] + d * x[0] + sn * c0;
      v[1] = cs * v[1] + d * x[1] + sn * c1;
      v[2] = cs * v[2] + d * x[2] + sn * c2;
    }
    double* o = sh.p[pb].L[s] + 4 * i;
    o[0] = v[0];
    o[1] = v[1];
    o[2] = v[2];
    o[3] = t;
  }
  // the lane's primitive, loaded here so that the latency passes under the walk down the tree
  // (issued with the loads above it held 40 registers over the trigonometry)
  PrimIn pin;
  if (valid && h * o_per + lane < o_end) load_prim(G, h * o_per + lane, pin);
  __syncthreads();
#pragma unroll 1
  for (int q = lane + h * kWave; q < n_rows; q += kWave * WPP) {
    const int s = q / 3, i = q - 3 * s;
    // row i of the wrist: Trans(x, y, z) Rz(tz) Ry(ty) Rx(tx)
    const int b = M.seg_wrist[s];
    const double hq = sh.p[pb].h[b + i];
    const double sx = sh.p[pb].sin[b + 3], cx = sh.p[pb].cos[b + 3];
    const double sy = sh.p[pb].sin[b + 4], cy = sh.p[pb].cos[b + 4];
    const double sz = sh.p[pb].sin[b + 5], cz = sh.p[pb].cos[b + 5];
    const double z = i == 0 ? cz : sz;
    const double r0 = i == 2 ? -sy : z * cy, r1 = i == 0 ? -sz : (i == 1 ? cz : 0.0),
                 r2 = i == 2 ? cy : z * sy;
    double v[3] = {r0, r1 * cx + r2 * sx, r2 * cx - r1 * sx};
    double t = hq;
    const int depth = M.seg_depth[s];
    if (a.adjoint && depth == 0) {
      // wrist dofs, component i: translations along camera axes; rotations about Rz Ry e_x,
      // Rz e_y, e_z through the wrist position
      float* df = ws.dof_frame + ((size_t)p * n_dof + b) * 8;
      const double ax[3] = {v[0], i == 0 ? -sz : (i == 1 ? cz : 0.0), i == 2 ? 1.0 : 0.0};
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        float* f = df + j * 8;
        f[1 + i] = i == j;
        f[4 + i] = 0.0f;
        float* g = f + 24;
        g[1 + i] = (float)ax[j];
        g[4 + i] = (float)hq;
        if (i == 0) {
          f[0] = 1.0f;
          f[7] = g[0] = g[7] = 0.0f;
        }
      }
    }
    // (four path entries per LDS read)
#pragma unroll 1
    for (int d0 = 0; d0 <= depth; d0 += 4) {
      const uint32_t path = *reinterpret_cast<const uint32_t*>(&M.seg_path[s][d0]);
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const double* l = sh.p[pb].L[(path >> (8 * d)) & 255u];
        const bool on = d0 + d <= depth;
        const double x = v[0], y = v[1], u = v[2];
        const double n0 = x * l[0] + y * l[4] + u * l[8];
        const double n1 = x * l[1] + y * l[5] + u * l[9];
        const double n2 = x * l[2] + y * l[6] + u * l[10];
        const double nt = x * l[3] + y * l[7] + u * l[11] + t;
        v[0] = on ? n0 : x;
        v[1] = on ? n1 : y;
        v[2] = on ? n2 : u;
        t = on ? nt : t;
      }
    }
    double* o = sh.p[pb].T[s] + 4 * i;
    o[0] = v[0];
    o[1] = v[1];
    o[2] = v[2];
    o[3] = t;
    if (a.adjoint) {
      // joint axes in the camera frame, component i: the second joint's axis is R_s a2; the
      // first's is R_s Rot(a2, q2)^T a1 (each rotation leaves its own axis fixed); both pass
      // through the segment origin
      const int dof2 = M.seg_dof[s][1];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int dof = M.seg_dof[s][j];
        if (dof < 0) continue;
        const double* a1 = M.seg_axis[s][j];
        double x[3] = {a1[0], a1[1], a1[2]};
        if (j == 0 && dof2 >= 0) {
          // Rot(a2, q2)^T x = c x - s (a2 x x) + (1 - c)(a2 . x) a2
          const double* a2 = M.seg_axis[s][1];
          const double sn = sh.p[pb].sin[dof2], cs = sh.p[pb].cos[dof2];
          const double dt = (1.0 - cs) * (a2[0] * x[0] + a2[1] * x[1] + a2[2] * x[2]);
          const double cr[3] = {a2[1] * x[2] - a2[2] * x[1], a2[2] * x[0] - a2[0] * x[2],
                                a2[0] * x[1] - a2[1] * x[0]};
          for (int k = 0; k < 3; ++k) x[k] = cs * x[k] - sn * cr[k] + dt * a2[k];
        }
        float* f = ws.dof_frame + ((size_t)p * n_dof + dof) * 8;
        f[1 + i] = (float)(v[0] * x[0] + v[1] * x[1] + v[2] * x[2]);
        f[4 + i] = (float)t;
        if (i == 0) f[0] = f[7] = 0.0f;
      }
      float* so = ws.seg_org + ((size_t)p * n_seg + s) * 4;
      so[i] = (float)t;
      if (i == 0) so[3] = 0.0f;
    }
  }
  // collision terms of Eq. 5, one per lane; they are differences of FP32 values, so their FP64
  // sum is exact in any order, and few are positive
  double kc = 0.0;
  int kc_mask = 0;
  if (valid && h == 0) {
    const double v = lane < M.n_kc ? fmax(-(sh.p[pb].h[kc_a] - sh.p[pb].h[kc_b]), 0.0) : 0.0;
    kc_mask = (int)__ballot(v > 0.0);
    for (int m = kc_mask; m; m &= m - 1) {
      const int l = __builtin_ctz(m);
      kc += read_lane(v, l);
    }
  }
  if (h == 0 && lane < kMaxRects * 4)
    sh.p[pb].rect[lane >> 2][lane & 3] = (lane & 1) ? INT_MIN : INT_MAX;
  __syncthreads();

  // primitive records and screen boxes, in type order; per-tree unions of the primitive boxes
  // (u0, v0 minima; u1, v1 maxima), accumulated with LDS atomics (cheaper than sixteen wave
  // reductions)
  if (valid) {
    const Tables L(n_prim);
    if (h * o_per + lane < o_end) {   // (at most one primitive per lane, see launch_eval_stage)
      const int k = pin.k;
      const int s = pin.seg;
      double F[12];
      mul34(sh.p[pb].T[s], pin.frame, F);
      const double* sz = pin.size;
      const int typ = pin.type;
      float rec[kRec];
      for (int i = 0; i < kRec; ++i) rec[i] = 0.0f;
      const double c[3] = {F[3], F[7], F[11]};
      const double* T = sh.p[pb].T[s];
      split(c[0], rec[0], rec[4]);
      split(c[1], rec[1], rec[5]);
      split(c[2], rec[2], rec[6]);
      rec[12] = (float)(c[0] - T[3]);
      rec[13] = (float)(c[1] - T[7]);
      rec[14] = (float)(c[2] - T[11]);
      rec[15] = __int_as_float(s);
      // the frame's columns are unit vectors to FP64 rounding, so the axis needs no
      // normalisation
      const double u[3] = {F[2], F[6], F[10]};
      // terms of the ray tests that do not depend on the pixel are formed here once, as the
      // same FP32 operations the tests would perform (so the tests' results are unchanged):
      // products with the ray's z component sz
      if (typ == HT_SPHERE) {
        rec[3] = (float)(sz[0] * sz[0]);
        rec[7] = fs.sz * rec[2];
      } else if (typ == HT_CYLINDER || typ == HT_CONE) {
        // circular cylinder (radius r0) or truncated cone (radius r0 at s = 0, r1 at s = L)
        const double r0 = sz[0], L = sz[1], r1 = typ == HT_CONE ? sz[2] : sz[0];
        rec[3] = typ == HT_CONE ? (float)r0 : (float)(r0 * r0);
        rec[7] = (float)L;
        rec[8] = (float)u[0];
        rec[9] = (float)u[1];
        rec[10] = (float)u[2];
        rec[11] = typ == HT_CONE ? (float)((r1 - r0) / L)
                                 : (float)(c[0] * u[0] + c[1] * u[1] + c[2] * u[2]);
        if (typ == HT_CYLINDER) {
          // sz uz, then the part of the cap centre perpendicular to the axis (q = c - (c.u) u:
          // q_z sz, q_x, q_y), whose product with d is the side reference's numerator
          const double cu = c[0] * u[0] + c[1] * u[1] + c[2] * u[2];
          rec[16] = fs.sz * rec[10];
          rec[17] = fs.sz * (float)(c[2] - cu * u[2]);
          rec[18] = (float)(c[0] - cu * u[0]);
          rec[19] = (float)(c[1] - cu * u[1]);
        }
      } else {
        // ellipsoid: Q = R diag(1/s^2) R^T with R the rotation part of F; elliptic cylinder:
        // the same without the axis term, Q = ex ex^T / a^2 + ey ey^T / b^2
        const bool ecyl = typ == HT_ECYLINDER;
        const double inv[3] = {pin.inv2[0], ecyl ? pin.inv2[2] : pin.inv2[1],
                               ecyl ? 0.0 : pin.inv2[2]};
        double Q[6] = {0, 0, 0, 0, 0, 0};
        for (int j = 0; j < 3; ++j) {
          const double r0 = F[0 * 4 + j], r1 = F[1 * 4 + j], r2 = F[2 * 4 + j];
          Q[0] += inv[j] * r0 * r0;
          Q[1] += inv[j] * r0 * r1;
          Q[2] += inv[j] * r0 * r2;
          Q[3] += inv[j] * r1 * r1;
          Q[4] += inv[j] * r1 * r2;
          Q[5] += inv[j] * r2 * r2;
        }
        rec[3] = (float)Q[0];
        rec[7] = (float)Q[1];
        rec[8] = (float)Q[2];
        rec[9] = (float)Q[3];
        rec[10] = (float)Q[4];
        rec[11] = (float)Q[5];
        if (ecyl) {
          rec[16] = (float)u[0];
          rec[17] = (float)u[1];
          rec[18] = (float)u[2];
          rec[19] = (float)sz[1];
        } else {
          rec[16] = rec[8] * fs.sz;
          rec[17] = rec[10] * fs.sz;
          rec[18] = rec[11] * fs.sz;
        }
      }
      float4* dst = tab + k * (kRec / 4);
      for (int i = 0; i < kRec / 4; ++i)
        dst[i] = make_float4(rec[4 * i], rec[4 * i + 1], rec[4 * i + 2], rec[4 * i + 3]);

      // Conservative pixel box of an axis-aligned 3D box of the solid, and its bounding capsule,
      // in FP32 (the rounding of a 600 mm coordinate, about 1e-4 mm or pixels, is covered by the
      // quarter-pixel pads) and without branches or selects per axis.  The solid is the convex
      // hull of a cross-section at c and one at c + L u (caps, not the sphere and the ellipsoid).
      // A section's reach along an axis is the root of
      //   r^2 (sphere), r^2 - r^2 u_i^2 (disc across u), sum_j F_ij^2 g_j^2 (ellipsoid, elliptic disc
      // with semi-axes g along the frame's columns);
      // columns that a type's definition leaves free are zero in the model's tables.
      const bool ball = typ == HT_SPHERE, round = typ == HT_CYLINDER || typ == HT_CONE;
      const bool capped = !ball && typ != HT_ELLIPSOID;
      const float s0 = (float)sz[0], s1 = (float)sz[1], s2 = (float)sz[2];
      const float r2 = ball || round ? s0 * s0 : 0.0f;
      const float g1 = typ == HT_ELLIPSOID ? s1 : (typ == HT_ECYLINDER ? s2 : 0.0f);
      const float g22 = round ? -r2 : (typ == HT_ELLIPSOID ? s2 * s2 : 0.0f);
      const float k1 = typ == HT_CONE ? s2 * fast_rcp(s0) : 1.0f;   // the second section's scale
      const float Lf = capped ? s1 : 0.0f;
      const float cf[3] = {(float)c[0], (float)c[1], (float)c[2]};
      float Ff[3][3], lo3[3], hi3[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j) Ff[i][j] = (float)F[i * 4 + j];
        const float f0 = Ff[i][0] * s0, f1 = Ff[i][1] * g1;
        const float q = fmaf(f0, f0, fmaf(f1, f1, fmaf(g22, Ff[i][2] * Ff[i][2], r2)));
        const float e = fast_sqrt(fmaxf(q, 0.0f));
        const float c1 = fmaf(Lf, Ff[i][2], cf[i]);
        lo3[i] = fminf(cf[i] - e, c1 - k1 * e);
        hi3[i] = fmaxf(cf[i] + e, c1 + k1 * e);
      }
      int4 box;
      // the same bounds unrounded, for the tile test below
      float bx0 = 0.0f, bx1 = (float)(fs.W - 1), by0 = 0.0f, by1 = (float)(fs.H - 1);
      if (!(lo3[2] > 1.0f)) {
        box = make_int4(0, fs.W - 1, 0, fs.H - 1);
      } else if (fs.bg > 0.0f && lo3[2] >= fs.bg) {
        box = make_int4(1, 0, 1, 0);   // entirely behind the background plane
      } else {
        const float izl = fast_rcp(lo3[2]), izh = fast_rcp(hi3[2]);
        const float xmin = fminf(lo3[0] * izl, lo3[0] * izh);
        const float xmax = fmaxf(hi3[0] * izl, hi3[0] * izh);
        const float ymin = fminf(lo3[1] * izl, lo3[1] * izh);
        const float ymax = fmaxf(hi3[1] * izl, hi3[1] * izh);
        const float lim = 1.0e6f;
        bx0 = fmaf(fs.fx, xmin, fs.cx) - 0.25f;
        bx1 = fmaf(fs.fx, xmax, fs.cx) + 0.25f;
        by0 = fmaf(fs.fy, ymin, fs.cy) - 0.25f;
        by1 = fmaf(fs.fy, ymax, fs.cy) + 0.25f;
        const float u0 = fminf(fmaxf(floorf(bx0), -1.0f), lim);
        const float u1 = fminf(fmaxf(ceilf(bx1), -1.0f), lim);
        const float v0 = fminf(fmaxf(floorf(by0), -1.0f), lim);
        const float v1 = fminf(fmaxf(ceilf(by1), -1.0f), lim);
        box.x = max((int)u0, 0);
        box.y = min((int)u1, fs.W - 1);
        box.z = max((int)v0, 0);
        box.w = min((int)v1, fs.H - 1);
      }
      float4 cap = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      float2 capr = make_float2(0.0f, INFINITY);
      if (a.cull && box.x <= box.y && box.z <= box.w) {
        // tighter: the exact image extent of a bounding capsule (segment q0-q1, radius cr),
        // intersected with the box above (the capsule reaches past a cylinder's ends).  An
        // ellipsoid with semi-axes a >= b >= c lies in the capsule along its a-axis from
        // -(a - b) to (a - b) with radius b.
        // longest semi-axis ia of an ellipsoid (the first of equal ones)
        const bool y_longer = s1 > s0;
        const float m01 = fmaxf(s0, s1);
        const int ia = s2 > m01 ? 2 : (y_longer ? 1 : 0);
        const bool ell = typ == HT_ELLIPSOID;
        const float sa = fmaxf(m01, s2);
        const float b2 = ia == 2 ? m01 : fmaxf(fminf(s0, s1), s2);   // the larger of the others
        const float o0 = ell ? b2 - sa : 0.0f, o1 = ell ? sa - b2 : Lf;
        const int col = ell ? ia : 2;
        float cr = ell ? b2 : (typ == HT_CONE || typ == HT_ECYLINDER ? fmaxf(s0, s2) : s0);
        cr += 0.01f + 1e-6f * (fabsf(cf[0]) + fabsf(cf[1]) + fabsf(cf[2]));
        float q0[3], q1[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const float ax = col == 0 ? Ff[i][0] : (col == 1 ? Ff[i][1] : Ff[i][2]);
          q0[i] = fmaf(o0, ax, cf[i]);
          q1[i] = fmaf(o1, ax, cf[i]);
        }
        float e[4];
        if (capsule_extent(q0, q1, cr, fs, e)) {
          const float lim = 1.0e6f;
          const int u0 = (int)fminf(fmaxf(floorf(e[0]), -1.0f), lim);
          const int u1 = (int)fminf(fmaxf(ceilf(e[1]), -1.0f), lim);
          const int v0 = (int)fminf(fmaxf(floorf(e[2]), -1.0f), lim);
          const int v1 = (int)fminf(fmaxf(ceilf(e[3]), -1.0f), lim);
          bx0 = fmaxf(bx0, e[0]);
          bx1 = fminf(bx1, e[1]);
          by0 = fmaxf(by0, e[2]);
          by1 = fminf(by1, e[3]);
          box.x = max(box.x, u0);
          box.y = min(box.y, u1);
          box.z = max(box.z, v0);
          box.w = min(box.w, v1);
          // the capsule's image is the convex hull of its end spheres' images, so it lies
          // within the larger of their bounding discs' radii of the segment joining the
          // discs' centres; a tile is reached when its centre is within that radius plus the
          // tile's half-diagonal (padded for the FP32 rounding)
          float D0[2], D1[2], r0, r1;
          sphere_image_disc(q0, cr, fs, D0, r0);
          sphere_image_disc(q1, cr, fs, D1, r1);
          const float reach = fmaxf(r0, r1) * 1.0001f + kTileHalfDiag + kReachPad;
          const float dx = D1[0] - D0[0], dy = D1[1] - D0[1];
          const float vv = fmaf(dx, dx, dy * dy);
          // (the first disc's centre stored less the tile-centre offset 3.5 px, so the ray
          // cast measures from a tile's corner pixel index)
          cap = make_float4(D0[0] - 3.5f, D0[1] - 3.5f, dx, dy);
          capr = make_float2(vv > 0.0f ? fast_rcp(vv) : 0.0f, reach * reach);
        }
      }
      tab[L.cap + k] = cap;
      reinterpret_cast<float2*>(tab + L.capr)[k] = capr;
      if (box.x > box.y || box.z > box.w) box = make_int4(1, 0, 1, 0);
      {
        // |x - cx| <= hx and |y - cy| <= hy for a tile's corner pixel (x, y), exact in FP32.
        // Rays pass through whole pixel coordinates, so the (padded) bounds round inwards here;
        // the tile rectangles, which size the gradient's work items, keep the box rounded outwards.
        // A tile tests 6 to 8 % fewer primitives (outwards and inwards: 1024 two-hand poses 118.8 and
        // 115.0 us, 64 uneven frames 88.1 and 83.2 us, 65536 poses 2456 and 2367 us).
        const float x0 = fmaxf(ceilf(bx0), 0.0f), x1 = fminf(floorf(bx1), (float)(fs.W - 1));
        const float y0 = fmaxf(ceilf(by0), 0.0f), y1 = fminf(floorf(by1), (float)(fs.H - 1));
        const bool none = box.x > box.y || !(x0 <= x1) || !(y0 <= y1);
        tab[L.box + k] = make_float4(0.5f * (x0 + x1 - (float)(kTile - 1)),
                                     none ? -1.0f : 0.5f * (x1 - x0 + (float)(kTile - 1)),
                                     0.5f * (y0 + y1 - (float)(kTile - 1)),
                                     none ? -1.0f : 0.5f * (y1 - y0 + (float)(kTile - 1)));
      }
      if (box.x <= box.y) {
        int* rq = sh.p[pb].rect[pin.root];
        atomicMin(rq + 0, box.x);
        atomicMax(rq + 1, box.y);
        atomicMin(rq + 2, box.z);
        atomicMax(rq + 3, box.w);
      }
    }
  }
  __syncthreads();
  if (active && h == 0) {
    // every lane computes the record from wave-uniform values (scalar instructions); lane 0
    // stores it
    PInfo pi{};
    pi.slot = slot_ok ? slot : -1;
    pi.valid = valid ? 1 : 0;
    pi.skip = skip ? 1 : 0;
    pi.kc = (float)kc;
    pi.kc_mask = kc_mask;
    pi.bg_td = bg_td;
    pi.bg_or = bg_or;
    if (slot_ok) {
      pi.TW = fs.TW;
      pi.W = fs.W;
      pi.bg = fs.bg;
      pi.sx = fs.sx;
      pi.sy = fs.sy;
      pi.sz = fs.sz;
      pi.cx = fs.cx;
      pi.cy = fs.cy;
      pi.words = fs.words;
      pi.tile_td = fs.tile_td;
      pi.tile_skin = fs.tile_skin;
      pi.grad_mask = fs.grad_mask;
    }
    // one tile rectangle per tree, as (x0, y0, x1, y1) inclusive; overlapping ones are merged
    // (into the lower index) so that no tile is visited twice.  Every index below is a
    // compile-time constant, so the rectangles stay in registers.
    int4 R[kMaxRects];
    bool live[kMaxRects];
#pragma unroll
    for (int r = 0; r < kMaxRects; ++r) {
      const int x0 = __builtin_amdgcn_readfirstlane(sh.p[pb].rect[r][0]);
      const int x1 = __builtin_amdgcn_readfirstlane(sh.p[pb].rect[r][1]);
      const int y0 = __builtin_amdgcn_readfirstlane(sh.p[pb].rect[r][2]);
      const int y1 = __builtin_amdgcn_readfirstlane(sh.p[pb].rect[r][3]);
      live[r] = valid && x0 <= x1;
      R[r] = make_int4(x0 >> 3, y0 >> 3, x1 >> 3, y1 >> 3);   // (kTile = 8)
    }
    // a sweep without a merge is the fixed point; each earlier sweep merges at least once.
    // Only the model's trees can hold rectangles (a one-hand model needs no merge, two hands
    // one pair test per sweep); the bounds are wave-uniform, so the skipped tests cost nothing.
    const int nr = M.n_roots;
#pragma unroll
    for (int sweep = 0; sweep < kMaxRects - 1; ++sweep) {
      if (sweep + 1 >= nr) break;
#pragma unroll
      for (int i = 0; i < kMaxRects; ++i) {
#pragma unroll
        for (int j = i + 1; j < kMaxRects; ++j) {
          if (j >= nr) break;
          if (live[i] && live[j] && R[i].x <= R[j].z && R[j].x <= R[i].z &&
              R[i].y <= R[j].w && R[j].y <= R[i].w) {
            R[i] = make_int4(min(R[i].x, R[j].x), min(R[i].y, R[j].y), max(R[i].z, R[j].z),
                             max(R[i].w, R[j].w));
            live[j] = false;
          }
        }
      }
    }
    int n = 0, nt = 0;
#pragma unroll
    for (int r = 0; r < kMaxRects; ++r) {
      if (live[r]) {
        const int tw = R[r].z - R[r].x + 1, th = R[r].w - R[r].y + 1;
        const int4 q = make_int4(R[r].x, R[r].y, tw, th);
#pragma unroll
        for (int d = 0; d <= r; ++d)
          if (d == n) pi.rect[d] = q;
        ++n;
        nt += tw * th;
      }
    }
    pi.n_rects = n;
    pi.n_tiles = nt;
    header(pi, lane);
  }
  return true;
}

constexpr int kFkSpread = 256;   // launches of at most this many particles: WPP = 4

// WPP wavefronts per particle (the host's choice, see launch_eval_stage).
template <int WPP>
__global__ __launch_bounds__(kBlock, WPP == 1 ? 4 : 3) void fk_kernel(EvalArgs a, Workspace ws) {
  constexpr int kPpb = kWavesPerBlock / WPP;
  __shared__ FkShared<kPpb> sh;
  // the wavefront index as a scalar, so that everything per particle is wave-uniform (scalar
  // instructions and branches)
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pb = w / WPP, h = w % WPP;           // particle in the workgroup, its wavefront
  const int p0 = blockIdx.x * kPpb, p = p0 + pb;
  // the work queues' counters of the ray cast that follows, and of one that reuses its tables
  if (blockIdx.x == 0 && threadIdx.x < 2 * kQueues) ws.counters[threadIdx.x * kQueueStride] = 0;
  fk_particle<kBlock, WPP>(a, ws, sh, p0, pb, h, lane, a.n_frames * a.n_particles,
                           ws.tables + (size_t)p * Tables(a.n_prim).words,
                           [&](const PInfo& pi, int l) {
                             if (l == 0) {
                               ws.pinfo[p] = pi;
                               ws.tiles[p] = pi.skip ? -1 : pi.n_tiles;
                             }
                           });
}

// ------------------------------------------------------------------------------------
// per-pixel background for the debug images

__global__ __launch_bounds__(kBlock) void debug_fill_kernel(ht_debug dbg, size_t n, float bg) {
  const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  if (dbg.depth) dbg.depth[i] = bg > 0.0f ? bg : 0.0f;
  if (dbg.hit) dbg.hit[i] = 0;
  if (dbg.rm) dbg.rm[i] = 0;
  if (dbg.winner) dbg.winner[i] = -1;
  if (dbg.margin) dbg.margin[i] = -INFINITY;
}

// ------------------------------------------------------------------------------------
// ray-primitive intersections (FP32; centres carried as hi + lo pairs)
//
// The ray is x = t d with d = ((u - cx) sx, (v - cy) sy, sz), formed in FP32 (to within a
// rounding of its components) and then taken as exact; depth = t sz.  Every test first forms
// the offset of the ray's closest-approach point from the primitive centre, which is accurate
// because the tests use that same FP32 d and the centre is a double-float pair; the
// hit decision and the half-chord then come from small, well-conditioned quantities.

// A test may report a miss as ok with a NaN entry (the half-chord of a ray that misses is the
// square root of a negative number): the caller compares entries as unsigned integers, and a
// NaN's bit pattern exceeds +inf's, so such an entry is never taken.
struct Hit {
  float t;        // ray parameter of the entry point
  bool ok;
  float nx, ny, nz;   // outward normal direction at the entry (unnormalised)
  float rx, ry, rz;   // entry point minus the primitive reference point
  float m;            // ray-surface margin (debug images only, MRG)
};

// Margin of a capped side and its two caps (the survey's rule, as the oracle computes it): a
// side root's slack is the least of the radial slack and the axial slacks s/L, (L - s)/L at the
// root (the radial slack alone when the ray misses the side); a cap's slack is its disc's
// radial slack at the cap point; the margin is the largest of the four.  radial: the side's
// radial slack; s_a, s_b: axial coordinates of the two side roots; cap0, cap1: the caps'.
__device__ __forceinline__ float capped_margin(float radial, bool side_hit, float s_a, float s_b,
                                               float L, float cap0, float cap1) {
  const float iL = 1.0f / L;
  const float sa = fminf(radial, fminf(s_a * iL, (L - s_a) * iL));
  const float sb = fminf(radial, fminf(s_b * iL, (L - s_b) * iL));
  const float side = side_hit ? fmaxf(sa, sb) : radial;
  return fmaxf(fmaxf(side, cap0), cap1);
}

template <bool GRAD, bool MRG = false>
__device__ __forceinline__ void sphere_test(const float* r, float dx, float dy, float dz,
                                            float inv_dd, Hit& h) {
  const float b = fmaf(dx, r[0], fmaf(dy, r[1], r[7]));   // r[7] = dz r[2]
  const float t0 = b * inv_dd;
  const float vx = fmaf(t0, dx, -r[0]) - r[4];
  const float vy = fmaf(t0, dy, -r[1]) - r[5];
  const float vz = fmaf(t0, dz, -r[2]) - r[6];
  const float rho2 = fmaf(vx, vx, fmaf(vy, vy, vz * vz));
  const float h2 = r[3] - rho2;
  h.ok = true;   // a miss (h2 < 0) has a NaN entry
  const float hs = fast_sqrt(h2 * inv_dd);
  h.t = t0 - hs;
  if (MRG) h.m = h2 / r[3];
  if (GRAD) {
    h.rx = fmaf(-hs, dx, vx);
    h.ry = fmaf(-hs, dy, vy);
    h.rz = fmaf(-hs, dz, vz);
    h.nx = h.rx;
    h.ny = h.ry;
    h.nz = h.rz;
  }
}

template <bool GRAD, bool MRG = false>
__device__ __forceinline__ void ellipsoid_test(const float* r, float dx, float dy, float dz,
                                               Hit& h) {
  const float q00 = r[3], q01 = r[7], q02 = r[8], q11 = r[9], q12 = r[10], q22 = r[11];
  // r[16..18] = (q02, q12, q22) dz
  const float qdx = fmaf(q00, dx, fmaf(q01, dy, r[16]));
  const float qdy = fmaf(q01, dx, fmaf(q11, dy, r[17]));
  const float qdz = fmaf(q02, dx, fmaf(q12, dy, r[18]));
  const float dqd = fmaf(dx, qdx, fmaf(dy, qdy, dz * qdz));
  const float cqd = fmaf(r[0], qdx, fmaf(r[1], qdy, r[2] * qdz));
  const float inv = fast_rcp(dqd);
  const float t0 = cqd * inv;
  const float vx = fmaf(t0, dx, -r[0]) - r[4];
  const float vy = fmaf(t0, dy, -r[1]) - r[5];
  const float vz = fmaf(t0, dz, -r[2]) - r[6];
  const float qvx = fmaf(q00, vx, fmaf(q01, vy, q02 * vz));
  const float qvy = fmaf(q01, vx, fmaf(q11, vy, q12 * vz));
  const float qvz = fmaf(q02, vx, fmaf(q12, vy, q22 * vz));
  // t0 carries the rounding of c.Qd; the linear term B re-centres the chord exactly
  const float B = fmaf(vx, qdx, fmaf(vy, qdy, vz * qdz));
  const float cc = -B * inv;
  const float m = fmaf(B, B * inv, 1.0f - fmaf(vx, qvx, fmaf(vy, qvy, vz * qvz)));
  h.ok = true;   // a miss (m < 0) has a NaN entry
  const float tin = cc - fast_sqrt(m * inv);
  h.t = t0 + tin;
  if (MRG) h.m = m;
  if (GRAD) {
    h.rx = fmaf(tin, dx, vx);
    h.ry = fmaf(tin, dy, vy);
    h.rz = fmaf(tin, dz, vz);
    h.nx = fmaf(tin, qdx, qvx);
    h.ny = fmaf(tin, qdy, qvy);
    h.nz = fmaf(tin, qdz, qvz);
  }
}

// Closed cylinder as the intersection of the infinite cylinder and the slab 0 <= s <= L:
// both intervals are expressed as offsets from the reference parameter t_r (the closest
// approach to the axis), so the hit test compares small accurate numbers.
//
// Margin of the cylinder at one pixel (debug images): offsets tau from t_r, radius^2 at tau
// is rho2 + 2 tau B + tau^2 A, axial coordinate a3 + tau da.
__device__ __forceinline__ float cylinder_margin(const float* r, bool par, float A, float B,
                                                 float rho2, float h2, float invA, float cc,
                                                 float a3, float da, float inv_da) {
  const float L = r[7];
  const float ir2 = 1.0f / r[3];
  const float hsf = fast_sqrt(fmaxf(h2, 0.0f) * invA);
  const float sa = fmaf(cc - hsf, da, a3), sb = fmaf(cc + hsf, da, a3);
  const float c0 = -a3 * inv_da, c1 = (L - a3) * inv_da;
  const float q0 = fmaf(c0, fmaf(c0, A, 2.0f * B), rho2);
  const float q1 = fmaf(c1, fmaf(c1, A, 2.0f * B), rho2);
  const bool axial = da != 0.0f;
  return capped_margin(par ? -INFINITY : h2 * ir2, !par && h2 >= 0.0f, sa, sb, L,
                       axial ? (r[3] - q0) * ir2 : -INFINITY,
                       axial ? (r[3] - q1) * ir2 : -INFINITY);
}

template <bool GRAD, bool MRG = false>
__device__ __forceinline__ void cylinder_test(const float* r, float dx, float dy, float dz,
                                              float dd, Hit& h) {
  const float ux = r[8], uy = r[9], uz = r[10], L = r[7];
  const float da = fmaf(dx, ux, fmaf(dy, uy, r[16]));   // r[16] = dz uz
  const float px = fmaf(-da, ux, dx), py = fmaf(-da, uy, dy), pz = fmaf(-da, uz, dz);
  const float A = fmaf(px, px, fmaf(py, py, pz * pz));
  const bool par = A < 1.0e-6f * dd;          // ray within ~1e-3 rad of the axis
  const float inv_da = fast_rcp(da);
  const float invA = fast_rcp(A);
  // (p . c = d . q: q, the cap centre's part perpendicular to the axis, is in r[17..19])
  const float t_side = fmaf(dx, r[18], fmaf(dy, r[19], r[17])) * invA;
  {
    // every lane first as if its ray were not near-parallel to the axis: the side-centred
    // reference, and a miss of the side surface (h2 < 0) gives a NaN half-chord, which fails
    // both interval comparisons.  The values equal the general path's for such lanes.
    const float tr = t_side;
    const float vx = fmaf(tr, dx, -r[0]) - r[4];
    const float vy = fmaf(tr, dy, -r[1]) - r[5];
    const float vz = fmaf(tr, dz, -r[2]) - r[6];
    const float a3 = fmaf(vx, ux, fmaf(vy, uy, vz * uz));
    const float wx = fmaf(-a3, ux, vx), wy = fmaf(-a3, uy, vy), wz = fmaf(-a3, uz, vz);
    const float rho2 = fmaf(wx, wx, fmaf(wy, wy, wz * wz));
    const float B = fmaf(wx, px, fmaf(wy, py, wz * pz));
    const float cc = -B * invA;
    const float h2 = fmaf(B, B * invA, r[3] - rho2);
    const float hs = fast_sqrt(h2 * invA);
    const float d0 = -a3 * inv_da, d1 = (L - a3) * inv_da;
    const float din = fminf(d0, d1), dout = fmaxf(d0, d1);
    const float s_in = cc - hs, s_out = cc + hs;
    h.ok = (s_in <= dout) & (din <= s_out);
    const float tin = fmaxf(s_in, din);
    {
      // a plain sum, as on the general path (where t_r is a select): not fused with t_r's
      // product
#pragma clang fp contract(off)
      h.t = tr + tin;
    }
    if (MRG) h.m = cylinder_margin(r, false, A, B, rho2, h2, invA, cc, a3, da, inv_da);
    if (GRAD) {
      const bool cap = din > s_in;
      h.rx = fmaf(tin, dx, vx);
      h.ry = fmaf(tin, dy, vy);
      h.rz = fmaf(tin, dz, vz);
      const float sgn = da > 0.0f ? -1.0f : 1.0f;
      h.nx = cap ? sgn * ux : fmaf(tin, px, wx);
      h.ny = cap ? sgn * uy : fmaf(tin, py, wy);
      h.nz = cap ? sgn * uz : fmaf(tin, pz, wz);
    }
  }
  // a near-parallel ray (its pixel lies within about half a pixel of the image of the axis's
  // vanishing point, so few wavefronts ever have one) sends the wavefront down the general
  // path, which recomputes every lane
  if (__builtin_expect(__ballot(par) == 0ull, 1)) return;
  // general path: near-parallel rays take the reference at the slab's middle
  const float t_mid = fmaf(0.5f, L, r[11]) * inv_da;    // r[11] = c . u
  const float tr = par ? t_mid : t_side;
  const float vx = fmaf(tr, dx, -r[0]) - r[4];
  const float vy = fmaf(tr, dy, -r[1]) - r[5];
  const float vz = fmaf(tr, dz, -r[2]) - r[6];
  const float a3 = fmaf(vx, ux, fmaf(vy, uy, vz * uz));
  const float wx = fmaf(-a3, ux, vx), wy = fmaf(-a3, uy, vy), wz = fmaf(-a3, uz, vz);
  const float rho2 = fmaf(wx, wx, fmaf(wy, wy, wz * wz));
  // t_side carries the rounding of the perpendicular part of d (large when the ray is close
  // to the axis); the linear term B of the side quadratic re-centres the chord exactly
  const float B = fmaf(wx, px, fmaf(wy, py, wz * pz));
  // near-parallel rays drop the linear term: a zero in place of 1/A (selects, no branch;
  // B is finite, so B * 0 = 0 and the values equal the parallel case's exactly)
  const float invA_s = par ? 0.0f : invA;
  const float cc = -B * invA_s;
  const float h2 = fmaf(B, B * invA_s, r[3] - rho2);
  const float hs = par ? INFINITY : fast_sqrt(fmaxf(h2, 0.0f) * invA);
  // slab 0 <= s <= L as offsets from t_r.  A ray perpendicular to the axis (da == 0) needs no
  // case of its own: 1/da is infinite, so the offsets are -inf and +inf inside the slab and
  // both +inf or both -inf outside it (only a ray exactly in a cap plane, a zero-margin
  // pixel, gives 0 * inf; min and max then drop it and the ray misses).
  const float d0 = -a3 * inv_da, d1 = (L - a3) * inv_da;
  const float din = fminf(d0, d1), dout = fmaxf(d0, d1);
  const float tin = fmaxf(cc - hs, din), tout = fminf(cc + hs, dout);
  h.ok = (h2 >= 0.0f) & (tin <= tout);
  h.t = tr + tin;
  if (MRG) h.m = cylinder_margin(r, par, A, B, rho2, h2, invA, cc, a3, da, inv_da);
  if (GRAD) {
    // entry point relative to p0 and the outward normal of the entry surface
    const bool cap = din > cc - hs;
    h.rx = fmaf(tin, dx, vx);
    h.ry = fmaf(tin, dy, vy);
    h.rz = fmaf(tin, dz, vz);
    const float sgn = da > 0.0f ? -1.0f : 1.0f;
    h.nx = cap ? sgn * ux : fmaf(tin, px, wx);
    h.ny = cap ? sgn * uy : fmaf(tin, py, wy);
    h.nz = cap ? sgn * uz : fmaf(tin, pz, wz);
  }
}

// Closed truncated cone: radius R(s) = r0 + k s on 0 <= s <= L.  As for the cylinder, the
// reference parameter t_r is the closest approach to the axis and every quantity is an offset
// from it.  With w, p the perpendicular parts of the offset and of d, a3 the axial coordinate
// at t_r and R0 = r0 + k a3, the side condition |w + tau p|^2 <= (R0 + k d_a tau)^2 is
// alpha tau^2 + 2 beta tau + gamma <= 0 with alpha = A - (k d_a)^2, beta = B - k d_a R0,
// gamma = rho^2 - R0^2.  For alpha >= 0 its solutions are the interval between the roots;
// for alpha < 0 (a ray steeper than the cone's flank) they are the two rays outside the roots,
// of which the slab meets at most one (the solid is convex).  The roots come from
// q = -(beta + sign(beta) sqrt(disc)), tau = q / alpha and gamma / q, finite as alpha -> 0.
template <bool GRAD, bool MRG = false>
__device__ __forceinline__ void cone_test(const float* r, float dx, float dy, float dz,
                                          float dd, Hit& h) {
  const float ux = r[8], uy = r[9], uz = r[10], L = r[7], r0 = r[3], k = r[11];
  const float da = fmaf(dx, ux, fmaf(dy, uy, dz * uz));
  const float px = fmaf(-da, ux, dx), py = fmaf(-da, uy, dy), pz = fmaf(-da, uz, dz);
  const float A = fmaf(px, px, fmaf(py, py, pz * pz));
  const bool par = A < 1.0e-6f * dd;
  const float inv_da = fast_rcp(da);
  const float t_side = fmaf(px, r[0], fmaf(py, r[1], pz * r[2])) * fast_rcp(A);
  const float cu = fmaf(r[0], ux, fmaf(r[1], uy, r[2] * uz));
  const float t_mid = (cu + 0.5f * L) * inv_da;
  const float tr = par ? t_mid : t_side;
  const float vx = fmaf(tr, dx, -r[0]) - r[4];
  const float vy = fmaf(tr, dy, -r[1]) - r[5];
  const float vz = fmaf(tr, dz, -r[2]) - r[6];
  const float a3 = fmaf(vx, ux, fmaf(vy, uy, vz * uz));
  const float wx = fmaf(-a3, ux, vx), wy = fmaf(-a3, uy, vy), wz = fmaf(-a3, uz, vz);
  const float rho2 = fmaf(wx, wx, fmaf(wy, wy, wz * wz));
  const float B = fmaf(wx, px, fmaf(wy, py, wz * pz));
  const float R0 = fmaf(k, a3, r0);
  const float kd = k * da;
  const float alpha = fmaf(-kd, kd, A);
  const float beta = fmaf(-kd, R0, B);
  const float gamma = fmaf(-R0, R0, rho2);
  const float disc = fmaf(beta, beta, -alpha * gamma);
  const float sq = fast_sqrt(fmaxf(disc, 0.0f));
  const float q = -(beta + copysignf(sq, beta));
  const float ra = q / alpha, rb = gamma / q;
  const float lo = fminf(ra, rb), hi = fmaxf(ra, rb);
  // slab 0 <= s <= L as offsets from t_r
  const float d0 = -a3 * inv_da, d1 = (L - a3) * inv_da;   // infinite for da == 0, as above
  const float din = fminf(d0, d1), dout = fmaxf(d0, d1);
  const bool has = disc >= 0.0f;
  float tin;
  bool side;
  if (alpha >= 0.0f) {
    tin = fmaxf(lo, din);
    side = lo >= din;
    h.ok = has & (tin <= fminf(hi, dout));
  } else {
    // outside the roots: the piece below lo, else the piece above hi
    const bool first = !has | (din <= fminf(dout, lo));
    const float t2 = fmaxf(din, hi);
    tin = first ? din : t2;
    side = !first & (hi >= din);
    h.ok = first ? (din <= dout) : (t2 <= dout);
  }
  h.t = tr + tin;
  if (MRG) {
    // the oracle's cone margin: disc / (|alpha| r_max^2) for the side (slack at each root the
    // least of it and the axial slacks), the caps' disc slacks with their own radii
    const float r1 = fmaf(k, L, r0), rmax2 = fmaxf(r0 * r0, r1 * r1);
    const float dsl = alpha != 0.0f ? disc / (fabsf(alpha) * rmax2) : INFINITY;
    const float s_a = fmaf(ra, da, a3), s_b = fmaf(rb, da, a3);
    const float c0 = -a3 * inv_da, c1 = (L - a3) * inv_da;
    const float q0 = fmaf(c0, fmaf(c0, A, 2.0f * B), rho2);
    const float q1 = fmaf(c1, fmaf(c1, A, 2.0f * B), rho2);
    const bool axial = da != 0.0f;
    const float iL = 1.0f / L;
    const bool fa = isfinite(ra), fb = isfinite(rb);
    const float sla = fa ? fminf(dsl, fminf(s_a * iL, (L - s_a) * iL)) : -INFINITY;
    const float slb = fb ? fminf(dsl, fminf(s_b * iL, (L - s_b) * iL)) : -INFINITY;
    const float side = has ? fmaxf(sla, slb) : ((fa || fb) ? dsl : -INFINITY);
    h.m = fmaxf(fmaxf(side, axial ? (r0 * r0 - q0) / (r0 * r0) : -INFINITY),
                axial ? (r1 * r1 - q1) / (r1 * r1) : -INFINITY);
  }
  if (GRAD) {
    h.rx = fmaf(tin, dx, vx);
    h.ry = fmaf(tin, dy, vy);
    h.rz = fmaf(tin, dz, vz);
    // side normal: perpendicular offset minus k R(s) along the axis; caps: -/+ u
    const float Rt = fmaf(kd, tin, R0);
    const float sgn = da > 0.0f ? -1.0f : 1.0f;
    h.nx = side ? fmaf(-k * Rt, ux, fmaf(tin, px, wx)) : sgn * ux;
    h.ny = side ? fmaf(-k * Rt, uy, fmaf(tin, py, wy)) : sgn * uy;
    h.nz = side ? fmaf(-k * Rt, uz, fmaf(tin, pz, wz)) : sgn * uz;
  }
}

// Closed elliptic cylinder: the side is x^T Q x <= 1 for the offset x from the first cap
// centre (Q = ex ex^T / a^2 + ey ey^T / b^2, Q u = 0), intersected with the slab 0 <= s <= L.
// The reference parameter is the closest approach to the axis in the Q metric.
template <bool GRAD, bool MRG = false>
__device__ __forceinline__ void ecylinder_test(const float* r, float dx, float dy, float dz,
                                               float dd, Hit& h) {
  const float q00 = r[3], q01 = r[7], q02 = r[8], q11 = r[9], q12 = r[10], q22 = r[11];
  const float ux = r[16], uy = r[17], uz = r[18], L = r[19];
  const float qdx = fmaf(q00, dx, fmaf(q01, dy, q02 * dz));
  const float qdy = fmaf(q01, dx, fmaf(q11, dy, q12 * dz));
  const float qdz = fmaf(q02, dx, fmaf(q12, dy, q22 * dz));
  const float dqd = fmaf(dx, qdx, fmaf(dy, qdy, dz * qdz));
  const float da = fmaf(dx, ux, fmaf(dy, uy, dz * uz));
  const bool par = dqd < 1.0e-6f * dd * (q00 + q11 + q22);
  const float inv = fast_rcp(dqd);
  const float inv_da = fast_rcp(da);
  const float cqd = fmaf(r[0], qdx, fmaf(r[1], qdy, r[2] * qdz));
  const float cu = fmaf(r[0], ux, fmaf(r[1], uy, r[2] * uz));
  const float tr = par ? (cu + 0.5f * L) * inv_da : cqd * inv;
  const float vx = fmaf(tr, dx, -r[0]) - r[4];
  const float vy = fmaf(tr, dy, -r[1]) - r[5];
  const float vz = fmaf(tr, dz, -r[2]) - r[6];
  const float qvx = fmaf(q00, vx, fmaf(q01, vy, q02 * vz));
  const float qvy = fmaf(q01, vx, fmaf(q11, vy, q12 * vz));
  const float qvz = fmaf(q02, vx, fmaf(q12, vy, q22 * vz));
  const float vqv = fmaf(vx, qvx, fmaf(vy, qvy, vz * qvz));
  const float B = fmaf(vx, qdx, fmaf(vy, qdy, vz * qdz));
  const float inv_s = par ? 0.0f : inv;     // as for the cylinder: selects, no branch
  const float cc = -B * inv_s;
  const float m = fmaf(B, B * inv_s, 1.0f - vqv);
  const float hs = par ? INFINITY : fast_sqrt(fmaxf(m, 0.0f) * inv);
  const float a3 = fmaf(vx, ux, fmaf(vy, uy, vz * uz));
  const float d0 = -a3 * inv_da, d1 = (L - a3) * inv_da;   // infinite for da == 0, as above
  const float din = fminf(d0, d1), dout = fmaxf(d0, d1);
  const float tin = fmaxf(cc - hs, din), tout = fminf(cc + hs, dout);
  h.ok = (m >= 0.0f) & (tin <= tout);
  h.t = tr + tin;
  if (MRG) {
    // in the unit-radius frame of the Q metric: radius^2 at offset tau is
    // vQv + 2 tau B + tau^2 dQd
    const float hsf = fast_sqrt(fmaxf(m, 0.0f) * inv);
    const float sa = fmaf(cc - hsf, da, a3), sb = fmaf(cc + hsf, da, a3);
    const float c0 = -a3 * inv_da, c1 = (L - a3) * inv_da;
    const float q0 = fmaf(c0, fmaf(c0, dqd, 2.0f * B), vqv);
    const float q1 = fmaf(c1, fmaf(c1, dqd, 2.0f * B), vqv);
    const bool axial = da != 0.0f;
    h.m = capped_margin(par ? -INFINITY : m, !par && m >= 0.0f, sa, sb, L,
                        axial ? 1.0f - q0 : -INFINITY, axial ? 1.0f - q1 : -INFINITY);
  }
  if (GRAD) {
    const bool cap = din > cc - hs;
    h.rx = fmaf(tin, dx, vx);
    h.ry = fmaf(tin, dy, vy);
    h.rz = fmaf(tin, dz, vz);
    const float sgn = da > 0.0f ? -1.0f : 1.0f;
    h.nx = cap ? sgn * ux : fmaf(tin, qdx, qvx);
    h.ny = cap ? sgn * uy : fmaf(tin, qdy, qvy);
    h.nz = cap ? sgn * uz : fmaf(tin, qdz, qvz);
  }
}

// ------------------------------------------------------------------------------------
// wave-uniform values: read once from lane 0 into scalar registers, so that the per-tile
// bookkeeping runs on the scalar unit and holds no vector registers

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float uni(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
template <class T>
__device__ __forceinline__ T* uni(T* x) {
  const uint64_t v = reinterpret_cast<uint64_t>(x);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}
// Walks a particle's tiles (the union of its rectangles, each row-major) in steps of the
// number of wavefronts per workgroup, without a division per tile.
using PInfoPtr = const __attribute__((address_space(4))) PInfo*;

__device__ __forceinline__ int4 load_rect(PInfoPtr pi, int r) {
  const __attribute__((address_space(4))) int* q =
      (const __attribute__((address_space(4))) int*)pi + 4 * r;   // rect is the first member
  return make_int4(q[0], q[1], q[2], q[3]);
}
// (a header in LDS)
__device__ __forceinline__ int4 load_rect(const PInfo* pi, int r) {
  const int4 q = pi->rect[r];
  return make_int4(uni(q.x), uni(q.y), uni(q.z), uni(q.w));
}

template <class Ptr>
struct TileWalk {
  Ptr pi;
  int n, ri, rx, ry, rw, rh, ox, oy;

  __device__ void load(int r) {
    const int4 q = load_rect(pi, r);
    rx = q.x;
    ry = q.y;
    rw = q.z;
    rh = q.w;
  }
  // position at tile t of the union
  __device__ void seek(int t) {
    while (t >= rw * rh && ri + 1 < n) {
      t -= rw * rh;
      load(++ri);
    }
    oy = t / rw;
    ox = t - oy * rw;
  }
  __device__ void start(Ptr p, int n_rects, int t) {
    pi = p;
    n = n_rects;
    ri = 0;
    load(0);
    seek(t);
  }
  __device__ void step(int s) {
    ox += s;
    while (ox >= rw) {
      ox -= rw;
      ++oy;
    }
    if (oy >= rh && ri + 1 < n) {
      const int t = (oy - rh) * rw + ox;
      load(++ri);
      seek(t);
    }
  }
  __device__ int tx() const { return rx + ox; }
  __device__ int ty() const { return ry + oy; }
};

// ------------------------------------------------------------------------------------
// persistent ray cast + cost terms + reduction

// Work items.  A launch of fewer particles than resident workgroups splits every particle into
// equal parts, one item per workgroup (the host chooses parts = resident workgroups / particles,
// rounded down).  Workgroups are dispatched to the chip's 8 XCDs round-robin (workgroup b on XCD
// b mod 8), each XCD with its own L2; an item is taken XCD-major, so that the parts of one
// particle (and the tables they stage) stay on one XCD.  A bijection of 0 .. G-1.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_major_item(int b, int G) {
  const int q = G / kXcds, rem = G % kXcds;
  const int x = b % kXcds, j = b / kXcds;
  return x * q + min(x, rem) + j;
}

// A larger launch takes whole particles, from kQueues queues, one per XCD: queue q holds the
// particles r with r mod kQueues = q (every frame of a batch is spread over all queues) and is
// worked off by the workgroups b with b mod kQueues = q.  A workgroup's first particle follows
// from its index, later ones come from its queue's counter.  Nothing but speed depends on
// where a workgroup runs.  (A static stride left the launch waiting on its slowest workgroup:
// 65536 poses of a 320x240 frame 3.42 ms against 2.75 ms; one counter for the launch cost about
// 20 ns per item, one after another on the one address: 4096 poses of 64 uneven frames 119 us
// against 99 us.)

// Gradient launches of at most kSelfSched particles build their work list in every wavefront of
// the ray cast (no work-list launch, no barrier): lane l holds the tile counts of particles
// 4l .. 4l + 3, two wavefront sums and a scan give the items.  Workgroup 0 stores the item
// offsets for the kernels that assemble the evaluation and adds the launch's evaluations to the
// counts.
constexpr int kSelfSched = 4 * kWave;
static_assert(kSelfSched == kSelfSchedMax, "four particles per lane");

struct WaveList {
  int off;       // offset of the lane's first particle's items
  int cnt[4];    // items of the lane's particles
  int total, tpi;
  bool interleave;

  // (first wavefront: the offsets also go to LDS, for load() after the next barrier)
  __device__ void build(const EvalArgs& a, const Workspace& ws, int lane, int* s_off) {
    const int n = a.n_frames * a.n_particles;
    int v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ws.tiles[src_of(a, min(4 * lane + j, n - 1))];
    int tiles = 0, evaluated = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = 4 * lane + j < n ? v[j] : -1;
      tiles += max(v[j], 0);
      evaluated += v[j] >= 0 ? 1 : 0;
    }
    tiles = uni(wave_sum(tiles));
    tpi = tiles_per_item(a, tiles);
    int mine = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cnt[j] = (max(v[j], 0) + tpi - 1) / tpi;
      mine += cnt[j];
    }
    int incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    off = incl - mine;
    total = __builtin_amdgcn_readlane(incl, kWave - 1);
    interleave = interleaved(a, total);
    if (threadIdx.x < kWave) {
      int o = off;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s_off[4 * lane + j] = o;
        if (blockIdx.x == 0 && 4 * lane + j < n) ws.item_off[4 * lane + j] = o;
        o += cnt[j];
      }
      if (lane == 0) s_off[kSelfSched] = total;
    }
    if (blockIdx.x == 0 && threadIdx.x < kWave) {
      evaluated = wave_sum(evaluated);
      if (lane == 0) {
        ws.item_off[n] = total;
        if (a.eval_count)
          atomicAdd(&a.eval_count[kCountSlots], (unsigned long long)evaluated);
      }
    }
  }
  // the lane's part again (the registers are not held over an item's tiles)
  __device__ __forceinline__ void load(const int* s_off, int lane) {
    int o[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) o[j] = s_off[4 * lane + j];
    off = o[0];
#pragma unroll
    for (int j = 0; j < 4; ++j) cnt[j] = o[j + 1] - o[j];
  }
  // the evaluated particle of an item, its first item and item count (wave-uniform)
  __device__ __forceinline__ int find(int item, int& first, int& n_it) const {
    int o = off, r = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t m = __builtin_amdgcn_ballot_w64(o <= item) &
                         __builtin_amdgcn_ballot_w64(item < o + cnt[j]);
      if (m) {
        const int l = __builtin_ctzll(m);
        r = 4 * l + j;
        first = __builtin_amdgcn_readlane(o, l);
        n_it = __builtin_amdgcn_readlane(cnt[j], l);
      }
      o += cnt[j];
    }
    return r;
  }
};

// What the tile loop needs of a particle's header, wave-uniform.
struct Head {
  int n_rects, n_tiles, TW, W;
  float sx, sy, sz, cx, cy, bg;
  const uint32_t* words;
  const float* tile_td;
  const int* tile_skin;
  const uint8_t* grad_mask;

  __device__ __forceinline__ explicit Head(PInfoPtr p)
      : n_rects(p->n_rects), n_tiles(p->n_tiles), TW(p->TW), W(p->W), sx(p->sx), sy(p->sy),
        sz(p->sz), cx(p->cx), cy(p->cy), bg(p->bg), words(p->words), tile_td(p->tile_td),
        tile_skin(p->tile_skin), grad_mask(p->grad_mask) {}
  // (a header in LDS)
  __device__ __forceinline__ explicit Head(const PInfo* p)
      : n_rects(uni(p->n_rects)), n_tiles(uni(p->n_tiles)), TW(uni(p->TW)), W(uni(p->W)),
        sx(uni(p->sx)), sy(uni(p->sy)), sz(uni(p->sz)), cx(uni(p->cx)), cy(uni(p->cy)),
        bg(uni(p->bg)), words(uni(p->words)), tile_td(uni(p->tile_td)),
        tile_skin(uni(p->tile_skin)), grad_mask(nullptr) {}
};

// Bound by the issue of vector instructions (65536 poses of a 320x240 frame: 1.84e9 of them, one
// every 3.2 cycles and SIMD, every cycle of the launch).  A multiply-add of vector registers takes
// 2.5 cycles, a comparison, select, minimum, conversion, FP64 or DPP instruction or one with a scalar
// operand 4.1, a transcendental 8 to 19, so the code around the tests counts those: boxes compared by
// distance from their centre (2 subtractions and 2 comparisons for 4), the nearest entry and the
// background plane by integer minimum, one comparison per match term.  65536 poses 2600 to 2440
// us, 1024 two-hand poses 128.0 to 120.7 us.  Fewer scalar instructions alone do not help: culling
// 16 tiles at a time (a lane per tile and quarter of the primitives) took 18 % of them away, added
// 5 % vector instructions, and 65536 poses took 2660 us.
//
// One wavefront's tiles t0, t0 + stride, ... below t_end of a particle whose tables are in LDS
// (s_tab): ray cast, cost terms and, for a gradient, the wrench rows wr ([segment][16-lane
// row][6], this wavefront's).  Adds the clamped depth terms to acc_td (per lane), the tiles'
// background depth sums to acc_bg (the same on every lane) and the match counts, less the
// background's, to acc_a and acc_o (wavefront totals).
template <bool GRAD, bool DEBUG, int NT, class Ptr>
__device__ __forceinline__ void cast_tiles(const EvalArgs& a, const TypeMasks& tm,
                                           const float4* s_tab, Ptr pi, const Head& hd, int t0,
                                           int stride, int t_end, int lane, int r, float* wr,
                                           double& acc_td, double& acc_bg, int& acc_a,
                                           int& acc_o) {
  const int n_prim = a.n_prim;
  const Tables L(n_prim);
  const float4* s_box = s_tab + L.box;
  const float4* s_cap = s_tab + L.cap;
  const float2* s_capr = reinterpret_cast<const float2*>(s_tab + L.capr);
  const float* recs = reinterpret_cast<const float*>(s_tab);
  // the lane's pixel offset within a tile as a ray component: ((lane & 7) - cx) sx and
  // ((lane >> 3) - cy) sy, so that a tile's rays cost one multiply-add per component
  const float lane_dx = ((float)(lane & 7) - hd.cx) * hd.sx;
  const float lane_dy = ((float)(lane >> 3) - hd.cy) * hd.sy;
  const float dz = hd.sz, dz2 = hd.sz * hd.sz;
  // depth of a hidden entry: the background plane, or none
  const float plane = hd.bg > 0.0f ? hd.bg : INFINITY;
  // gradient: the lane's place in the fold of a row's sums (below)
  const bool odd = lane & 1, odd2 = lane & 2, upper = lane & 8;
  const bool writer = (lane & 4) == 0 && (lane & 10) != 10;
  const int wr_lane = (lane >> 4) * 6 + (upper ? 4 : 0) + (lane & 3);
  TileWalk<Ptr> walk;
  if (t0 < t_end) walk.start(pi, hd.n_rects, t0);
  for (int t = t0; t < t_end; t += stride, walk.step(stride)) {
    const int tx = walk.tx(), ty = walk.ty();
    const int x0 = tx * kTile, y0 = ty * kTile;
    const float x0f = (float)x0, y0f = (float)y0;
    // culling, one lane per primitive: screen box overlap, then the distance of the tile's
    // centre from the primitive's image segment
    // (the three loads are issued together, the index clamped, so no branch waits on LDS;
    // the segment test runs only where some lane's box overlaps; the second half is skipped
    // outright for models of at most 64 primitives)
    uint64_t mk[2] = {0ull, 0ull};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half * kWave >= n_prim) break;
      const int k = lane + half * kWave;
      const int kk = min(k, n_prim - 1);
      const float4 b = s_box[kk];
      const float4 cp = s_cap[kk];
      const float2 cq = s_capr[kk];
      // one ballot per comparison, combined on the scalar unit with the half's primitive
      // lanes (a ballot of the combined condition routes its lane mask through a vector
      // register and back)
      const int left = n_prim - half * kWave;
      uint64_t m = (left >= kWave ? ~0ull : (1ull << left) - 1ull) &
                   __builtin_amdgcn_ballot_w64(fabsf(x0f - b.x) <= b.y) &
                   __builtin_amdgcn_ballot_w64(fabsf(y0f - b.z) <= b.w);
      if (m) {
        // on every lane (a uniform branch), the result a lane mask combined on the scalar
        // unit: no per-lane branch whose outcome would go through a vector register
        // tile centre (x0 + 3.5, y0 + 3.5) minus the first disc's centre (cp: less 3.5)
        const float wx = x0f - cp.x, wy = y0f - cp.y;
        const float sp = fminf(fmaxf(fmaf(wx, cp.z, wy * cp.w) * cq.x, 0.0f), 1.0f);
        const float ex = fmaf(-sp, cp.z, wx), ey = fmaf(-sp, cp.w, wy);
        m &= __builtin_amdgcn_ballot_w64(fmaf(ex, ex, ey * ey) <= cq.y);
      }
      mk[half] = m;
    }
    if ((mk[0] | mk[1]) == 0ull) continue;

    const int tile_idx = ty * hd.TW + tx;
    const int u = x0 + (lane & 7), v = y0 + (lane >> 3);
    const uint32_t word = global_ptr(hd.words)[(size_t)tile_idx * kTilePx + lane];
    // the tile's background sums, loaded with the words (one address for every lane) so
    // that their latency overlaps the tests; lane 0 subtracts them after the tests
    const float bg_td = global_ptr(hd.tile_td)[tile_idx];
    const int bg_sk = global_ptr(hd.tile_skin)[tile_idx];
    // (a pixel outside the image is 0, so the skin bit stands on valid pixels only)
    const bool valid = word >= kValidBit;
    const float od = (float)(word & 0xFFFFu);
    const bool os = word >= (kValidBit | kSkinBit);
    const float dx = fmaf(x0f, hd.sx, lane_dx);
    const float dy = fmaf(y0f, hd.sy, lane_dy);
    const float dd = fmaf(dx, dx, fmaf(dy, dy, dz2));
    const float inv_dd = fast_rcp(dd);
    float tmin = INFINITY;
    int win = -1;   // tracked for the gradient and the debug images only
    float wnx = 0, wny = 0, wnz = 0, wrx = 0, wry = 0, wrz = 0;
    float wm = -INFINITY, mmax = -INFINITY;   // margins (debug images only)

#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int typ = 0; typ < NT; ++typ) {
        uint64_t m = mk[half] & tm.m[typ][half];
        while (m) {
          const int k = __builtin_ctzll(m) + half * kWave;
          m &= m - 1;
          const float* r = recs + k * kRec;
          Hit h;
          if (typ == HT_SPHERE) sphere_test<GRAD, DEBUG>(r, dx, dy, dz, inv_dd, h);
          else if (typ == HT_CYLINDER) cylinder_test<GRAD, DEBUG>(r, dx, dy, dz, dd, h);
          else if (typ == HT_ELLIPSOID) ellipsoid_test<GRAD, DEBUG>(r, dx, dy, dz, h);
          else if (typ == HT_CONE) cone_test<GRAD, DEBUG>(r, dx, dy, dz, dd, h);
          else ecylinder_test<GRAD, DEBUG>(r, dx, dy, dz, dd, h);
          // nearest entry in front of the camera: as unsigned integers the bit patterns of
          // non-negative floats keep their order and negative ones (entries behind the
          // camera) exceed +inf; exact ties keep the first tested (branch-free selects)
          if (!GRAD && !DEBUG) {
            const float t = h.ok ? h.t : INFINITY;
            tmin = __uint_as_float(min(__float_as_uint(t), __float_as_uint(tmin)));
            continue;
          }
          const bool take = h.ok & (__float_as_uint(h.t) < __float_as_uint(tmin));
          tmin = take ? h.t : tmin;
          if (GRAD || DEBUG) win = take ? k : win;
          if (DEBUG) {
            // the nearest primitive's margin, and the largest of the tested ones (misses)
            wm = take ? h.m : wm;
            mmax = fmaxf(mmax, h.m);
          }
          if (GRAD) {
            wnx = take ? h.nx : wnx;
            wny = take ? h.ny : wny;
            wnz = take ? h.nz : wnz;
            wrx = take ? h.rx : wrx;
            wry = take ? h.ry : wry;
            wrz = take ? h.rz : wrz;
          }
        }
      }
    }
    // depth of the nearest entry (without one infinite); behind the background plane it is
    // hidden
    const float zmin = tmin * dz;
    const bool any = __float_as_uint(tmin) < 0x7F800000u;
    const bool hit = zmin < plane;
    if (GRAD || DEBUG) win = hit ? win : -1;
    float rd = fminf(zmin, plane);
    if (!(hd.bg > 0.0f)) rd = hit ? rd : 0.0f;
    const float diff = fabsf(od - rd);
    float td = fminf(diff, kDClamp);
    td = valid ? td : 0.0f;
    // (kept in FP32 up to here: the select would be moved behind the conversion, where it takes
    // two instructions)
    asm("" : "+v"(td));
    acc_td += (double)td;
    // one ballot per comparison, combined on the scalar unit
    const uint64_t m_valid = __builtin_amdgcn_ballot_w64(valid);
    const uint64_t m_os = __builtin_amdgcn_ballot_w64(os);
    const uint64_t m_rm = __builtin_amdgcn_ballot_w64(hit) &
                          (__builtin_amdgcn_ballot_w64(diff < kDMatch) |
                           __builtin_amdgcn_ballot_w64(od == 0.0f));
    acc_a += __builtin_popcountll(m_os & m_rm);
    acc_o += __builtin_popcountll(m_valid & (m_os | m_rm));
    {
      // read back here (a convergent read, so the wait for the loads stays after the tests)
      const int bgs = __builtin_amdgcn_readfirstlane(bg_sk);
      acc_bg += (double)bg_td;
      acc_o -= bgs;
    }
    // the debug images have the host's W x H of the debug slot; a frame slot of another
    // size would write past them, so stores outside that extent are dropped
    if (DEBUG && valid && u < a.dbg_W && v < a.dbg_H) {
      const size_t pix = ((size_t)r * a.dbg_H + v) * a.dbg_W + u;
      if (a.dbg.depth) a.dbg.depth[pix] = rd;
      if (a.dbg.hit) a.dbg.hit[pix] = hit ? 1 : 0;
      if (a.dbg.rm) a.dbg.rm[pix] = m_rm >> lane & 1 ? 1 : 0;
      if (a.dbg.winner) a.dbg.winner[pix] = win;
      if (a.dbg.margin) a.dbg.margin[pix] = any ? wm : mmax;
    }
    if (GRAD) {
      // adjoint: coefficient of the depth term, then the per-segment wrench
      bool act = valid && hit && diff < kDClamp && od != rd;
      // the call's mask (one frame), else the frame's slot mask
      const uint8_t* gmask = a.pixel_mask ? a.pixel_mask : hd.grad_mask;
      if (act && gmask) act = global_ptr(gmask)[(size_t)v * hd.W + u] != 0;
      int seg = -1;
      float kap = 0.0f;
      float mx = 0, my = 0, mz = 0;
      if (act) {
        const float* r = recs + win * kRec;
        seg = __float_as_int(r[15]);
        const float nd = fmaf(wnx, dx, fmaf(wny, dy, wnz * dz));
        // (the hardware reciprocal: a quotient would expand into a range-safe sequence of
        // ten instructions; nd is a dot product of normal and ray, far from the range ends)
        kap = ((rd > od ? dz : -dz)) * fast_rcp(nd);
        // lever arm from the segment origin: (entry - ref) + (ref - origin)
        const float lx = wrx + r[12], ly = wry + r[13], lz = wrz + r[14];
        mx = kap * (ly * wnz - lz * wny);
        my = kap * (lz * wnx - lx * wnz);
        mz = kap * (lx * wny - ly * wnx);
      }
      const float fx = kap * wnx, fy = kap * wny, fz = kap * wnz;
      // Segments present in this tile, one at a time (uniform loop): the six components' sums
      // over each 16-lane row, folded so that lanes share the work.  The first step adds
      // neighbours and leaves one component of a pair on the even and the other on the odd
      // lanes (what a lane keeps and what it hands over are chosen before the loop), the second
      // leaves four components on a quad's lanes, and the last joins both packed values: lanes
      // 0 to 3 and 8, 9 of a row hold its six sums and one LDS atomic adds them to the row's
      // accumulators (distinct addresses, a wavefront's adds in program order: deterministic).
      // Each component's lanes are added in one order: neighbours, halves of a quad, quads 0 and 3
      // and 1 and 2, the two pairs.  12 vector operations on sums and one atomic a segment and
      // tile, where six full row totals took 24 and six (two-hand refined generation of 1024
      // poses 318 us with those, 314 us folded; gradients of 256 poses 52.7 and 51.2 us).
      const float keep[3] = {odd ? my : mx, odd ? fx : mz, odd ? fz : fy};
      const float give[3] = {odd ? mx : my, odd ? mz : fx, odd ? fy : fz};
      uint64_t left = __builtin_amdgcn_ballot_w64(act);
      while (left) {
        const int s = __builtin_amdgcn_readlane(seg, __builtin_ctzll(left));
        const bool mine = seg == s;
        left &= ~__builtin_amdgcn_ballot_w64(mine);
        float v[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
          v[q] = (mine ? keep[q] : 0.0f) + dpp<0xB1>(mine ? give[q] : 0.0f);
        float e = (odd2 ? v[1] : v[0]) + dpp<0x4E>(odd2 ? v[0] : v[1]);
        float f = v[2] + dpp<0x4E>(v[2]);
        e += dpp<0x124>(e);
        f += dpp<0x124>(f);
        const float sum = (upper ? f : e) + dpp<0x128>(upper ? e : f);
        if (writer) atomicAdd(wr + s * 24 + wr_lane, sum);
      }
    }
  }
}

// NT: primitive types the model uses (3: spheres, cylinders, ellipsoids; kNumTypes: also
// cones and elliptic cylinders), so a model without the latter keeps the smaller register
// footprint.  The forward cast asks for eight wavefronts per SIMD, the gradient cast for six (80
// vector registers, about ten spilled around the tile loop): six workgroups per CU take a small
// launch's items, a few more than its nominal grid of five, in one round, where five leave the
// last ones to a second round (two-hand refined generation 304 us with five, 296 us with six, 299
// us with seven; gradients of 128 two-hand poses 48.2, 45.3 and 46.8 us).  SELF: the wavefronts
// build the work list (at most kSelfSched particles).
template <bool GRAD, bool DEBUG, int NT, bool SELF>
__global__ __attribute__((amdgpu_flat_work_group_size(1, kBlock),
                          amdgpu_waves_per_eu(GRAD ? 6 : DEBUG ? 1 : 8)))
void raycast_kernel(EvalArgs a, Workspace ws, TypeMasks tm) {
  static_assert(!(GRAD && DEBUG) && !(SELF && !GRAD), "forward, debug or gradient");
  // the particle's tables, then (gradient) the wrench rows: per wavefront, segment and 16-lane
  // row the six wrench components of the item
  extern __shared__ float4 s_tab[];
  __shared__ int s_next[2];
  __shared__ double s_td[2][kWavesPerBlock];
  __shared__ int s_a[2][kWavesPerBlock], s_o[2][kWavesPerBlock];

  // the wavefront index as a scalar, so that the tile walk, the tile's coordinates and the
  // observation addresses are wave-uniform (scalar instructions)
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_seg = a.n_seg;
  const Tables L(a.n_prim);
  float* s_wr = reinterpret_cast<float*>(s_tab + L.words);   // [wave][seg][row][6]
  const int parts = a.parts;
  const int G = gridDim.x, n_eval = a.n_frames * a.n_particles;
  // Forward: whole particles from the queues, or the particle's parts, one per workgroup.
  // Gradient: the work list's items, one per workgroup or from the queues.
  __shared__ int s_off[SELF ? kSelfSched + 1 : 1];
  WaveList list;
  if constexpr (GRAD && SELF) {
    list.build(a, ws, lane, s_off);
  } else if constexpr (GRAD) {
    list.total = scalar_ptr(ws.list)[0];
    list.tpi = scalar_ptr(ws.list)[1];
    list.interleave = scalar_ptr(ws.list)[2] != 0;
  }
  const int units = GRAD ? list.total : n_eval;
  const bool queued = units > G;
  const int queue = blockIdx.x % kQueues;
  // workgroups of this queue, and the units it holds
  const int groups = (G - queue + kQueues - 1) / kQueues;
  const int held = (units - queue + kQueues - 1) / kQueues;
  int* counter = ws.counters + (a.src ? kCounterInts : 0) + queue * kQueueStride;
  int n_counted = 0;

  // (a gradient launch can have fewer items than workgroups: the first ones take them)
  const int end = queued ? held : GRAD ? units : n_eval * parts;
  int unit = queued ? (int)blockIdx.x / kQueues
                    : ((int)blockIdx.x < end ? xcd_major_item(blockIdx.x, end) : end);
  for (int round = 0; unit < end; ++round) {
    const int buf = round & 1;
    // the next unit is taken now, so that the atomic's latency passes under this one's work
    int next = end;
    if (queued && tid == 0) next = groups + atomicAdd(counter, 1);
    // evaluated particle; forward: its part; gradient: the item's place among the particle's
    const int item = queued ? unit * kQueues + queue : unit;
    int r, part = 0, first_item = 0, n_it = 1;
    if constexpr (GRAD && SELF) {
      if (round) list.load(s_off, lane);
      r = list.find(item, first_item, n_it);
    } else if constexpr (GRAD) {
      r = scalar_ptr(ws.item_map)[item];
      first_item = scalar_ptr(ws.item_off)[r];
      n_it = scalar_ptr(ws.item_off)[r + 1] - first_item;
    } else {
      r = item / parts;
      part = item - r * parts;
    }
    const int p = a.src ? uni(src_of(a, r)) : r;   // the workspace particle of its kinematics
    const PInfoPtr pi = scalar_ptr(ws.pinfo + p);
    const int n_tiles = pi->n_tiles;
    const bool skip = !GRAD && pi->skip != 0;   // (a skipped particle has no gradient items)
    if (!GRAD && part == 0 && !skip) ++n_counted;
    const bool on = !skip && (GRAD || part < active_parts(n_tiles, parts));
    if (on) {
    const float4* src = ws.tables + (size_t)p * L.words;
    for (int i = tid; i < L.words; i += kBlock) s_tab[i] = src[i];
    const Head hd(pi);
    if (GRAD) {
      float* wr = s_wr + wave * n_seg * 24;
      for (int i = lane; i < n_seg * 24; i += kWave) wr[i] = 0.0f;
    }
    __syncthreads();
    // tiles t0, t0 + stride, ... below t_end.  Gradient item c of a particle with n_it items:
    // tiles c tpi .. (c + 1) tpi - 1, or, when interleaved, c, c + n_it, c + 2 n_it, ...;
    // wavefront w takes every fourth of them
    const int c = item - first_item;
    const int gap = GRAD ? (list.interleave ? n_it : 1) : parts;
    const int stride = gap * kWavesPerBlock;
    const int t0 = GRAD ? (list.interleave ? c : c * list.tpi) + wave * gap
                        : part * kWavesPerBlock + wave;
    const int t_end = GRAD && !list.interleave ? min((c + 1) * list.tpi, n_tiles) : n_tiles;
    double acc_td = 0.0;   // exact: the FP32 terms are multiples of 2^-15 mm
    double acc_bg = 0.0;   // the tiles' background depth sums (the same on every lane)
    int acc_a = 0, acc_o = 0;   // wavefront totals: popcounts of lane masks (scalar unit)

    cast_tiles<GRAD, DEBUG, NT>(a, tm, s_tab, pi, hd, t0, stride, t_end, lane, r,
                                GRAD ? s_wr + wave * n_seg * 24 : nullptr, acc_td, acc_bg, acc_a,
                                acc_o);

    acc_td = wave_sum(acc_td) - acc_bg;
    if (lane == 0) {
      s_td[buf][wave] = acc_td;
      s_a[buf][wave] = acc_a;
      s_o[buf][wave] = acc_o;
    }
    }
    if (tid == 0) s_next[buf] = next;
    __syncthreads();
    if (on) {
      if (tid == 0) {
        const double td = ((s_td[buf][0] + s_td[buf][1]) + s_td[buf][2]) + s_td[buf][3];
        const int sa = s_a[buf][0] + s_a[buf][1] + s_a[buf][2] + s_a[buf][3];
        const int so = s_o[buf][0] + s_o[buf][1] + s_o[buf][2] + s_o[buf][3];
        if (!GRAD && a.direct) {
          // the whole particle: its cost follows here (no finalize launch)
          a.cost[r] = particle_cost(pi, td, sa, so);
        } else {
          ws.partial[item] = Partial{td, sa, so};
        }
      }
      if (GRAD) {
        for (int i = tid; i < n_seg * 6; i += kBlock) {
          const int s = i / 6, q = i % 6;
          float v = 0.0f;
#pragma unroll
          for (int w = 0; w < kWavesPerBlock; ++w) {
            const float* c = s_wr + (w * n_seg + s) * 24 + q;
            v += (c[0] + c[6]) + (c[12] + c[18]);
          }
          ws.wrench[(size_t)item * n_seg * 6 + i] = v;
        }
        __syncthreads();   // the rows are read before the next item clears them
      }
    }
    unit = uni(s_next[buf]);
  }
  if (!GRAD && tid == 0 && n_counted && a.eval_count)
    atomicAdd(&a.eval_count[blockIdx.x % kCountSlots], (unsigned long long)n_counted);
}

// ------------------------------------------------------------------------------------
// small forward launches: the whole evaluation in one launch

// The last part of a particle to finish writes its cost (small launches: 16 poses of a 64x64
// frame 13.0 to 12.0 us, a frame's ingest with one pose 57 to 54.5 us without a finalize launch;
// of the larger ones 256 poses of a 320x240 frame took 29.3 instead of 30.0 us, 200 of the
// paper's model 46.4 instead of 46.2, a two-hand refined generation 303.6 instead of 303.0, so
// they keep theirs).  Called by every lane of the workgroup's first wavefront with the part's
// sums, which are exact in any order.  A partial passes through agent-scope atomic stores, which
// write through this XCD's L2 and have reached memory once waited for; the part is counted after
// that wait, and the last part acquires before it reads.  (A release in place of the wait adds the
// write-back of the L2's other lines, none of which are read here, once a part: 256 poses of a
// 64x64 frame 18.8 us against 15.0 us.)
__device__ __forceinline__ void finish_part(const EvalArgs& a, const Workspace& ws, int r,
                                            int item, int n_parts, double td, int sa, int so,
                                            const PInfo& pi, int lane) {
  if (n_parts == 1) {
    if (lane == 0) a.cost[r] = particle_cost(&pi, td, sa, so);
    return;
  }
  int before = 0;
  if (lane == 0) {
    uint64_t* q = reinterpret_cast<uint64_t*>(ws.partial + item);
    __hip_atomic_store(q, (uint64_t)__double_as_longlong(td), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, (uint64_t)(uint32_t)so << 32 | (uint32_t)sa, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    before = __hip_atomic_fetch_add(a.done + r, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (uni(before) + 1 != n_parts) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  double d = 0.0;
  int ia = 0, io = 0;
  for (int i = lane; i < n_parts; i += kWave) {
    uint64_t* q = reinterpret_cast<uint64_t*>(ws.partial + (size_t)r * a.parts + i);
    const uint64_t q0 = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t q1 = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    d += __longlong_as_double(q0);
    ia += (int)(uint32_t)q1;
    io += (int)(uint32_t)(q1 >> 32);
  }
  d = wave_sum(d);
  ia = wave_sum(ia);
  io = wave_sum(io);
  if (lane == 0) a.cost[r] = particle_cost(&pi, d, ia, io);
}

// One workgroup per part of a particle: the kinematics (repeated in every part, on CUs that would
// be idle otherwise), its tables kept in LDS, then the part's tiles.  A chain of latencies (about
// 5 us of kinematics, 1 us per tile of a wavefront): against separate launches it saves one launch
// gap and the tables' way through memory, and a finalize launch where it writes the costs (16
// poses of a 64x64 frame 18.1 to 12.1 us, 64 of a 128x128 frame 18.2 to 13.2 us).  Workgroups of
// eight and sixteen wavefronts, with fewer parts, lost more to the barriers than they saved (15.8
// and 17.3 us against 14.9 with four, each with a finalize launch).
// FINISH: the costs are written here (else the partials are assembled by the next kernel).
template <int NT, bool FINISH>
__global__ __launch_bounds__(kBlock) void small_eval_kernel(EvalArgs a, Workspace ws,
                                                            TypeMasks tm) {
  extern __shared__ float4 s_tab[];
  __shared__ FkShared<1> sh;
  __shared__ PInfo s_head;
  __shared__ double s_td[kWavesPerBlock];
  __shared__ int s_a[kWavesPerBlock], s_o[kWavesPerBlock];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int parts = a.parts, n_total = a.n_frames * a.n_particles;
  const int item = blockIdx.x, r = item / parts, part = item - r * parts;
  if (FINISH && a.done_next && item == 0)
    for (int i = tid; i < a.done_ints; i += kBlock) a.done_next[i] = 0;
  const bool cast = fk_particle<kBlock, kWavesPerBlock>(
      a, ws, sh, r, 0, wave, lane, n_total, s_tab, [&](const PInfo& pi, int l) {
        if (l == 0) {
          s_head = pi;
          if (!FINISH && part == 0) ws.pinfo[r] = pi;
        }
      });
  if (!cast) return;   // (a skipped particle)
  __syncthreads();
  const Head hd(&s_head);
  double acc_td = 0.0, acc_bg = 0.0;
  int acc_a = 0, acc_o = 0;
  cast_tiles<false, false, NT>(a, tm, s_tab, &s_head, hd, part * kWavesPerBlock + wave,
                               parts * kWavesPerBlock, hd.n_tiles, lane, r, nullptr, acc_td, acc_bg,
                               acc_a, acc_o);
  acc_td = wave_sum(acc_td) - acc_bg;
  if (lane == 0) {
    s_td[wave] = acc_td;
    s_a[wave] = acc_a;
    s_o[wave] = acc_o;
  }
  __syncthreads();
  if (FINISH ? wave != 0 : tid != 0) return;
  const double td = ((s_td[0] + s_td[1]) + s_td[2]) + s_td[3];
  const int sa = s_a[0] + s_a[1] + s_a[2] + s_a[3];
  const int so = s_o[0] + s_o[1] + s_o[2] + s_o[3];
  if (!FINISH)
    ws.partial[item] = Partial{td, sa, so};
  else if (part < active_parts(hd.n_tiles, parts))
    finish_part(a, ws, r, item, active_parts(hd.n_tiles, parts), td, sa, so, s_head, lane);
  if (lane == 0 && part == 0 && a.eval_count)
    atomicAdd(&a.eval_count[blockIdx.x % kCountSlots], 1ull);
}

// ------------------------------------------------------------------------------------
// finalize: combine partials in item order, Eq. 4-5, and the kinematic adjoint

// This lane's partial among a particle's first 64 parts (items b .. b + parts - 1), loaded
// before the number of active parts is known: the index is clamped into the particle's items
// and the value is used only when its part is active.
__device__ __forceinline__ Partial first_partial(const Workspace& ws, int b, int parts, int lane) {
  return ws.partial[b + min(lane, parts - 1)];
}

// S_d, S_and, S_or of a particle: the ROI's background totals plus its items' partials,
// summed by the lanes of one wavefront (pr0: this lane's first_partial, loaded early by the
// caller).  Every depth term is a multiple of 2^-15 mm, so the FP64 sums are exact and equal
// to any other summation order.
__device__ inline void wave_partial_sums(double bg_td, double bg_or, const Workspace& ws, int b,
                                         int e, int lane, const Partial& pr0, double& S_d,
                                         long long& S_and, long long& S_or) {
  const bool in0 = b + lane < e;
  double d = in0 ? pr0.td : 0.0;
  int sa = in0 ? pr0.a : 0, so = in0 ? pr0.o : 0;
  for (int i = b + kWave + lane; i < e; i += kWave) {
    const Partial pr = ws.partial[i];
    d += pr.td;
    sa += pr.a;
    so += pr.o;
  }
  d = wave_sum(d);
  sa = wave_sum(sa);
  so = wave_sum(so);
  S_d = bg_td + d;
  S_and = sa;
  S_or = (long long)bg_or + so;
}

// Forward: one wavefront per particle.
__global__ __launch_bounds__(kBlock) void finalize_kernel(EvalArgs a, Workspace ws) {
  const int lane = threadIdx.x & (kWave - 1);
  // evaluated particle, wave-uniform (its record and item range are scalar loads)
  const int p = blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_total = a.n_frames * a.n_particles;
  if (p >= n_total) return;
  // the header and the first partials are independent loads
  const int b = p * a.parts;
  const PInfo& pi = ws.pinfo[src_of(a, p)];
  const Partial pr0 = first_partial(ws, b, a.parts, lane);
  const int e = b + active_parts(pi.n_tiles, a.parts);
  double S_d;
  long long S_and, S_or;
  wave_partial_sums(pi.bg_td, pi.bg_or, ws, b, e, lane, pr0, S_d, S_and, S_or);
  if (pi.skip) return;
  if (!pi.valid) {
    if (lane == 0) a.cost[p] = no_cost(pi.slot);
    return;
  }
  if (lane == 0) a.cost[p] = cost_from_sums(S_d, S_and, S_or, pi.kc);
}

// Gradient: one workgroup per particle.  Threads (segment, component) sum the per-item
// wrenches in item order; then one thread per pose parameter applies the kinematic adjoint
//   dE/dh_j = (1/S_or) sum_{s moved by j} a_j . (M_s + (q_s - q_j) x F_s)   (rotation)
//   dE/dh_j = (1/S_or) sum_{s moved by j} e_j . F_s                       (translation)
// with M_s, F_s the moment about the segment origin q_s and the force of segment s.
__global__ __launch_bounds__(kBlock) void finalize_grad_kernel(EvalArgs a, Workspace ws) {
  __shared__ double s_W[HT_MAX_SEG * 6];
  __shared__ double s_part[kWavesPerBlock][HT_MAX_SEG * 6];
  __shared__ double s_inv_or;
  __shared__ float s_org[HT_MAX_SEG * 4];
  __shared__ int s_kca[HT_MAX_KC], s_kcb[HT_MAX_KC];
  const int p = blockIdx.x, t = threadIdx.x;   // evaluated particle
  const int ps = src_of(a, p);                  // the workspace particle of its kinematics
  const int n_dof = a.n_dof, n_seg = a.n_seg;
  // every load that depends on the particle index alone is issued here: the item range, the
  // record, and this thread's pose parameter (descendant mask, camera-frame axis and point;
  // threads past n_dof have none).  The record is tested only after the sums below (a skipped
  // or invalid particle has no items), so no branch holds these loads back.
  const int b = ws.item_off[p], e = ws.item_off[p + 1];
  const PInfo& pi = ws.pinfo[ps];
  const int j = t, jc = min(t, n_dof - 1);   // loads clamped in bounds, unconditional
  const uint32_t desc = j < n_dof ? a.model->dof_desc[jc] : 0u;
  const float4* f4 = reinterpret_cast<const float4*>(ws.dof_frame + ((size_t)ps * n_dof + jc) * 8);
  const float4 f0 = f4[0], f1 = f4[1];
  const float fr[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
  // segment origins and collision pairs for the adjoint below, loaded into registers now and
  // staged in LDS after the wrench loads have been issued (one value per thread)
  static_assert(HT_MAX_SEG * 4 <= kBlock, "one segment-origin value per thread");
  const float org_v = t < n_seg * 4 ? ws.seg_org[(size_t)ps * n_seg * 4 + t] : 0.0f;
  const int kc_i = t < HT_MAX_KC ? t : 0;
  const int kca_v = a.model->kc_a[kc_i], kcb_v = a.model->kc_b[kc_i];
  // wave q sums items b+q, b+q+4, ... (kFinItems at a time, loads first); lane l sums values
  // l, l+64, l+128; then the four partial sums are added in a fixed order
  const int nv = n_seg * 6, lane = t & (kWave - 1);
  const int q = __builtin_amdgcn_readfirstlane(t >> 6);   // wave-uniform
  // the first partials, for the second wavefront's cost sums below; loaded by every wavefront
  // (unconditionally, so that no branch waits on them), issued with the wrench loads
  const Partial pr0 = first_partial(ws, b, max(e - b, 1), lane);
  constexpr int kFinItems = 4;
  double acc[3] = {0.0, 0.0, 0.0};
  for (int i = b + q; i < e; i += kFinItems * kWavesPerBlock) {
    // the loads are unconditional (items and offsets clamped into the particle's), so they are
    // in flight together; items past the end and lanes past nv add zero
    float v[kFinItems][3];
#pragma unroll
    for (int u = 0; u < kFinItems; ++u) {
      const float* src = ws.wrench + (size_t)min(i + u * kWavesPerBlock, e - 1) * nv;
#pragma unroll
      for (int k = 0; k < 3; ++k) v[u][k] = src[min(lane + k * kWave, nv - 1)];
    }
#pragma unroll
    for (int u = 0; u < kFinItems; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (i + u * kWavesPerBlock < e)
          acc[k] += lane + k * kWave < nv ? (double)v[u][k] : 0.0;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (lane + k * kWave < nv) s_part[q][lane + k * kWave] = acc[k];
  if (t < n_seg * 4) s_org[t] = org_v;
  if (t < HT_MAX_KC) {
    const bool on = t < a.model->n_kc;
    s_kca[t] = on ? kca_v : -1;
    s_kcb[t] = on ? kcb_v : -1;
  }
  // the cost sums go to the second wavefront, which has no pose parameter (at most 64 of them,
  // all in the first), so they overlap the first one's wrench sums
  static_assert(HT_MAX_DOF <= kWave, "pose parameters fit the first wavefront");
  double S_d = 0.0;
  long long S_and = 0, S_or = 0;
  if (q == 1) wave_partial_sums(pi.bg_td, pi.bg_or, ws, b, e, lane, pr0, S_d, S_and, S_or);
  if (pi.skip) return;
  if (!pi.valid) {
    if (t == 0) a.cost[p] = no_cost(pi.slot);
    for (int i = t; i < n_dof; i += kBlock) a.grad[(size_t)p * n_dof + i] = 0.0f;
    return;
  }
  if (q == 1 && lane == 0) {
    a.cost[p] = cost_from_sums(S_d, S_and, S_or, pi.kc);
    s_inv_or = S_or > 0 ? 1.0 / (double)S_or : 0.0;
  }
  __syncthreads();
  if (t < nv) s_W[t] = ((s_part[0][t] + s_part[1][t]) + s_part[2][t]) + s_part[3][t];
  __syncthreads();
  if (j < n_dof) {
    const float* f = fr;
    const float* org = s_org;
    const bool trans = f[0] != 0.0f;
    const double ax = f[1], ay = f[2], az = f[3];
    double g = 0.0;
    // the segments this parameter moves, in increasing order, four per round (their LDS reads
    // issued together)
    for (uint32_t m = desc; m;) {
      int sg[4];
      bool has[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        has[q] = m != 0u;
        sg[q] = has[q] ? __builtin_ctz(m) : 0;
        m &= m - 1u;
      }
      double t[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double* W = s_W + sg[q] * 6;
        const double lx = (double)org[sg[q] * 4 + 0] - f[4];
        const double ly = (double)org[sg[q] * 4 + 1] - f[5];
        const double lz = (double)org[sg[q] * 4 + 2] - f[6];
        const double mx = W[0] + (ly * W[5] - lz * W[4]);
        const double my = W[1] + (lz * W[3] - lx * W[5]);
        const double mz = W[2] + (lx * W[4] - ly * W[3]);
        t[q] = trans ? ax * W[3] + ay * W[4] + az * W[5] : ax * mx + ay * my + az * mz;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (has[q]) g += t[q];
    }
    g *= s_inv_or;
    // collision term of Eq. 5: the pairs whose term is positive (recorded by the kinematics)
    for (int m = pi.kc_mask; m; m &= m - 1) {
      const int i = __builtin_ctz(m);
      if (s_kca[i] == j) g -= kLambdaK;
      if (s_kcb[i] == j) g += kLambdaK;
    }
    a.grad[(size_t)p * n_dof + j] = (float)g;
  }
}

// ------------------------------------------------------------------------------------
// gradient refinement update, fused with the assembly of the preceding evaluation
//
// One workgroup per refined particle r.  First the evaluation that precedes this update is
// assembled, one wavefront per evaluated particle, as the finalize kernels would (the cost of
// Eq. 4-5 from the item partials; with gradients the per-segment wrench sums in item order
// and the kinematic adjoint, one lane per pose parameter): the particle itself after the
// gradient evaluation of the selected particles (wavefront 0), or its four candidates after a
// candidate evaluation (wavefront j: candidate j).  Then wavefront 0, one lane per dimension:
//   accept  - take the longest of the four steps that lowers E (the first in halving order);
//             when the candidates were evaluated with gradients the accepted one's becomes
//             the particle's gradient; no step lowers E: the particle stops refining;
//   propose - four candidates x - eta * (g_s / max|g_s|) / 2^j, j = 0..3, g_s = eta * dE/dh,
//             clamped to the bounds; a particle that has stopped (or whose g_s is zero or not
//             finite, which stops it) writes its own position four times, and its candidates
//             are skipped by the evaluation (its active flag is 0);
//   gather  - write the refined positions and costs back into the swarm.

// Cost of evaluated particle p and, with grad, lane j's component of its gradient (lanes past
// n_dof: 0), assembled by one wavefront.  W, org: this wavefront's LDS rows ([n_seg * 6]
// wrench sums, [n_seg * 4] segment origins).  Returns false for a particle that was skipped
// (not evaluated).  Holds no barrier.
__device__ bool assemble_wave(const EvalArgs& a, const Workspace& ws, int p, bool grad,
                              double* W, float* org, float& cost, float& g) {
  const int lane = threadIdx.x & (kWave - 1);
  const int n_seg = a.n_seg, n_dof = a.n_dof, nv = n_seg * 6;
  const int ps = uni(src_of(a, p));
  // its items: of the work list (gradient), or its parts
  const int b = grad ? scalar_ptr(ws.item_off)[p] : p * a.parts;
  const int parts = grad ? max(scalar_ptr(ws.item_off)[p + 1] - b, 1) : a.parts;
  // loads that depend on the particle alone, issued before any branch: the record, the first
  // partials, this lane's pose-parameter frame and segment-origin values (clamped indices)
  const PInfoPtr ph = scalar_ptr(ws.pinfo + ps);
  const Partial pr0 = first_partial(ws, b, parts, lane);
  const int jc = min(lane, n_dof - 1);
  const float4* f4 = reinterpret_cast<const float4*>(ws.dof_frame + ((size_t)ps * n_dof + jc) * 8);
  const float4 f0 = f4[0], f1 = f4[1];
  const uint32_t desc = lane < n_dof ? a.model->dof_desc[jc] : 0u;
  const float* org_src = ws.seg_org + (size_t)ps * n_seg * 4;
  const float o0 = org_src[min(lane, n_seg * 4 - 1)];
  const float o1 = org_src[min(lane + kWave, n_seg * 4 - 1)];
  g = 0.0f;
  if (ph->skip) return false;
  const int e = b + (grad ? (ph->n_tiles ? parts : 0) : active_parts(ph->n_tiles, parts));
  double S_d;
  long long S_and, S_or;
  wave_partial_sums(ph->bg_td, ph->bg_or, ws, b, e, lane, pr0, S_d, S_and, S_or);
  if (!ph->valid) {
    cost = no_cost(ph->slot);
    return true;
  }
  cost = cost_from_sums(S_d, S_and, S_or, ph->kc);
  if (!grad) return true;
  // wrench rows summed in item order (lane l: values l, l + 64, l + 128), kAsmItems items'
  // loads in flight at a time (indices clamped into the particle's items; past the end adds
  // zero): each round is one memory latency, and small gradient launches give a particle
  // some 30 items
  constexpr int kAsmItems = 16;
  double acc[3] = {0.0, 0.0, 0.0};
  for (int i0 = b; i0 < e; i0 += kAsmItems) {
    float v[kAsmItems][3];
#pragma unroll
    for (int u = 0; u < kAsmItems; ++u) {
      const float* src = ws.wrench + (size_t)min(i0 + u, e - 1) * nv;
#pragma unroll
      for (int k = 0; k < 3; ++k) v[u][k] = src[min(lane + k * kWave, nv - 1)];
    }
#pragma unroll
    for (int u = 0; u < kAsmItems; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        acc[k] += (i0 + u < e && lane + k * kWave < nv) ? (double)v[u][k] : 0.0;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (lane + k * kWave < nv) W[lane + k * kWave] = acc[k];
  if (lane < n_seg * 4) org[lane] = o0;
  if (lane + kWave < n_seg * 4) org[lane + kWave] = o1;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // the kinematic adjoint of the finalize kernel, lane j = pose parameter j
  const int j = lane;
  if (j < n_dof) {
    const double inv_or = S_or > 0 ? 1.0 / (double)S_or : 0.0;
    const bool trans = f0.x != 0.0f;
    const double ax = f0.y, ay = f0.z, az = f0.w;
    double acc_g = 0.0;
    // the segments this parameter moves, in increasing order, kAdjRound per round: their LDS
    // reads are issued together (one segment per round waited on the reads of each in turn;
    // eight per round measured no faster than four)
    constexpr int kAdjRound = 4;
    for (uint32_t m = desc; m;) {
      int sg[kAdjRound];
      bool has[kAdjRound];
#pragma unroll
      for (int q = 0; q < kAdjRound; ++q) {
        has[q] = m != 0u;
        sg[q] = has[q] ? __builtin_ctz(m) : 0;
        m &= m - 1u;
      }
      double t[kAdjRound];
#pragma unroll
      for (int q = 0; q < kAdjRound; ++q) {
        const double* Ws = W + sg[q] * 6;
        const double lx = (double)org[sg[q] * 4 + 0] - f1.x;
        const double ly = (double)org[sg[q] * 4 + 1] - f1.y;
        const double lz = (double)org[sg[q] * 4 + 2] - f1.z;
        const double mx = Ws[0] + (ly * Ws[5] - lz * Ws[4]);
        const double my = Ws[1] + (lz * Ws[3] - lx * Ws[5]);
        const double mz = Ws[2] + (lx * Ws[4] - ly * Ws[3]);
        t[q] = trans ? ax * Ws[3] + ay * Ws[4] + az * Ws[5] : ax * mx + ay * my + az * mz;
      }
#pragma unroll
      for (int q = 0; q < kAdjRound; ++q)
        if (has[q]) acc_g += t[q];
    }
    acc_g *= inv_or;
    for (int m = ph->kc_mask; m; m &= m - 1) {
      const int i = __builtin_ctz(m);
      if (a.model->kc_a[i] == j) acc_g -= kLambdaK;
      if (a.model->kc_b[i] == j) acc_g += kLambdaK;
    }
    g = (float)acc_g;
  }
  return true;
}

__global__ __launch_bounds__(kBlock) void refine_update_kernel(EvalArgs a, Workspace ws,
                                                               RefineArgs ra) {
  __shared__ double s_W[kWavesPerBlock][HT_MAX_SEG * 6];
  __shared__ float s_org[kWavesPerBlock][HT_MAX_SEG * 4];
  __shared__ float s_cost[kWavesPerBlock];
  __shared__ float s_g[kWavesPerBlock][HT_MAX_DOF];
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = blockIdx.x;                       // refined particle (frame * K + rank)
  const int n_dof = ra.n_dof;
  const bool on = lane < n_dof;
  const int d = on ? lane : 0;
  const size_t xi = (size_t)r * n_dof + d;
  // the inputs of wavefront 0's decisions below, loaded before the assembly so that their
  // latency overlaps it (no kernel writes them meanwhile; this one writes them only after
  // reading them); buffers a mode does not use are allocated, their values unused
  const int act_in = ra.active[r];
  const float x_in = ra.rx[xi], c_in = ra.rcost[r], g_in = ra.grad[xi];
  float cx_in[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) cx_in[j] = ra.cand[((size_t)r * 4 + j) * n_dof + d];
  const int trans_in = a.model->dof_trans[d];
  const float lo_in = a.model->lo[d], hi_in = a.model->hi[d];
  // 1. the preceding evaluation: the particle itself (propose only), else its candidates
  const bool mine = ra.op.accept ? true : w == 0;
  if (mine) {
    const int p = ra.op.accept ? r * 4 + w : r;
    float c = INFINITY, g = 0.0f;
    if (!assemble_wave(a, ws, p, ra.eval_grad, s_W[w], s_org[w], c, g)) c = INFINITY;
    if (lane == 0) s_cost[w] = c;
    if (lane < HT_MAX_DOF) s_g[w][lane] = g;
  }
  __syncthreads();
  if (w != 0) return;
  bool act = act_in != 0;
  float x = x_in;
  float c, gd;
  if (!ra.op.accept) {
    // the gradient evaluation of the selected particle: its cost and gradient
    c = s_cost[0];
    gd = s_g[0][d];
    if (on) ra.grad[xi] = gd;
    if (lane == 0) ra.rcost[r] = c;
  } else {
    c = c_in;
    gd = g_in;
  }
  if (ra.op.accept && act) {
    // the four candidates' costs (a skipped one counts as +inf) and positions
    float cc[4], cx[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cc[j] = s_cost[j];
      cx[j] = cx_in[j];
    }
    int pick = -1;
#pragma unroll
    for (int j = 3; j >= 0; --j)
      if (cc[j] < c) pick = j;
    if (pick < 0) {
      act = false;
      if (lane == 0) ra.active[r] = 0;
    } else {
      float nx = cx[0], ng = s_g[0][d];
      c = cc[0];
#pragma unroll
      for (int j = 1; j < 4; ++j) {
        nx = pick == j ? cx[j] : nx;
        ng = pick == j ? s_g[j][d] : ng;
        c = pick == j ? cc[j] : c;
      }
      x = nx;
      if (on) {
        ra.rx[xi] = x;
        if (ra.eval_grad) {
          gd = ng;
          ra.grad[xi] = gd;
        }
      }
      if (lane == 0) ra.rcost[r] = c;
    }
  }
  if (ra.op.propose) {
    const float eta = trans_in ? ra.eta_trans : ra.eta_rot;
    const float gs = on ? eta * gd : 0.0f;
    float gmax = fabsf(gs);
    bool fin = isfinite(gs);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) gmax = fmaxf(gmax, __shfl_xor(gmax, o));
    fin = __ballot(!fin) == 0ull;
    const bool ok = act && fin && gmax > 0.0f;
    // a particle without a usable step stops refining: its candidates are not evaluated
    if (act && !ok && lane == 0) ra.active[r] = 0;
    if (on) {
      for (int j = 0; j < 4; ++j) {
        float xn = x;
        if (ok) {
          const float step = eta * (gs / gmax) * ldexpf(1.0f, -j);
          xn = fminf(fmaxf(x - step, lo_in), hi_in);
        }
        ra.cand[((size_t)r * 4 + j) * n_dof + d] = xn;
      }
    }
  }
  if (ra.op.gather) {
    const int f = r / ra.K;
    if (ra.sw.stop_gen && ra.sw.stop_gen[f] != 0) return;
    const size_t gp = (size_t)f * ra.sw.n_particles + ra.sel[r];
    if (on) ra.sw.x[gp * n_dof + d] = x;
    if (lane == 0) ra.sw.cost[gp] = c;
  }
}

hipError_t launch_refine_update(const EvalArgs& a, const Workspace& ws, const RefineArgs& ra,
                                hipStream_t s) {
  if (ra.n_ref == 0) return hipSuccess;
  hipLaunchKernelGGL(refine_update_kernel, dim3(ra.n_ref), dim3(kBlock), 0, s, a, ws, ra);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------

// The ray-cast variant of a launch, and its LDS bytes (the tables, and a gradient's wrench rows).
template <int NT>
static const void* raycast_fn_nt(bool grad, bool dbg, bool self) {
  if (grad)
    return self ? reinterpret_cast<const void*>(&raycast_kernel<true, false, NT, true>)
                : reinterpret_cast<const void*>(&raycast_kernel<true, false, NT, false>);
  return dbg ? reinterpret_cast<const void*>(&raycast_kernel<false, true, NT, false>)
             : reinterpret_cast<const void*>(&raycast_kernel<false, false, NT, false>);
}

static const void* raycast_fn(bool grad, bool dbg, bool all_types, bool self) {
  return all_types ? raycast_fn_nt<kNumTypes>(grad, dbg, self) : raycast_fn_nt<3>(grad, dbg, self);
}

static size_t raycast_lds(bool grad, int n_prim, int n_seg) {
  return (size_t)Tables(n_prim).words * 16 +
         (grad ? (size_t)kWavesPerBlock * n_seg * 24 * sizeof(float) : 0);
}

// Workgroups of a ray-cast variant that are resident on one CU at once (its registers and
// LDS decide).  The persistent grid is capped at this many per CU: a workgroup beyond it
// starts only when another has finished, and its statically assigned first item then
// finishes late (a 128-particle launch spent half its time in that tail).
int raycast_groups_per_cu(bool grad, bool dbg, bool all_types, bool self, int n_prim,
                          int n_seg) {
  int r = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, raycast_fn(grad, dbg, all_types, self),
                                                   kBlock, raycast_lds(grad, n_prim, n_seg)) != hipSuccess ||
      r < 1) {
    (void)hipGetLastError();
    r = 1;
  }
  return r;
}

// The evaluation is one to four launches on one stream; `stage` selects one so the host can
// bracket each with HIP events when profiling.
hipError_t launch_eval_stage(int stage, const EvalArgs& a, const Workspace& ws, hipStream_t s) {
  const int n_total = a.n_frames * a.n_particles;
  if (n_total == 0) return hipSuccess;
  const bool dbg = a.dbg.depth || a.dbg.hit || a.dbg.rm || a.dbg.winner || a.dbg.margin;
  switch (stage) {
    case kStageSmall: {
      const TypeMasks tm = a.type_masks;
      const bool all = (tm.m[HT_CONE][0] | tm.m[HT_CONE][1] | tm.m[HT_ECYLINDER][0] |
                        tm.m[HT_ECYLINDER][1]) != 0ull;
      const size_t lds = raycast_lds(false, a.n_prim, a.n_seg);
      const auto f = a.finish ? (all ? small_eval_kernel<kNumTypes, true> : small_eval_kernel<3, true>)
                              : (all ? small_eval_kernel<kNumTypes, false> : small_eval_kernel<3, false>);
      hipLaunchKernelGGL(f, dim3(n_total * a.parts), dim3(kBlock), lds, s, a, ws, tm);
      break;
    }
    case kStageFk:
      if (a.src) break;   // the kinematics of the previous evaluation are reused
      // wavefronts per particle: at least one per 64 primitives (a lane sets up one primitive);
      // four while every particle still has a CU of its own (256 poses of a 320x240 frame 29.9 us,
      // 31.1 us with one; gradients of them 49.4 and 51.1 us), else few, the kernel being bound by
      // its FP64 instructions (4096 poses of 64 uneven frames 83, 92 and 106 us with one, two, four)
      if (n_total <= kFkSpread)
        hipLaunchKernelGGL(fk_kernel<4>, dim3(n_total), dim3(kBlock), 0, s, a, ws);
      else if (a.n_prim > kWave)
        hipLaunchKernelGGL(fk_kernel<2>, dim3((n_total + 1) / 2), dim3(kBlock), 0, s, a, ws);
      else
        hipLaunchKernelGGL(fk_kernel<1>, dim3((n_total + 3) / 4), dim3(kBlock), 0, s, a, ws);
      break;
    case kStageSched:
      // (the forward cast needs no list, a small gradient cast builds its own)
      if (a.grad && n_total > kSelfSched)
        hipLaunchKernelGGL(sched_kernel, dim3(1), dim3(kSchedBlock), 0, s, a, ws);
      break;
    case kStageRaycast: {
      const TypeMasks tm = a.type_masks;
      const bool all = (tm.m[HT_CONE][0] | tm.m[HT_CONE][1] | tm.m[HT_ECYLINDER][0] |
                        tm.m[HT_ECYLINDER][1]) != 0ull;
      if (dbg) {
        const size_t n = (size_t)a.n_particles * a.dbg_H * a.dbg_W;
        hipLaunchKernelGGL(debug_fill_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, s, a.dbg, n, a.dbg_bg);
      }
      const void* f = raycast_fn(a.grad != nullptr, dbg, all, n_total <= kSelfSched);
      EvalArgs ka = a;
      Workspace kw = ws;
      TypeMasks kt = tm;
      void* args[] = {&ka, &kw, &kt};
      return hipLaunchKernel(f, dim3(a.grid), dim3(kBlock), args,
                             (unsigned)raycast_lds(a.grad != nullptr, a.n_prim, a.n_seg), s);
    }
    case kStageFinalize:
      if (a.grad)
        hipLaunchKernelGGL(finalize_grad_kernel, dim3(n_total), dim3(kBlock), 0, s, a, ws);
      else
        hipLaunchKernelGGL(finalize_kernel, dim3((n_total + kWavesPerBlock - 1) / kWavesPerBlock),
                           dim3(kBlock), 0, s, a, ws);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ht
