// Internal types shared by the host runtime (mvf_runtime.cpp) and the HIP
// kernels (mvf_kernels.hip).  Not part of the public ABI.
//
// Device volume layout ("brick-linear"): a volume of dims (nx, ny, nz) is
// padded to bricks of 8x8x8 voxels, bd = ceil(dims / 8) bricks per axis.
// Bricks are numbered z-fastest, brick(bx, by, bz) = (bx * bd.y + by) * bd.z
// + bz, so a column of bricks (fixed bx, by) is one contiguous run.  Inside a
// brick voxels are x-fastest: (z & 7) * 64 + (y & 7) * 8 + (x & 7); one
// z-slice of a brick is 64 consecutive elements, exactly one wavefront.
//
// Planes, each padded to a 256-byte multiple, in one slab per volume:
//   F     float32  TSDF in truncation units; NaN while the voxel is
//                  unobserved (W == 0), so one trilinear read both
//                  interpolates and tests that all 8 corners were observed
//   W     uint16   running weight
//   C     uint32   RGBA8 colour, A = colour weight
//   flag  uint8    per brick: 1 if some voxel of the brick may hold
//                  F <= 2^-100 (set by integration, never cleared except by
//                  a full recompute); 0 guarantees F > 0 or NaN everywhere
//                  in the brick, which lets the raycast skip it exactly.
//   dist  uint8    per brick: Chebyshev distance, in bricks, to the nearest
//                  flagged brick, capped at kDistCap (0 = flagged); every
//                  brick within dist - 1 of this one is unflagged.  Derived
//                  from the flags after each integration.
//   colm  uint64   per brick column (bx, by) and 64 bricks of it along z:
//                  word (bx * bd[1] + by) * col_words(bd[2]) + (bz >> 6),
//                  bit bz & 63 equal to the brick's flag (maintained with
//                  the flags; the distance transform reads only these),
//                  then one word that is always zero.
//   fmask uint64   per brick: bit z2 * 16 + y2 * 4 + x2 set if some voxel of
//                  the 2x2x2 sub-block (x2, y2, z2) of the brick may hold
//                  F <= 2^-100 (same monotone rule as flag, which equals
//                  fmask != 0).
//   cmask uint64   per brick: the same bits for cells: bit (x2, y2, z2) set
//                  if a voxel of [2 x2, 2 x2 + 2] x [2 y2, 2 y2 + 2] x
//                  [2 z2, 2 z2 + 2] (brick-local, reaching into the +x, +y,
//                  +z neighbour bricks) may hold F <= 2^-100, i.e. some cell
//                  whose base voxel lies in that sub-block may have a corner
//                  F <= 2^-100.  fmask dilated by one sub-block; derived
//                  after each integration with the distance transform.
#pragma once
#include <stdint.h>

#ifndef MVF_HD
#if defined(__HIPCC__)
#define MVF_HD __host__ __device__ __forceinline__
#else
#define MVF_HD inline
#endif
#endif

namespace mvf {

constexpr int kBrick = 8;
constexpr int kBrickVox = 512;
constexpr float kFlagThreshold = 0x1p-100f;
constexpr int kDistCap = 12;

// 64-bit words per brick column of the colm flag bits
MVF_HD int col_words(int bd2) { return (bd2 + 63) >> 6; }
// Lines of the brick distance transform: (bx, kDistRows columns along y,
// 64-brick word of the columns).
constexpr int kDistRows = 64 - 2 * kDistCap;
MVF_HD int dist_lines(const int bd[3]) { return bd[0] * ((bd[1] + kDistRows - 1) / kDistRows) * col_words(bd[2]); }

struct DevVolume {
    float* F;
    uint16_t* W;
    uint32_t* C;
    uint8_t* flag;
    uint8_t* dist;
    uint64_t* colm;          // per brick column: flags as bits along z
    uint64_t* fmask;         // per brick: sub-block flags
    uint64_t* cmask;         // per brick: cell sub-block flags
    int32_t dims[3];
    int32_t off[3];
    int32_t bd[3];
    int32_t id;          // public volume id (hit output, tie-break)
    float o[3];          // grid origin
    float s;             // voxel size
    float inv_s;         // 1 / s (binary32, correctly rounded)
    float mu;            // trunc_voxels * s (binary32)
    float inv_mu;        // 1 / mu
    int32_t w_max;
    int32_t frame;       // index of the stream's frame in the frame table
    int32_t zt_base;     // first entry of this volume in the launch's z table
    int32_t line_base;   // distance lines of the launch's volumes before this one
    // world box that a raycast looks for samples in: the sample domain grown
    // by a voxel
    float ray_lo[3], ray_hi[3];
};

struct DevFrame {
    const float* range;      // H*W: depth * ray-length factor, 0 = invalid
    const uint32_t* color;   // H*W packed RGB (may be null)
    float* rmax;             // [0]: max range of the frame (for clipping); [1 + b]: per prep block
    int32_t rmax_parts;      // prep blocks of this frame (ceil(width / 32) * ceil(height / 8))
    const float* tmax;       // maximum range of each 8x8 pixel tile (row-major), then the minimum of each
                             // (tiles_x * tiles_y further on; 0 where a pixel has no range), or null
    int32_t tiles_x, tiles_y;
    int32_t width, height;
    float fx, fy, cx, cy;
    float T[12];
    // raycast outputs
    float* depth;
    float* vertex;
    float* normal;
    int32_t* hit;
    float* best_t;           // per-pixel running best (multi-wave raycast)
    int32_t* best_id;
    int32_t* record;         // per pixel: k of the nearest crossing's second sample, -1 = none; or null
    int32_t out_w, out_h;
    float inv_cells_x;       // 1 / cells_x (rounded; the kernel corrects the quotient)
    // raycast range bounds per 8x8 output-pixel cell (cells_x * cells_y,
    // row-major), or null: the nearest and farthest camera distance of any
    // sample the march may have to evaluate; a cell no brick reaches holds
    // (inf, 0).  Written by launch_ray_bounds_merge.
    float* rb_lo;
    float* rb_hi;
    int32_t cells_x, cells_y;
};

struct RayParams {
    float delta;             // step * s (binary32); all volumes of a call share one grid
    int32_t kmax;            // floor(t_far / delta)
};

// 64-bit counters written by kernels.  kCntSlots copies, each on its own
// 128-byte line (slot k at counters + k * kCntNum), spread the atomics of
// many blocks over several addresses; a reader sums the slots.
enum Counter { kCntUpdated = 0, kCntBand = 1, kCntBricks = 2, kCntDeep = 3, kCntNum = 16 };
constexpr int kCntSlots = 64;

// Launch parameters that live in device memory with the other tables of a call.
struct LaunchHeader {
    int32_t nvol;          // entries of the volume table used by integration
    int32_t total_items;   // integration work items
    int32_t zchunk;        // bricks per integration item along z
    int32_t nstreams;      // frames in the frame table
    int32_t total_tiles;   // raycast pixel tiles over all streams
    int32_t total_bricks;  // bricks over all volumes of the table (distance transform)
    int32_t first_wave;    // raycast: 1 = start from no hit, 0 = merge with best_t/best_id
    RayParams rp;
    int32_t total_z;       // entries of the integration z table (sum of 8 * bd[2])
    int32_t total_lines;   // distance lines over all volumes of the table
    int32_t rb_parity;     // raycast range bounds: which half of RayBounds::counts this launch fills
    int32_t list_parity;   // integration: which of the two visited-item counts this launch uses
};

// Footprint of one brick in the raycast range bounds: cells [x0, x1] x
// [y0, y1] of its volume's frame and the camera distances [dn, df] of its box.
struct RayBoundEntry {
    uint16_t x0, x1, y0, y1;
    float dn, df;
};

// Range-bound footprints of a launch.  Volume v of the table appends to
// entries + brick_base[v] (room for all its bricks) and counts its entries
// in counts[rb_parity * cap + v]; the merge reads them and clears the other
// half for the next launch.
struct RayBounds {
    RayBoundEntry* entries;
    uint32_t* counts;          // 2 * cap, zero before first use
    int32_t cap;               // volume slots per half (>= nvol)
};

// Frame preparation input for one stream.
struct PrepItem {
    const float* depth;
    const uint8_t* rgb;
    int32_t depth_pitch, rgb_pitch;
    int32_t width, height;
    float fx, fy, cx, cy;
    float* range;
    uint32_t* color;
    float* rmax;             // [0] frame's maximum range, [1 + b] maximum of prep block b
    float* tmax;             // maximum range of each 8x8 pixel tile, ceil(width / 8) per row; the
                             // minima follow (ceil(width / 8) * ceil(height / 8) further on)
};

// Items that frame preparation takes as kernel arguments.
constexpr int kPrepInline = 16;
struct PrepArgs {
    PrepItem item[kPrepInline];
};

// The raycast's work: pixel tiles of 8x8 (one range-bound cell each), each
// marched by 2^level one-wavefront blocks of 64 >> level pixels, 2^level lanes
// per ray.  More lanes per ray make a tile's longest chain of rounds shorter
// and its work larger, so the level is chosen tile by tile (TileOrder).
constexpr int kRayTile = 8;
constexpr int kRayLevels = 5;
constexpr int kBoundCell = kRayTile;   // output pixels per side of a raycast range-bound cell
constexpr int kXcds = 8;
// pixels of a block of a level: 8x8, 8x4, 4x4, 4x2, 2x2
MVF_HD constexpr int ray_block_w(int level) { return kRayTile >> (level / 2); }
MVF_HD constexpr int ray_block_h(int level) { return kRayTile >> ((level + 1) / 2); }
// Default of the schedule's ray_lanes.
constexpr int kRayLanes = 4;
// Blocks that a launch order may take beyond its tiles' own (each level's tiles
// are rounded to whole windows of kXcds: less than 8 * 31).
constexpr int kRaySlack = 512;
// Wavefronts of the raycast kernel that a compute unit holds.
constexpr int kRayWavesPerCu = 20;

// A launch order to compute for that many raycast tiles from their last
// durations, longest first (a slow tile started late bounds the launch), with
// each tile's level; tiles 0: none.  The order begins with a RayPlan.  Block
// of the launch -> (tile, part): from block[level] on, 8 tiles at a time (one
// per XCD, over which blocks are dealt round-robin), all the parts of a tile
// on one XCD (they gather the same bricks).
struct RayPlan {
    int32_t pos[8];     // first position in the order of each level (higher levels come first)
    int32_t block[8];   // its first block; [kRayLevels]: the number of blocks
};
constexpr int kRayPlanInts = 16;
struct TileOrder {
    uint32_t* cost;     // per tile: its longest block in the last launch, scaled to level 0; zeroed by the ordering
    int32_t* order;     // RayPlan, then the tiles
    int32_t tiles;
    int32_t level;      // of every tile when a duration is missing
    int32_t max_blocks; // of the raycast launch
    int32_t slots;      // wavefronts the device holds
    int32_t fresh;      // ignore the durations (of another image size)
};

// Integration work item: a brick column (8x8 voxel columns) of one volume
// over a chunk of zchunk bricks along z.  Items of table entry v are
// [item_base[v], item_base[v+1]).
//
// z table: for volume v and local z in [0, 8 * bd[2]), entry
// vols[v].zt_base + z holds 3 floats: T[8], T[9], T[10] times
// (x_w(z) - T[11]), the camera-frame offset of the voxel plane z (binary32,
// the same operations as the voxel test).  Written by launch_ztable before
// the integration kernel runs; ztab holds >= hdr->total_z entries.
struct IntegrateLaunch {
    const LaunchHeader* hdr;
    const DevVolume* vols;
    const DevFrame* frames;
    const int32_t* item_base;  // nvol + 1 prefix sums
    unsigned long long* counters;
    float* ztab;
    // per item, kVisitPerItem bytes: byte j is 1 if brick bz0 + j of the
    // item may hold a voxel the frame updates (written by the z-table
    // launch), or null (visit all); needs zchunk <= kVisitPerItem
    uint8_t* visit;
    // optional (tiles > 0): block 0 computes a raycast tile order instead of
    // integrating; the grid has one more block
    TileOrder order;
    // visited work, compacted (needs visit): the z-table launch appends
    // every brick to visit voxel by voxel to list and every deep brick (each
    // voxel updated with phi = 1, proved by the visit test) to deep_list,
    // both as item * 8 + j (brick j of the item; room for total_items *
    // zchunk each); list_count[hdr->list_parity] counts both (visited bricks
    // in the low 32 bits, deep bricks in the high 32).  Integration gives
    // each entry a wavefront, the visited bricks first.  The z-table launch
    // also zeroes list_count[list_parity ^ 1] for the next launch, so the
    // two words must be zero before first use.
    int32_t* list;
    unsigned long long* list_count;
    int32_t* deep_list;
};
constexpr int kVisitPerItem = 8;

struct RaycastLaunch {
    const LaunchHeader* hdr;
    const DevVolume* vols;      // table
    const DevFrame* frames;     // one per stream
    const int32_t* lists;       // concatenated per-stream lists of table indices, nearest first
    const int32_t* list_base;   // per stream: [list_base[s], list_base[s+1])
    const int32_t* tile_base;   // per stream: first pixel tile; nstreams + 1 entries
    uint32_t* tile_cost;        // TileOrder::cost, zero before the launch
    const int32_t* tile_order;  // TileOrder::order
};

// Host-side launchers (defined in mvf_kernels.hip).  All return hipError_t
// as int (0 = success).
// Frame preparation of n frames, their items in pinned host memory (read when
// the launch runs if there are more than kPrepInline).  With tsrc set the
// launch also copies tbytes (a multiple of 16, 16-byte aligned) from tsrc,
// pinned host memory, to tdst.
int launch_frame_prep(const PrepItem* items, int n, int max_w, int max_h, void* stream, const void* tsrc = nullptr,
                      void* tdst = nullptr, size_t tbytes = 0);
int launch_volume_init(DevVolume v, void* stream);
// The z table of a launch and, when L.visit is set, the visit pass over
// the launch's `bricks` bricks (total_items * zchunk; one thread per brick,
// up to 2048 blocks of 512 threads, which then walk the rest); must precede
// launch_integrate on the stream.
int launch_ztable(const IntegrateLaunch& L, int bricks, void* stream);
// Integration kernel: blocks of 256 threads, 4 items in flight per block; a
// grid smaller than total_items / 4 walks the items (plus block 0 when
// L.order.tiles is set).
// With ev_start/ev_stop (hipEvent_t) the kernel's own dispatch records them.
int launch_integrate(const IntegrateLaunch& L, int blocks, void* stream, void* ev_start = nullptr,
                     void* ev_stop = nullptr);
// Raycast kernel; blocks: TileOrder::max_blocks.
int launch_raycast(const RaycastLaunch& L, int blocks, void* stream, void* ev_start = nullptr,
                   void* ev_stop = nullptr);
// Column flag words from the brick flags.
int launch_column_flags(DevVolume v, void* stream);
// Brick distance transform of every volume in the table; lines and bricks:
// their totals, for the grid (the header's count).  brick_base: nvol + 1 prefix sums of the volumes' brick counts (each a
// multiple of 64).  With frames and rb.entries set, the last pass also
// collects the range-bound footprints (as launch_ray_bounds_collect).
int launch_brick_distance(const LaunchHeader* hdr, const DevVolume* vols, const int32_t* brick_base,
                          int lines, int bricks, void* stream, const DevFrame* frames = nullptr,
                          RayBounds rb = RayBounds{});
// Range-bound footprints of the bricks of every volume of the table whose
// cell mask is not empty, for the volume's frame.
int launch_ray_bounds_collect(const LaunchHeader* hdr, const DevVolume* vols, const int32_t* brick_base,
                              const DevFrame* frames, RayBounds rb, int blocks, void* stream);
// Range bounds of every cell of each stream's frame from the footprints of
// the stream's volumes (lists / list_base as in RaycastLaunch); clears the
// other half of rb.counts.  max_cells_x/y: largest cell grid of the frames.
// One more block computes `order`, if given.
int launch_ray_bounds_merge(const LaunchHeader* hdr, const DevFrame* frames, const int32_t* lists,
                            const int32_t* list_base, const int32_t* brick_base, RayBounds rb, int nstreams,
                            int max_cells_x, int max_cells_y, void* stream, TileOrder order = TileOrder{});
// bytes (a multiple of 16) from device to pinned memory, both 16-byte aligned.
int launch_swap_copy(const void* src, void* dst, size_t bytes, void* stream);
// Elements [e0, e0 + n) of a volume's canonical plane (0: F, 1: weights, 2:
// colours) to out, pinned host memory.
int launch_read_plane(DevVolume v, int plane, uint32_t e0, uint32_t n, void* out, void* stream);
// Canonical planes (null: empty) into the volume's bricks, with the brick
// flags and sub-block masks; full: weights and colours too, else only F.
int launch_import(DevVolume v, const float* F, const uint16_t* W, const uint32_t* C, bool full, void* stream);
// Surface points of one volume of nbricks bricks: scratch of
// extract_buffer_bytes(nbricks) device bytes laid out by extract_buffers, and
// a pinned host word that receives the number of points.  With cap > 0 the
// first cap points are written (V, N: 3 floats each; G: 3 ints, or null) in
// brick order.
struct ExtractBuffers {
    uint32_t* list;      // bricks with a set cell mask, in brick order
    uint32_t* counts;    // points of each listed brick
    uint32_t* group_n;   // points of each 16 listed bricks
    uint32_t* chunk_n;   // listed bricks of each 1024 bricks
    uint32_t* super_n;   // points of each 1024 listed bricks
    uint32_t* list_n;
    long long* total;    // pinned
};
size_t extract_buffer_bytes(size_t nbricks);
ExtractBuffers extract_buffers(void* mem, size_t nbricks, long long* total);
int launch_extract(DevVolume v, const ExtractBuffers& B, float* V, float* N, int32_t* G, long long cap, void* stream);
int launch_fill_u64(unsigned long long* p, int n, unsigned long long value, void* stream);

// Placement counting of one frame on the lattice of side `cell` (metres):
// endpoints inside one of the boxes (h_t[3], dims[3], global voxels) are left
// out.  The pose and the boxes travel in the launch's arguments.
constexpr int kPlaceTable = 8192;     // hash slots, a power of two
constexpr int kMaxPlaceBoxes = 64;
struct PlacementCount {
    const float* depth;
    int32_t depth_pitch, width, height;
    float fx, fy, cx, cy;
    float T[12];
    float o[3];                // grid origin
    float cell, voxel;
    unsigned long long* table; // 2 * table_size words, empty before the count and after the collection
    int32_t table_size;
    int32_t n_boxes;
    int* overflow;             // bit 0: table full, bit 1: a cell or voxel index out of range
    int32_t boxes[6 * kMaxPlaceBoxes];
};
// What a count found (pinned host memory).
struct PlacementCells {
    int32_t n, overflow;
    unsigned long long key[kPlaceTable];
    unsigned long long count[kPlaceTable];
};
int launch_placement_clear(unsigned long long* table, int table_size, int* overflow, void* stream);
// The count and its collection into *out (pinned), which also empties the table.
int launch_placement_count(const PlacementCount& P, PlacementCells* out, void* stream);

// Camera tracking (mvf_track.hip).  The pose estimate and the statistics of
// every Gauss-Newton step live in device memory.
constexpr int kTrackSums = 29;          // A (21, upper triangle), b (6), pairs, sum r^2
constexpr int kTrackThreads = 256;
constexpr int kTrackPixPerThread = 4;
constexpr int kTrackMaxSteps = 64;

struct TrackState {
    double T[12];        // estimate, camera-to-world, row-major 3x4
    float T32[12];       // its binary32 rounding (the association reads it)
    int32_t steps;
    uint32_t ticket;     // blocks of the running step that have finished
    int32_t pairs[kTrackMaxSteps];
    double sq_err[kTrackMaxSteps];
};

struct TrackLaunch {
    const float* V;      // current level: vertex and normal maps, w x h x 3, camera frame
    const float* N;
    int32_t w, h;
    const float* Vm;     // model level: world maps of the same size
    const float* Nm;
    float fx, fy, cx, cy;
    float Tm[12];        // the model's camera-to-world pose
    float eps_d, cos_theta;
    TrackState* state;
    double* partials;    // track_blocks(w, h) x kTrackSums
};

// The maps of one pyramid level: depth in, vertex and normal maps out; for
// levels >= 1 also the subsampled model maps out.
struct TrackMapLevel {
    const float* D;
    int32_t pitch, w, h;
    float fx, fy, cx, cy;
    float* V;
    float* N;
    float* Vm;
    float* Nm;
};
constexpr int kTrackMapsMax = 5;
struct TrackMaps {
    TrackMapLevel level[3];
    int32_t levels;
    int32_t first[kTrackMapsMax];  // first block of each map (set by launch_track_maps)
    const float* Vm;     // full-size model maps, or null (no model)
    const float* Nm;
    TrackState* state;   // set up for a call that starts from T, or null
    double T[12];
};

// Edge-preserving smoothing of a depth map (out: w x h, pitch w).
int launch_track_smooth(const float* D, int pitch, int w, int h, float delta, float* out, void* stream);
int launch_track_down(const float* D, int pitch, int w, int h, float tau, float* D2, void* stream);
int launch_track_maps(TrackMaps M, void* stream);
int track_blocks(int w, int h);
// Step `step`: association, reduction, solve and update; with `out` (pinned
// host memory) also the call's result.
int launch_icp_step(const TrackLaunch& L, int step, TrackState* out, void* stream);

struct DiffVolume {
    const float* F;
    const uint16_t* W;
    int32_t dims[3];
    int32_t off[3];
    float o[3];
    float s, inv_s;
};
int launch_diffray_backward(DiffVolume v, const float* T, float fx, float fy, float cx, float cy,
                            int width, int height, RayParams rp, const float* grad_depth,
                            const int32_t* record, float* grad_F, double* partials,
                            int n_partials, double* grad_xi, void* stream);
int diffray_partials_needed(int width, int height);
// Allocation-free backward: a static device array holds the pose partials of
// at most kDiffScratchBlocks 16x16-pixel blocks (768 KiB per GPU).
constexpr int kDiffScratchBlocks = 16384;
constexpr int kMaxDevices = 64;
// Take the current device's address of the static array (once per device;
// the device must be current).  0 on success, else a hipError_t.
int diffray_scratch_init(int device);
// That address, or null before diffray_scratch_init(device) succeeded.
double* diffray_scratch(int device);

}  // namespace mvf
