// The raycast's launch order, computed by one block of another launch (device
// code of mvf_kernels.hip, and of the self-test that runs it alone).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mvf_internal.h"

namespace mvf {

// ---------------------------------------------------------------------------
// Launch order of the raycast's tiles and each tile's level, from their last
// durations t (the longest block of a tile or of one next to it, scaled to
// level 0): a counting sort, longest first, by quarter octaves.  The levels
// follow from a bound on a block's duration, a tile taking the lowest level
// that keeps it, and the bound is the one for which kOrderTail times itself
// plus the whole work, shared by all the wavefronts that the device holds, is
// smallest.  (Any kOrderTail from 0.3 to 0.6 is as good: 128^3 at 320 x 240
// 21.5 us, one 512^3 volume at 640 x 480 46; with 1 it is 40 and 49, with 4
// 40 and 68.  Bounds by half octaves: 55 for 50 us.  Durations of the tile
// alone, without its neighbours: 78 us for 55, since a tile that was quick and
// became slow at a low level ends the launch late.)
// Run by one block of any size: each thread takes kOrderBatch tiles per
// round with all their loads in flight, and counts and places them with
// LDS atomics (aggregating a wavefront's lanes per bin with ballots first
// serialised the block: up to ~90 us per order in the integration launch's
// block 0, longer than the integration it runs beside).
constexpr int kOrderBins = 64;
constexpr int kOrderBatch = 8;
constexpr float kOrderTail = 0.5f;
constexpr int kOrderFloor = 1;   // levels below the uniform one that a tile may take

// Duration of a tile's longest block at level 0 over that at a level
static __device__ __forceinline__ float ray_speedup(int level)
{
    return level == 0 ? 1.0f : level == 1 ? 1.6f : level == 2 ? 2.4f : level == 3 ? 3.7f : 4.6f;
}
// the lowest level that keeps a tile of duration e at level 0 within th
static __device__ __forceinline__ int ray_level(float e, float th, int least)
{
    int l = 0;
#pragma unroll
    for (int q = 0; q < kRayLevels - 1; ++q) l += e > th * ray_speedup(q) ? 1 : 0;
    return max(l, least);
}
// the summed durations of such a tile's blocks at a level: 300 ticks for each, and
// what grows with the rounds
static __device__ __forceinline__ float ray_work(float e, int level)
{
    const float g = level == 0 ? 1.0f : level == 1 ? 1.5f : level == 2 ? 1.8f : level == 3 ? 2.15f : 2.7f;
    return 300.0f * (float)(1 << level) + fmaxf(e - 300.0f, 0.0f) * g;
}

// 0: not known; 1..63: quarter octaves from 16 ticks (0.16 us) to 10 ms
static __device__ __forceinline__ int cost_bin(uint32_t t)
{
    if (t == 0) return 0;
    const int e = 31 - __builtin_clz(max(t, 16u));
    return min(4 * (e - 4) + (int)(max(t, 16u) >> (e - 2) & 3u) + 1, kOrderBins - 1);
}

static __device__ __forceinline__ float bin_middle(int b)
{
    return b == 0 ? 0.0f : (1.125f + 0.25f * (float)((b - 1) & 3)) * (float)(16u << ((b - 1) >> 2));
}

// hist: kOrderBins words of LDS
static __device__ void tile_order_block(const TileOrder& O, int* hist)
{
    const int nt = blockDim.x;
    RayPlan* const plan = reinterpret_cast<RayPlan*>(O.order);
    int32_t* const order = O.order + kRayPlanInts;
    for (int i = threadIdx.x; i < kOrderBins; i += nt) hist[i] = 0;
    __syncthreads();
    uint32_t c[kOrderBatch];
    for (int pass = 0; pass < 2; ++pass) {
        for (int g0 = 0; g0 < O.tiles; g0 += kOrderBatch * nt) {
            // (a single round's costs stay in registers)
            if (pass == 0 || O.tiles > kOrderBatch * nt) {
#pragma unroll
                for (int k = 0; k < kOrderBatch; ++k) {
                    const int g = g0 + k * nt + (int)threadIdx.x;
                    c[k] = g < O.tiles && !O.fresh ? O.cost[g] : 0;
                }
            }
#pragma unroll
            for (int k = 0; k < kOrderBatch; ++k) {
                const int g = g0 + k * nt + (int)threadIdx.x;
                if (g >= O.tiles) continue;
                const int bin = cost_bin(c[k]);
                // the place within a bin is the atomics' order (the launch
                // order only steers the timing)
                if (pass == 0) {
                    atomicAdd(&hist[bin], 1);
                } else {
                    order[atomicAdd(&hist[bin], 1)] = g;
                    O.cost[g] = 0;
                }
            }
        }
        __syncthreads();
        if (pass == 0 && threadIdx.x < 64) {
            // lane b: bin 63 - b, so that the longest come first
            const int lane = threadIdx.x, b = kOrderBins - 1 - lane;
            const int n = hist[b];
            const bool unknown = hist[0] > 0;
            const int floor_level = max(O.level - kOrderFloor, 0);
            // lane c weighs the bound bin_middle(c)
            const float th = bin_middle(lane);
            float work = 0.0f, blocks = 0.0f;
            for (unsigned long long some = __ballot(n > 0); some; some &= some - 1) {
                const int q = __builtin_ctzll(some);
                const float m = (float)__builtin_amdgcn_readlane(n, q), e = bin_middle(kOrderBins - 1 - q);
                const int l = ray_level(e, th, floor_level);
                work += m * ray_work(e, l);
                blocks += m * (float)(1 << l);
            }
            float best = blocks <= (float)(O.max_blocks - kRaySlack) ? kOrderTail * th * (float)O.slots + work : INFINITY;
            int at = lane;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const float y = __shfl_xor(best, o);
                const int z = __shfl_xor(at, o);
                if (y < best || (y == best && z < at)) { best = y; at = z; }
            }
            const int level = unknown ? O.level : best < INFINITY ? ray_level(bin_middle(b), bin_middle(at), floor_level) : floor_level;
            // positions: exclusive sums over the lanes
            int sum = n;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(sum, o);
                if (lane >= o) sum += y;
            }
            hist[b] = sum - n;
            // first position of each level, on a whole window of tiles
            int pos = 0, blk = 0;
#pragma unroll
            for (int l = kRayLevels - 1; l >= 0; --l) {
                if (lane == 0) { plan->pos[l] = pos; plan->block[l] = blk; }
                // tiles at this level or above
                const unsigned long long m = __ballot(level >= l);
                const int upto = l == 0 ? O.tiles : m ? __shfl(sum, 63 - __builtin_clzll(m)) : 0;
                const int end = min((upto + kXcds - 1) / kXcds * kXcds, O.tiles);
                if (end > pos) {
                    blk += (end - pos + kXcds - 1) / kXcds * kXcds << l;
                    pos = end;
                }
            }
            if (lane == 0) plan->block[kRayLevels] = blk;
        }
        __syncthreads();
    }
}

}  // namespace mvf
