// Camera tracking kernels for gfx950 (Depth Map Conversion and Camera
// Tracking sections of Salvato, Finman, Leonard, arXiv 1511.07106; the
// tracker is KinectFusion's projective point-to-plane ICP, which the paper
// cites).  Built with -ffp-contract=off and IEEE division/sqrt: every
// decision (pixel validity, the model pixel a vertex projects to, the
// distance and normal tests) is the binary32 contract of the CPU reference;
// residuals, Jacobians and the normal-equation sums are binary64.
//
// One Gauss-Newton step is one launch: its blocks associate pixels and reduce
// their pairs' 6x6 system to binary64 partials, and the last block to finish
// sums the partials in a fixed order, solves the system by Cholesky and moves
// the pose estimate, which stays in device memory.  A whole coarse-to-fine run
// is enqueued without a host round trip.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mvf_internal.h"

namespace mvf {

static __device__ __forceinline__ bool depth_valid(float d) { return d > 0.0f && d <= 3.4e38f; }

static __device__ __forceinline__ float qnanf() { return __builtin_nanf(""); }

// Edge-preserving smoothing before the pyramid: for a valid pixel the
// binomial-weighted (C(6, dx + 3) C(6, dy + 3)) mean of the valid depths of
// its 7x7 window inside the image within delta of its own depth; invalid
// pixels give 0.  Binary32, the window row by row (the weights and their
// sums are small integers, exact).  A 16x16 tile of pixels reads its
// 22x22 neighbourhood from LDS, where a depth that is not valid is a NaN: one
// comparison then decides a tap, and a tap left out adds zero instead of
// branching (640x480: 8.7 -> 6.2 us).
__global__ __launch_bounds__(256) void mvf_track_smooth_kernel(const float* __restrict__ D, int pitch, int w, int h,
                                                               float delta, float* __restrict__ out)
{
    __shared__ float tile[22][23];
    const int x0 = blockIdx.x * 16 - 3, y0 = blockIdx.y * 16 - 3;
    for (int i = threadIdx.x; i < 22 * 22; i += 256) {
        const int ty = i / 22, tx = i - ty * 22;
        const int xx = x0 + tx, yy = y0 + ty;
        const float d = (xx >= 0 && xx < w && yy >= 0 && yy < h) ? D[(size_t)yy * pitch + xx] : 0.0f;
        tile[ty][tx] = depth_valid(d) ? d : qnanf();
    }
    __syncthreads();
    const int lx = threadIdx.x & 15, ly = threadIdx.x >> 4;
    const int x = blockIdx.x * 16 + lx, y = blockIdx.y * 16 + ly;
    if (x >= w || y >= h) return;
    const float d0 = tile[ly + 3][lx + 3];
    const float c6[7] = { 1.0f, 6.0f, 15.0f, 20.0f, 15.0f, 6.0f, 1.0f };
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int dy = 0; dy < 7; ++dy)
#pragma unroll
        for (int dx = 0; dx < 7; ++dx) {
            const float d = tile[ly + dy][lx + dx];
            const bool take = fabsf(d - d0) <= delta;
            const float wt = c6[dx] * c6[dy];
            num = num + wt * (take ? d : 0.0f);
            den = den + (take ? wt : 0.0f);
        }
    const float r = __builtin_isnan(d0) ? 0.0f : num / den;
    out[(size_t)y * w + x] = r;
}

// Level l+1 depth (floor(w/2) x floor(h/2)): mean of the valid depths of the
// 2x2 block within tau of the block's first valid one (order (0,0), (1,0),
// (0,1), (1,1)), 0 when the block has none.
__global__ __launch_bounds__(256) void mvf_track_down_kernel(const float* __restrict__ D, int pitch, int w, int h,
                                                             float tau, float* __restrict__ D2)
{
    const int w2 = w / 2, h2 = h / 2;
    const int x = blockIdx.x * 16 + (threadIdx.x & 15);
    const int y = blockIdx.y * 16 + (threadIdx.x >> 4);
    if (x >= w2 || y >= h2) return;
    const float q[4] = { D[(size_t)(2 * y) * pitch + 2 * x], D[(size_t)(2 * y) * pitch + 2 * x + 1],
                         D[(size_t)(2 * y + 1) * pitch + 2 * x], D[(size_t)(2 * y + 1) * pitch + 2 * x + 1] };
    bool have = false;
    float ref = 0.0f, sum = 0.0f;
    int n = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (!depth_valid(q[k])) continue;
        if (!have) { ref = q[k]; have = true; }
        if (fabsf(q[k] - ref) <= tau) { sum = sum + q[k]; ++n; }
    }
    D2[(size_t)y * w2 + x] = n ? sum / (float)n : 0.0f;
}

static __device__ __forceinline__ void vertex_at(const float* D, int pitch, int x, int y, float fx, float fy,
                                                 float cx, float cy, float v[3])
{
    const float d = D[(size_t)y * pitch + x];
    if (!depth_valid(d)) { v[0] = v[1] = v[2] = qnanf(); return; }
    v[0] = (((float)x - cx) / fx) * d;
    v[1] = (((float)y - cy) / fy) * d;
    v[2] = d;
}

// Vertex map v = K^-1 [x y 1]^T D and normal map n = (v(x+1,y) - v(x,y)) x
// (v(x,y+1) - v(x,y)), normalised (camera frame, NaN where undefined).
static __device__ __forceinline__ void vertex_normal(const TrackMapLevel& L, int x, int y)
{
    const size_t p = (size_t)y * L.w + x;
    float v00[3];
    vertex_at(L.D, L.pitch, x, y, L.fx, L.fy, L.cx, L.cy, v00);
    float n[3] = { qnanf(), qnanf(), qnanf() };
    if (!__builtin_isnan(v00[2]) && x + 1 < L.w && y + 1 < L.h) {
        float v10[3], v01[3];
        vertex_at(L.D, L.pitch, x + 1, y, L.fx, L.fy, L.cx, L.cy, v10);
        vertex_at(L.D, L.pitch, x, y + 1, L.fx, L.fy, L.cx, L.cy, v01);
        if (!__builtin_isnan(v10[2]) && !__builtin_isnan(v01[2])) {
            const float a[3] = { v10[0] - v00[0], v10[1] - v00[1], v10[2] - v00[2] };
            const float b[3] = { v01[0] - v00[0], v01[1] - v00[1], v01[2] - v00[2] };
            const float c[3] = { (a[1] * b[2]) - (a[2] * b[1]), (a[2] * b[0]) - (a[0] * b[2]),
                                 (a[0] * b[1]) - (a[1] * b[0]) };
            const float len = sqrtf(((c[0] * c[0]) + (c[1] * c[1])) + (c[2] * c[2]));
            if (len > 0.0f) {
                n[0] = c[0] / len;
                n[1] = c[1] / len;
                n[2] = c[2] / len;
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        L.V[3 * p + a] = v00[a];
        L.N[3 * p + a] = n[a];
    }
}

// All maps of a tracking call in one launch (each is a few microseconds of
// latency on its own), numbered by M.first: map z < levels is the vertex and
// normal map of that level, the rest are the model maps of levels 1 .., level
// l taking the sample (2^l x, 2^l y) of the full-size model.  Block 0 also
// sets up the call's state.
__global__ __launch_bounds__(256) void mvf_track_maps_kernel(TrackMaps M)
{
    if (M.state && blockIdx.x == 0) {
        if (threadIdx.x < 12) {
            M.state->T[threadIdx.x] = M.T[threadIdx.x];
            M.state->T32[threadIdx.x] = (float)M.T[threadIdx.x];
        }
        if (threadIdx.x == 0) {
            M.state->steps = 0;
            M.state->ticket = 0;
        }
    }
    int z = 0;
    while (z + 1 < kTrackMapsMax && (int)blockIdx.x >= M.first[z + 1]) ++z;
    const int block = (int)blockIdx.x - M.first[z];
    const int tiles_x = (M.level[z < M.levels ? z : z - M.levels + 1].w + 15) / 16;
    const int ty = block / tiles_x, tx = block - ty * tiles_x;
    const int x = tx * 16 + (threadIdx.x & 15);
    const int y = ty * 16 + (threadIdx.x >> 4);
    if (z < M.levels) {
        const TrackMapLevel& L = M.level[z];
        if (x < L.w && y < L.h) vertex_normal(L, x, y);
        return;
    }
    const int l = z - M.levels + 1;
    const TrackMapLevel& L = M.level[l];
    if (x >= L.w || y >= L.h) return;
    const size_t s = ((size_t)y << l) * M.level[0].w + ((size_t)x << l), d = (size_t)y * L.w + x;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        L.Vm[3 * d + a] = M.Vm[3 * s + a];
        L.Nm[3 * d + a] = M.Nm[3 * s + a];
    }
}

// Left-multiplied SE(3) exponential Exp(xi) T, xi = (rho, omega), binary64.
static __device__ __forceinline__ void se3_left_update(const double xi[6], double T[12])
{
    const double w0 = xi[3], w1 = xi[4], w2 = xi[5];
    const double th = sqrt(w0 * w0 + w1 * w1 + w2 * w2);
    const double W[9] = { 0.0, -w2, w1, w2, 0.0, -w0, -w1, w0, 0.0 };
    double W2[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) W2[3 * i + j] = W[3 * i] * W[j] + W[3 * i + 1] * W[3 + j] + W[3 * i + 2] * W[6 + j];
    double a, b, c;
    if (th < 1e-10) {
        a = 1.0;
        b = 0.5;
        c = 1.0 / 6.0;
    } else {
        const double s = sin(th), co = cos(th);
        a = s / th;
        b = (1.0 - co) / (th * th);
        c = (th - s) / (th * th * th);
    }
    double R[9], Vm[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double I = (i % 4 == 0) ? 1.0 : 0.0;
        R[i] = I + a * W[i] + b * W2[i];
        Vm[i] = I + b * W[i] + c * W2[i];
    }
    double t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) t[i] = Vm[3 * i] * xi[0] + Vm[3 * i + 1] * xi[1] + Vm[3 * i + 2] * xi[2];
    double out[12];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            out[4 * i + j] = R[3 * i] * T[j] + R[3 * i + 1] * T[4 + j] + R[3 * i + 2] * T[8 + j];
        out[4 * i + 3] = R[3 * i] * T[3] + R[3 * i + 1] * T[7] + R[3 * i + 2] * T[11] + t[i];
    }
#pragma unroll
    for (int i = 0; i < 12; ++i) T[i] = out[i];
}

// Value i of the 32 a wavefront's lanes hold (x[i]), summed over the lanes, in
// lanes 2 i and 2 i + 1.  The pairing is that of adding lane + 32, + 16, ...,
// + 1 in turn, but a step keeps only half of the values in each half of the
// lanes: 32 exchanges where one tree per value takes 192.
template <int N>
static __device__ __forceinline__ void halve_sums(double (&x)[32], int lane)
{
    const bool up = (lane & (2 * N)) != 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double keep = up ? x[N + i] : x[i];
        const double give = up ? x[i] : x[N + i];
        x[i] = keep + __shfl_xor(give, 2 * N);
    }
}

static __device__ __forceinline__ double wave_sums32(double (&x)[32], int lane)
{
    halve_sums<16>(x, lane);
    halve_sums<8>(x, lane);
    halve_sums<4>(x, lane);
    halve_sums<2>(x, lane);
    halve_sums<1>(x, lane);
    return x[0] + __shfl_xor(x[0], 1);
}

// The Gauss-Newton update from a step's sums: solve A xi = -b by Cholesky,
// T <- Exp(xi) T.  Fewer than 6 pairs, or an A that is not positive definite,
// leave T as it is.  Every loop is unrolled, so the matrices stay in registers.
static __device__ __forceinline__ void solve_update(const double* tot, TrackState* state)
{
    const int pairs = (int)tot[27];
    if (pairs < 6) return;
    double A[6][6], L[6][6], y[6], xi[6];
    int k = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = i; j < 6; ++j) { A[i][j] = tot[k]; A[j][i] = tot[k]; ++k; }
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double s = A[j][j];
#pragma unroll
        for (int q = 0; q < j; ++q) s -= L[j][q] * L[j][q];
        ok = ok && s > 0.0;
        L[j][j] = sqrt(s);
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            double t = A[i][j];
#pragma unroll
            for (int q = 0; q < j; ++q) t -= L[i][q] * L[j][q];
            L[i][j] = t / L[j][j];
        }
    }
    if (!ok) return;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        double s = -tot[21 + i];
#pragma unroll
        for (int q = 0; q < i; ++q) s -= L[i][q] * y[q];
        y[i] = s / L[i][i];
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double s = y[i];
#pragma unroll
        for (int q = i + 1; q < 6; ++q) s -= L[q][i] * xi[q];
        xi[i] = s / L[i][i];
    }
    double T[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) T[i] = state->T[i];
    se3_left_update(xi, T);
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        state->T[i] = T[i];
        state->T32[i] = (float)T[i];
    }
}

// One Gauss-Newton step over the current maps (w x h).  Per block the sums of
// its pairs (A upper triangle 21, b 6, pairs, sum r^2) go to
// partials[block * kTrackSums ...]; the last block to finish sums them in a fixed
// order, writes the step's statistics and updates the estimate.
//
// Bound: load latency, the chain own maps -> model maps -> reduction -> solve.
// So a thread's four pixels are loaded together and their model samples
// gathered together, and the last block adds the partials in eight runs side by
// side, a lane's loads in flight together (in one run, 300 additions one after
// the other, the sum took 4.7 us of a step).  13 us a step at 640x480: before,
// 16.5; as an association kernel of 14 us, whose threads took one pixel after
// the other, and a solve kernel of 71 us, whose lanes read the partials from
// memory one by one, 85.
//
// The partials cross the XCDs' L2 caches: they are stored and loaded with
// device-scope atomics, and a block takes its ticket when its stores have
// reached that scope.  (A fence would write the whole L2 back, once a block.)
constexpr int kSegLanes = 32;                            // lanes of a run of blocks, one per sum
constexpr int kSegments = kTrackThreads / kSegLanes;
constexpr int kSegLoads = 20;                            // a lane's loads in flight
static_assert(kTrackSums <= kSegLanes, "one lane per sum");
__global__ __launch_bounds__(kTrackThreads) void mvf_icp_step_kernel(TrackLaunch L, int nblocks, int step,
                                                                     TrackState* out)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    __shared__ double part[kTrackThreads / 64][kTrackSums];
    __shared__ double seg_sum[kSegments][kTrackSums];
    __shared__ double tot[kTrackSums];
    __shared__ bool last;
    double acc[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i] = 0.0;
    float T[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) T[i] = L.state->T32[i];
    const float* Tm = L.Tm;
    const float e2 = L.eps_d * L.eps_d;
    const int npix = L.w * L.h;
    const int base = blockIdx.x * kTrackThreads * kTrackPixPerThread;
    float v[kTrackPixPerThread][3], n[kTrackPixPerThread][3];
#pragma unroll
    for (int k = 0; k < kTrackPixPerThread; ++k) {
        // past the image: the last pixel, dropped below
        const int p = min(base + k * kTrackThreads + (int)threadIdx.x, npix - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[k][a] = L.V[3 * p + a];
            n[k][a] = L.N[3 * p + a];
        }
    }
    // keep the four pixels' loads, and below their gathers, together: left to
    // itself the compiler waits for each pixel's in turn
    __builtin_amdgcn_sched_barrier(0);
    // camera to world to the model's pixel; a pixel without a vertex, a normal
    // or a model pixel reads sample 0 and is dropped below
    bool in[kTrackPixPerThread];
    float vm[kTrackPixPerThread][3], nm[kTrackPixPerThread][3];
#pragma unroll
    for (int k = 0; k < kTrackPixPerThread; ++k) {
        bool ok = base + k * kTrackThreads + (int)threadIdx.x < npix;
        float vg[3], ng[3], d[3], q[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            ok = ok && !__builtin_isnan(v[k][a]) && !__builtin_isnan(n[k][a]);
            vg[a] = (((T[4 * a] * v[k][0]) + (T[4 * a + 1] * v[k][1])) + (T[4 * a + 2] * v[k][2])) + T[4 * a + 3];
            ng[a] = ((T[4 * a] * n[k][0]) + (T[4 * a + 1] * n[k][1])) + (T[4 * a + 2] * n[k][2]);
            d[a] = vg[a] - Tm[4 * a + 3];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) q[a] = ((Tm[a] * d[0]) + (Tm[4 + a] * d[1])) + (Tm[8 + a] * d[2]);
        const float iz = 1.0f / q[2];
        const float ur = floorf((((L.fx * q[0]) * iz) + L.cx) + 0.5f);
        const float vr = floorf((((L.fy * q[1]) * iz) + L.cy) + 0.5f);
        ok = ok && q[2] > 0.0f && ur >= 0.0f && ur <= (float)(L.w - 1) && vr >= 0.0f && vr <= (float)(L.h - 1);
        in[k] = ok;
        const size_t m = ok ? (size_t)vr * L.w + (size_t)ur : 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            vm[k][a] = L.Vm[3 * m + a];
            nm[k][a] = L.Nm[3 * m + a];
            v[k][a] = vg[a];
            n[k][a] = ng[a];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kTrackPixPerThread; ++k) {
        bool ok = in[k];
#pragma unroll
        for (int a = 0; a < 3; ++a) ok = ok && !__builtin_isnan(vm[k][a]) && !__builtin_isnan(nm[k][a]);
        const float dv[3] = { v[k][0] - vm[k][0], v[k][1] - vm[k][1], v[k][2] - vm[k][2] };
        const float dist2 = ((dv[0] * dv[0]) + (dv[1] * dv[1])) + (dv[2] * dv[2]);
        const float dot = ((n[k][0] * nm[k][0]) + (n[k][1] * nm[k][1])) + (n[k][2] * nm[k][2]);
        ok = ok && dist2 <= e2 && fabsf(dot) >= L.cos_theta;
        if (!ok) continue;
        const double g[3] = { v[k][0], v[k][1], v[k][2] };
        const double nn[3] = { nm[k][0], nm[k][1], nm[k][2] };
        const double r = nn[0] * (g[0] - (double)vm[k][0]) + nn[1] * (g[1] - (double)vm[k][1]) +
                         nn[2] * (g[2] - (double)vm[k][2]);
        const double J[6] = { nn[0], nn[1], nn[2], g[1] * nn[2] - g[2] * nn[1], g[2] * nn[0] - g[0] * nn[2],
                              g[0] * nn[1] - g[1] * nn[0] };
        int kk = 0;
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = i; j < 6; ++j) acc[kk++] += J[i] * J[j];
#pragma unroll
        for (int i = 0; i < 6; ++i) acc[21 + i] += J[i] * r;
        acc[27] += 1.0;
        acc[28] += r * r;
    }
    // wavefront tree (fixed pairing), then the block's waves in order
    const double sum = wave_sums32(acc, lane);
    if (!(lane & 1) && (lane >> 1) < kTrackSums) part[wave][lane >> 1] = sum;
    __syncthreads();
    if (threadIdx.x < kTrackSums) {
        double s = 0.0;
#pragma unroll
        for (int wv = 0; wv < kTrackThreads / 64; ++wv) s += part[wv][threadIdx.x];
        __hip_atomic_store(&L.partials[(size_t)blockIdx.x * kTrackSums + threadIdx.x], s, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&L.state->ticket, 1u) + 1 == (uint32_t)nblocks;
    __syncthreads();
    if (!last) return;
    // the step's sums, one lane per sum: the blocks in kSegments runs, each in
    // order, then the runs in order
    {
        const int sum = threadIdx.x % kSegLanes, seg = threadIdx.x / kSegLanes;
        const int per = (nblocks + kSegments - 1) / kSegments;
        const int b1 = min(nblocks, (seg + 1) * per);
        double s = 0.0;
        for (int b0 = seg * per; b0 < b1; b0 += kSegLoads) {
            double x[kSegLoads];
#pragma unroll
            for (int i = 0; i < kSegLoads; ++i)
                x[i] = b0 + i < b1 && sum < kTrackSums
                           ? __hip_atomic_load(&L.partials[(size_t)(b0 + i) * kTrackSums + sum], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT)
                           : 0.0;
#pragma unroll
            for (int i = 0; i < kSegLoads; ++i) s += x[i];
        }
        if (sum < kTrackSums) seg_sum[seg][sum] = s;
    }
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x < kTrackSums) {
#pragma unroll
        for (int i = 0; i < kSegments; ++i) s += seg_sum[i][threadIdx.x];
    }
    if (threadIdx.x < kTrackSums) tot[threadIdx.x] = s;
    __syncthreads();
    TrackState* state = L.state;
    if (threadIdx.x == 0) {
        state->ticket = 0;
        state->pairs[step] = (int)tot[27];
        state->sq_err[step] = tot[28];
        state->steps = step + 1;
        solve_update(tot, state);
    }
    if (!out) return;
    // the call's result, to the host
    __syncthreads();
    if (threadIdx.x < 12) out->T[threadIdx.x] = state->T[threadIdx.x];
    if (threadIdx.x <= (unsigned)step && threadIdx.x < kTrackMaxSteps) {
        out->pairs[threadIdx.x] = state->pairs[threadIdx.x];
        out->sq_err[threadIdx.x] = state->sq_err[threadIdx.x];
    }
    if (threadIdx.x == 0) out->steps = step + 1;
}

int launch_track_smooth(const float* D, int pitch, int w, int h, float delta, float* out, void* stream)
{
    dim3 grid((w + 15) / 16, (h + 15) / 16);
    hipLaunchKernelGGL(mvf_track_smooth_kernel, grid, dim3(256), 0, (hipStream_t)stream, D, pitch, w, h, delta, out);
    return (int)hipGetLastError();
}

int launch_track_down(const float* D, int pitch, int w, int h, float tau, float* D2, void* stream)
{
    dim3 grid((w / 2 + 15) / 16, (h / 2 + 15) / 16);
    if (grid.x == 0 || grid.y == 0) return 0;
    hipLaunchKernelGGL(mvf_track_down_kernel, grid, dim3(256), 0, (hipStream_t)stream, D, pitch, w, h, tau, D2);
    return (int)hipGetLastError();
}

int launch_track_maps(TrackMaps M, void* stream)
{
    if (M.levels < 1 || M.levels > 3) return (int)hipErrorInvalidValue;
    const int maps = M.levels + (M.Vm ? M.levels - 1 : 0);
    int blocks = 0;
    for (int z = 0; z < kTrackMapsMax; ++z) {
        M.first[z] = z < maps ? blocks : 0x7fffffff;
        if (z >= maps) continue;
        const TrackMapLevel& L = M.level[z < M.levels ? z : z - M.levels + 1];
        blocks += ((L.w + 15) / 16) * ((L.h + 15) / 16);
    }
    hipLaunchKernelGGL(mvf_track_maps_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, M);
    return (int)hipGetLastError();
}

int track_blocks(int w, int h)
{
    return (w * h + kTrackThreads * kTrackPixPerThread - 1) / (kTrackThreads * kTrackPixPerThread);
}

int launch_icp_step(const TrackLaunch& L, int step, TrackState* out, void* stream)
{
    const int nb = track_blocks(L.w, L.h);
    if (nb <= 0 || step < 0 || step >= kTrackMaxSteps) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(mvf_icp_step_kernel, dim3(nb), dim3(kTrackThreads), 0, (hipStream_t)stream, L, nb, step, out);
    return (int)hipGetLastError();
}

}  // namespace mvf
