// krt_image.hip -- deterministic ray-tracing imaging pass (Sec. 2.2.2): the
// formal solution of eq. imaging-formal along lines of sight toward a camera
// on a grid axis, in every Doppler channel, over the scattering emissivity
// that the Monte Carlo pass tallied toward that camera.
//
// Per cell and channel k, from the far side of the grid to the camera:
//   I <- I exp(-dtau_k) + j_k dl (1 - exp(-dtau_k)) / dtau_k + S_emis,k (1 - exp(-dtau_k)),
//   dtau_k = (k0 H(a, x_k - n_cam.v) + kappa_abs) dl   (eq. imaging-alphas; kappa_abs
//   an optional grey absorption, zero when absent),
// with x_k the lab-frame centre of channel k.
//
// Layout.  One lane per pixel and channel, or per pixel and four consecutive
// channels (image_plan says where), so the lanes of a wave read the emissivity of consecutive
// channels from consecutive addresses and a cell's fields at one address per
// pixel of the wave: the pass streams the emissivity array once.  The
// Voigt table sits in LDS.  The recurrence is affine in I, so a ray can be
// cut into segments: the wave of segment s folds its cells into a map
// I -> A_s I + B_s, and the maps are composed in order, far side first,
// through LDS.  Short rays on small grids take several segments so that the
// launch still fills the chip; long ones take one.  A wave issues the loads
// of a chunk of cells together and then folds them in order (the march is a
// dependent chain, its memory is not).
//
// Memory bounds it: along z and y the cells of a ray are megabytes apart, and
// what counts is how much a wave takes from each place.  128^3 x 64 channels,
// velocity, source function and absorption, toward -z (1.1 GB): 247 us with
// one channel a lane (256 bytes a cell and wave), 205 us with four (1 KB; by
// the kernel's own events, as all figures here; 222 us in a trace of first
// passes, 5.0 TB/s, near the rate of a copy).  More waves with shorter chunks
// (eight per SIMD) only spread the same reads over more places: 400 us.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "krt_internal.h"
#include "krt_kernels.h"
#include "krt_device.h"
#include "krt_image.h"

namespace krt {

constexpr int kImgVoigtFloats = kOffVoigtWing + 4 * kVoigtWingN;  // core and wing of H(a, x)
// cells whose loads are in flight together
template <int V>
constexpr int kImgChunk = V == 1 ? 8 : 4;
constexpr int kImgWaves = 8;            // waves per block
constexpr int kImgMaxSeg = kImgWaves;   // segments of one ray (waves of one block)
constexpr int kImgMinSegCells = 4;      // shortest segment worth a wave
constexpr int64_t kImgTargetWaves = 16384;  // twice the chip's resident waves at 8 per SIMD, at one channel a lane
constexpr int64_t kImgQuadWaves = 2048;     // two per SIMD of 256 compute units

// fields of a chunk of cells along the ray (the arrays a kernel instance does
// not read are never written and cost nothing)
template <int V>
struct ImgChunk {
    float k0[kImgChunk<V>], v[kImgChunk<V>], ab[kImgChunk<V>], j[kImgChunk<V>][V], s[kImgChunk<V>][V];
};

// V consecutive channels.  Four a lane are read as a stream (128^3 x 64 with
// source toward +y: 168 us, plain 181); with one a lane other waves read the
// rest of a line (100^3 x 9 channels: 33 us plain, 37 us as a stream).
template <int V>
__device__ __forceinline__ void img_stream(const float *p, float (&o)[V]) {
    typedef float vec __attribute__((ext_vector_type(V), aligned(4)));
    vec x;
    if constexpr (V == 1) x = *reinterpret_cast<const vec *>(p);
    else x = __builtin_nontemporal_load(reinterpret_cast<const vec *>(p));
#pragma unroll
    for (int k = 0; k < V; ++k) o[k] = x[k];
}

// loads of cells t .. t + M - 1 of the segment; cell t sits at offset o
// (fields) and o * nch (channels)
template <int V, bool kVel, bool kAbs, bool kSrc, int M>
__device__ __forceinline__ void img_load(const ImageParams &Q, int64_t o, int64_t step, int64_t cstep,
                                         const float *pe, const float *ps, ImgChunk<V> &b) {
#pragma unroll
    for (int u = 0; u < M; ++u) {
        const int64_t oc = o + u * step;
        b.k0[u] = Q.k0[oc];
        if constexpr (kVel) b.v[u] = Q.vel_axis[oc];
        if constexpr (kAbs) b.ab[u] = Q.kabs[oc];
        img_stream<V>(pe + u * cstep, b.j[u]);
        if constexpr (kSrc) img_stream<V>(ps + u * cstep, b.s[u]);
    }
}

// H(a, |x|) from the core / wing table in LDS, without a branch: the lanes
// of a wave span channels on both sides of |x| = 8, so the two pieces share
// one address computation and one LDS read
__device__ __forceinline__ float img_voigt(const float *T, float xa) {
    const bool core = xa < 8.0f;
    const float w = 8.0f * f_rcp(xa);
    const float t = core ? xa * 64.0f : w * (float)kVoigtWingN;
    const int i = max(0, min((int)t, core ? kVoigtCoreN - 1 : kVoigtWingN - 1));
    const float f = t - (float)i;
    const float4 c = *reinterpret_cast<const float4 *>(T + (core ? kOffVoigtCore : kOffVoigtWing) + 4 * i);
    const float G = fmaf(f, fmaf(f, fmaf(f, c.w, c.z), c.y), c.x);
    return core ? G : G * w * w * (1.0f / 64.0f);
}

template <int V, bool kVel, bool kAbs, bool kSrc, int M>
__device__ __forceinline__ void img_fold(const ImageParams &Q, const float *TV, const float (&xk)[V],
                                         const ImgChunk<V> &b, float (&A)[V], float (&B)[V]) {
#pragma unroll
    for (int u = 0; u < M; ++u)
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const float xg = kVel ? xk[k] - Q.sgnf * b.v[u] : xk[k];
            const float H = (b.k0[u] > 0.0f) ? img_voigt(TV, fabsf(xg)) : 0.0f;
            const float dtau = (kAbs ? fmaf(b.k0[u], H, b.ab[u]) : b.k0[u] * H) * Q.dl;
            const float att = f_exp(-dtau);
            // (1 - e^{-dtau}) / dtau, with its series below 1e-3
            const float frac = (dtau < 1e-3f) ? 1.0f - dtau * (0.5f - dtau * (1.0f / 6.0f)) : (1.0f - att) * f_rcp(dtau);
            B[k] = fmaf(B[k], att, b.j[u][k] * Q.dl * frac);
            if constexpr (kSrc) B[k] = fmaf(b.s[u][k], dtau * frac, B[k]);
            A[k] *= att;
        }
}

template <int V, bool kVel, bool kAbs, bool kSrc>
__device__ __forceinline__ void image_body(const ImageParams &Q, int nseg, int seglen) {
    __shared__ float4 tv4[kImgVoigtFloats / 4];
    __shared__ float2 part[kImgWaves][V][64];  // (A_s, B_s) of every wave's segment
    float *TV = reinterpret_cast<float *>(tv4);
    const float4 *src = reinterpret_cast<const float4 *>(Q.tab);
    for (int i = threadIdx.x; i < kImgVoigtFloats / 4; i += blockDim.x) tv4[i] = src[i];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int seg = wave % nseg;                // segment of the ray, far side = 0
    const int grp = wave / nseg;                // group of 64 lanes' (pixel, V channels)
    const int64_t tid = ((int64_t)blockIdx.x * (kImgWaves / nseg) + grp) * 64 + lane;
    const int per = (Q.nch + V - 1) / V;        // lanes of a pixel
    const int64_t pix = tid / per;
    // the last lane of a pixel takes its last V channels: where V does not
    // divide nch it repeats some of its neighbour's, to the same bits
    const int c = min((int)(tid - pix * per) * V, Q.nch - V);
    const bool live = pix < Q.npix;
    // an index, not an address: that costs a spill at 64 registers
    const int64_t at = V == 1 ? tid : pix * Q.nch + c;
    float A[V], B[V];
#pragma unroll
    for (int k = 0; k < V; ++k) { A[k] = 1.0f; B[k] = 0.0f; }
    if (live) {
        // pixel -> first cell of its column and the stride along the ray
        const int p0 = (int)(pix % Q.n0), p1 = (int)(pix / Q.n0);
        int64_t cell0;
        if (Q.d == 0) cell0 = ((int64_t)p1 * Q.n[1] + p0) * Q.n[0];           // (k, j)
        else if (Q.d == 1) cell0 = (int64_t)p1 * Q.n[1] * Q.n[0] + p0;         // (k, i)
        else cell0 = (int64_t)p1 * Q.n[0] + p0;                                // (j, i)
        const int nl = Q.n[Q.d];
        const int t0 = seg * seglen, t1 = min(nl, t0 + seglen);
        // step t (far side first) is cell s = t toward +axis cameras, nl - 1 - t otherwise
        const int64_t step = Q.sgn > 0 ? Q.stride : -Q.stride;
        const int64_t cstep = step * Q.nch;
        int64_t o = cell0 + (int64_t)(Q.sgn > 0 ? t0 : nl - 1 - t0) * Q.stride;
        const float *pe = Q.emis + o * Q.nch + c;
        const float *ps = kSrc ? Q.srcf + o * Q.nch + c : nullptr;
        float xk[V];
#pragma unroll
        for (int k = 0; k < V; ++k) xk[k] = Q.ch_lo + ((float)(c + k) + 0.5f) * Q.ch_w;
        const int nfull = max(0, t1 - t0) / kImgChunk<V>;
        ImgChunk<V> cur{};
        for (int i = 0; i < nfull; ++i) {
            img_load<V, kVel, kAbs, kSrc, kImgChunk<V>>(Q, o, step, cstep, pe, ps, cur);
            img_fold<V, kVel, kAbs, kSrc, kImgChunk<V>>(Q, TV, xk, cur, A, B);
            o += kImgChunk<V> * step;
            pe += kImgChunk<V> * cstep;
            if constexpr (kSrc) ps += kImgChunk<V> * cstep;
        }
        for (int t = t0 + nfull * kImgChunk<V>; t < t1; ++t) {  // ragged end of the segment
            img_load<V, kVel, kAbs, kSrc, 1>(Q, o, step, cstep, pe, ps, cur);
            img_fold<V, kVel, kAbs, kSrc, 1>(Q, TV, xk, cur, A, B);
            o += step;
            pe += cstep;
            if constexpr (kSrc) ps += cstep;
        }
    }
    if (nseg == 1) {
        if (live) {
#pragma unroll
            for (int k = 0; k < V; ++k) Q.out[at + k] = B[k];
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < V; ++k) part[wave][k][lane] = make_float2(A[k], B[k]);
    __syncthreads();
    if (seg == 0 && live) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
            float I = 0.0f;
            for (int s = 0; s < nseg; ++s) {
                const float2 p = part[wave + s][k][lane];
                I = fmaf(p.x, I, p.y);
            }
            Q.out[at + k] = I;
        }
    }
}

// Without a source function the fold of one channel a lane fits the register
// budget of eight waves per SIMD (64 VGPRs), the occupancy that hides the
// memory latency; the others would spill and keep the compiler's budget.
template <bool kVel, bool kAbs>
__global__ void __launch_bounds__(64 * kImgWaves) __attribute__((amdgpu_waves_per_eu(8, 8)))
image_kernel(ImageParams Q, int nseg, int seglen) {
    image_body<1, kVel, kAbs, false>(Q, nseg, seglen);
}

template <bool kVel, bool kAbs>
__global__ void __launch_bounds__(64 * kImgWaves) image_src_kernel(ImageParams Q, int nseg, int seglen) {
    image_body<1, kVel, kAbs, true>(Q, nseg, seglen);
}

template <bool kVel, bool kAbs>
__global__ void __launch_bounds__(64 * kImgWaves) image_quad_kernel(ImageParams Q, int nseg, int seglen) {
    image_body<4, kVel, kAbs, false>(Q, nseg, seglen);
}

// Three waves per SIMD (one workgroup per compute unit), although 127 registers
// would allow four: 128^3 x 64 toward -z 202 us with three, 220 with four.
template <bool kVel, bool kAbs>
__global__ void __launch_bounds__(64 * kImgWaves) __attribute__((amdgpu_waves_per_eu(3, 3)))
image_quad_src_kernel(ImageParams Q, int nseg, int seglen) {
    image_body<4, kVel, kAbs, true>(Q, nseg, seglen);
}

struct ImgPlan {
    int v, nseg;
    int64_t groups;  // waves per segment
};

// Channels a lane and segments of a ray: segments are doubled while the launch
// has fewer waves than keep the chip busy and they stay at least
// kImgMinSegCells cells long.
static ImgPlan image_plan(int64_t npix, int nch, int nl, int v) {
    ImgPlan p{v, 1, (npix * ((nch + v - 1) / v) + 63) / 64};
    while (p.nseg < kImgMaxSeg && p.groups * p.nseg < kImgTargetWaves / v &&
           (nl + 2 * p.nseg - 1) / (2 * p.nseg) >= kImgMinSegCells)
        p.nseg *= 2;
    return p;
}

static int64_t image_blocks(const ImgPlan &p) { return (p.groups * p.nseg + kImgWaves - 1) / kImgWaves; }

// How full the chip is on average over a launch of `blocks` workgroups, `round`
// of which are resident: a few past a full round take as long as a whole one.
static double image_fill(int64_t blocks, int64_t round) {
    return (double)blocks / (double)(round * ((blocks + round - 1) / round));
}

// Four channels a lane (16-byte loads, 1 KB of a cell's channels a wave) or one.
// Four read less often but run as fewer, larger workgroups.  Both were timed on
// 73,000 images of 20^3 to 128^3 cells and 4 to 64 channels, all directions and
// fields, with inputs in and out of the cache (times of four over one, cached /
// not); what separates them:
//  - whether four fill the chip as well as one does (`fits`; three quarters of
//    that where velocity makes each lookup's work shared and inputs stay
//    cached): with a source function, or velocity and up to 100 MB, 0.85 / 0.73
//    where they fit and 1.00 / 0.91, slower in half of them, where not; beyond
//    100 MB without a source function 1.03 / 0.93;
//  - velocity and absorption without a source function, where one a lane spills:
//    0.79 / 0.69 unless the chip is less than 0.65 full;
//  - neither velocity nor source function: 0.88 / 0.78 across x and nearly full,
//    1.02 / 0.84 along x, slower in half of them; a source function along x
//    without velocity: slower in a third;
//  - few channels, since neighbouring cells share lines that the stream does not
//    keep (200^3 x 4 toward +x 43 us with one, 167 with four): below 24 along x,
//    12 across;
//  - whole pieces of 64 bytes (32, 48, 64 channels) and a full chip: 0.82 / 0.73
//    in any case but a source function along x (64^3 x 32 15.5 us, 10.8).
// Over the images that take four it is 0.85 / 0.74; one would be more than 3%
// faster in 4% of them, 8% in 1%.  128^3 x 64 with velocity, source and
// absorption toward -z: 247 us with one, 205 with four.
static ImgPlan image_plan(const ImageParams &Q, int64_t round_single, int64_t round_quad) {
    const int nl = Q.n[Q.d];
    const bool along = Q.d == 0, vel = Q.vel_axis != nullptr, src = Q.srcf != nullptr;
    const ImgPlan single = image_plan(Q.npix, Q.nch, nl, 1);
    if (Q.nch < (along ? 24 : 12)) return single;
    const ImgPlan quad = image_plan(Q.npix, Q.nch, nl, 4);
    if (quad.groups * quad.nseg < kImgQuadWaves) return single;
    const double fill = image_fill(image_blocks(quad), round_quad);
    const double mb = 4e-6 * (src ? 2.0 : 1.0) * (double)Q.npix * nl * Q.nch;
    const bool fits = fill >= (vel && mb <= 60.0 ? 0.75 : 0.97) * image_fill(image_blocks(single), round_single);
    const bool pieces = Q.nch % 16 == 0 && Q.nch >= 32 && Q.nch <= 64 && fill >= 0.9 &&
                        (Q.nch < 64 || vel || src || image_blocks(quad) <= round_quad);
    const bool take = src ? (along ? vel && fits : fits || pieces)
                          : (vel && Q.kabs && fill >= 0.65) || pieces ||
                                (fits && mb <= 100.0 && (vel || (!along && fill >= 0.85)));
    return take ? quad : single;
}

template <bool kVel, bool kAbs, bool kSrc>
static hipError_t launch_image_t(const ImageParams &Q, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    auto quad = image_quad_kernel<kVel, kAbs>;
    auto single = image_kernel<kVel, kAbs>;
    if constexpr (kSrc) {
        quad = image_quad_src_kernel<kVel, kAbs>;
        single = image_src_kernel<kVel, kAbs>;
    }
    static std::atomic<int> resident[2] = {{0}, {0}};  // workgroups a compute unit holds: one, four channels a lane
    int per_cu[2];
    for (int k = 0; k < 2; ++k)
        if ((per_cu[k] = resident[k].load()) == 0) {
            hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu[k], k ? quad : single, 64 * kImgWaves, 0);
            if (e != hipSuccess) return e;
            resident[k].store(per_cu[k] = std::max(per_cu[k], 1));
        }
    const ImgPlan p = image_plan(Q, (int64_t)Q.cus * per_cu[0], (int64_t)Q.cus * per_cu[1]);
    const int nl = Q.n[Q.d], seglen = (nl + p.nseg - 1) / p.nseg;
    const dim3 grid((unsigned)image_blocks(p)), block(64 * kImgWaves);
    hipExtLaunchKernelGGL(p.v == 4 ? quad : single, grid, block, 0, s, start, stop, 0, Q, p.nseg, seglen);
    return hipGetLastError();
}

hipError_t launch_image_timed(const ImageParams &Q, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    const int64_t n = Q.npix * (int64_t)Q.nch;
    if (n <= 0) {  // nothing to launch: an empty interval
        if (start) { hipError_t e = hipEventRecord(start, s); if (e != hipSuccess) return e; }
        if (stop) { hipError_t e = hipEventRecord(stop, s); if (e != hipSuccess) return e; }
        return hipSuccess;
    }
    const int key = (Q.vel_axis ? 4 : 0) | (Q.kabs ? 2 : 0) | (Q.srcf ? 1 : 0);
    switch (key) {
        case 0: return launch_image_t<false, false, false>(Q, s, start, stop);
        case 1: return launch_image_t<false, false, true>(Q, s, start, stop);
        case 2: return launch_image_t<false, true, false>(Q, s, start, stop);
        case 3: return launch_image_t<false, true, true>(Q, s, start, stop);
        case 4: return launch_image_t<true, false, false>(Q, s, start, stop);
        case 5: return launch_image_t<true, false, true>(Q, s, start, stop);
        case 6: return launch_image_t<true, true, false>(Q, s, start, stop);
        default: return launch_image_t<true, true, true>(Q, s, start, stop);
    }
}

hipError_t launch_image(const ImageParams &Q, hipStream_t s) { return launch_image_timed(Q, s, nullptr, nullptr); }

}  // namespace krt
