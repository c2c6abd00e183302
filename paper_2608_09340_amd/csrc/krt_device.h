// krt_device.h -- device helpers shared by the transport and escape kernels:
// Philox4x32-10, the uniform map, hardware transcendental wrappers, the tally
// bin rule and the LDS table lookups (Voigt profile, atom-velocity sampler).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "krt_internal.h"
#include "krt_kernels.h"

namespace krt {

// ------------------------------------------------------------------ Philox ---
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): ten rounds of two 32x32
// multiplies with key schedule increments (W0, W1) between rounds.
__device__ __forceinline__ uint4 philox(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
        uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
        uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
        uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
    }
    return c;
}

// The two blocks of one event, philox((ev, id, 0)) and philox((ev, id, 1)).
// Their first three rounds share most of their products: those of the packet's
// id alone are kept per packet, those of the event alone are made once, so the
// pair takes 34 wide multiplies instead of 40, and one three-way xor per output
// word instead of two.
struct PhiloxPacket {
    uint32_t bk, hk, la;
};
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ PhiloxPacket philox_packet(uint32_t plo, uint32_t phi, uint32_t k0, uint32_t k1) {
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * phi;
    const uint64_t q = (uint64_t)0xD2511F53u * ((uint32_t)(p1 >> 32) ^ plo ^ k0);
    PhiloxPacket p;
    p.bk = (uint32_t)p1 ^ (k0 + 0x9E3779B9u);
    p.hk = (uint32_t)(q >> 32) ^ (k1 + 0xBB67AE85u);
    p.la = (uint32_t)q;
    return p;
}
__device__ __forceinline__ void philox_pair(const PhiloxPacket &pk, uint32_t ev, uint32_t k0, uint32_t k1, uint4 &A,
                                            uint4 &B) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * ev;              // round 1
    const uint32_t z = (uint32_t)(p0 >> 32) ^ k1;
    const uint64_t pa = (uint64_t)0xCD9E8D57u * z, pb = (uint64_t)0xCD9E8D57u * (z ^ 1u);  // round 2
    const uint64_t q = (uint64_t)0xCD9E8D57u * (pk.hk ^ (uint32_t)p0);                     // round 3
    const uint64_t ra = (uint64_t)0xD2511F53u * ((uint32_t)(pa >> 32) ^ pk.bk);
    const uint64_t rb = (uint64_t)0xD2511F53u * ((uint32_t)(pb >> 32) ^ pk.bk);
    k0 += 2u * 0x9E3779B9u;
    k1 += 2u * 0xBB67AE85u;
    A = make_uint4(xor3((uint32_t)(q >> 32), (uint32_t)pa, k0), (uint32_t)q, xor3((uint32_t)(ra >> 32), pk.la, k1),
                   (uint32_t)ra);
    B = make_uint4(xor3((uint32_t)(q >> 32), (uint32_t)pb, k0), (uint32_t)q, xor3((uint32_t)(rb >> 32), pk.la, k1),
                   (uint32_t)rb);
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const uint64_t a0 = (uint64_t)0xD2511F53u * A.x, a1 = (uint64_t)0xCD9E8D57u * A.z;
        const uint64_t b0 = (uint64_t)0xD2511F53u * B.x, b1 = (uint64_t)0xCD9E8D57u * B.z;
        A = make_uint4(xor3((uint32_t)(a1 >> 32), A.y, k0), (uint32_t)a1, xor3((uint32_t)(a0 >> 32), A.w, k1),
                       (uint32_t)a0);
        B = make_uint4(xor3((uint32_t)(b1 >> 32), B.y, k0), (uint32_t)b1, xor3((uint32_t)(b0 >> 32), B.w, k1),
                       (uint32_t)b0);
    }
}

// uniform on (0,1): the odd multiple (w >> 9) 2^-23 + 2^-24, exact in binary32;
// the 23 bits go into the mantissa of a number in [1, 2), and the difference is
// exact
__device__ __forceinline__ float u01(uint32_t w) {
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w, 9)) - (1.0f - 0x1p-24f);
}

// ------------------------------------------------------------- fast math ---
constexpr float kPiF = 3.14159265358979f;
constexpr uint32_t kMaxCrossings = 1u << 30;  // per packet: a packet that never interacts is retired as stuck
constexpr float kInvSqrtPiF = 0.564189583547756f;
constexpr float kInvSqrt2F = 0.707106781186547524f;
constexpr float kLn2F = 0.693147180559945f;
__device__ __forceinline__ float f_log(float x) { return __builtin_amdgcn_logf(x) * kLn2F; }
__device__ __forceinline__ float f_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896f); }
__device__ __forceinline__ float f_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float f_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float f_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
// sin / cos of 2 pi r (the hardware takes revolutions)
__device__ __forceinline__ float sin_rev(float r) { return __builtin_amdgcn_sinf(r); }
__device__ __forceinline__ float cos_rev(float r) { return __builtin_amdgcn_cosf(r); }

// a or b, both evaluated: where lanes differ a branch costs more than either
template <class V>
__device__ __forceinline__ V sel(bool c, V a, V b) {
    return __builtin_unpredictable(c) ? a : b;
}

// ------------------------------------------------------------------- bins ---
// Index rule shared by every tally: edges[k] (k = 0..nb) are the binary32 values
// of lo + (hi - lo) * k / nb computed in FP64 on the host; the bin is 1 + the
// largest k with edges[k] <= x, 0 below edges[0], nb + 1 at or above edges[nb],
// -1 for NaN.  The first guess from (x - lo) / width is corrected against the
// edges themselves, so the result is exact whatever the rounding of the guess.
__device__ __forceinline__ int bin_index(float x, const float *edges, int nb, float inv_w) {
    if (!(x == x)) return -1;
    const float e0 = edges[0];
    if (x < e0) return 0;
    if (x >= edges[nb]) return nb + 1;
    int k = (int)((x - e0) * inv_w);
    k = max(0, min(nb - 1, k));
    while (k > 0 && edges[k] > x) --k;
    while (k < nb - 1 && edges[k + 1] <= x) ++k;
    return k + 1;
}

// The channel k (0 <= k < nb) that bin_index puts x in is floor(x / width - lo /
// width) unless x is within rounding of an edge.  Returns that guess and sets
// `sure` if its fraction is nearer to one half than `safe`, one half less the
// bound on the rounding in widths; else the edges decide (bin_index, less one).
// off: -lo / width.
__device__ __forceinline__ int channel_guess(float x, float inv_w, float off, float safe, bool &sure) {
    const float t = fmaf(x, inv_w, off);
    const float fl = floorf(t);
    sure = fabsf((t - fl) - 0.5f) < safe;
    return (int)fl;
}

// ----------------------------------------------------------- LDS lookups ---
// The entry of |x| in the Voigt table: its core and wing pieces share one address
// and one read.  (int) of a float that may be NaN is 0 here, and none of the
// indices below can be negative, so only the upper ends are clamped.
struct VoigtEntry {
    float4 c;
    float f, w;   // position in the interval, 8 / |x|
    int row;      // of 4 floats: core 0 .. 511, wing 512 .. 639
};
__device__ __forceinline__ VoigtEntry voigt_entry(const float *T, float xa) {
#pragma clang fp contract(off)
    static_assert(kOffVoigtCore == 0 && kOffVoigtWing == 4 * kVoigtCoreN, "the wing follows the core");
    const bool core = xa < 8.0f;
    VoigtEntry e;
    e.w = 8.0f * f_rcp(xa);
    const float t = sel(core, xa * 64.0f, e.w * (float)kVoigtWingN);
    const int i = min((int)t, sel(core, kVoigtCoreN - 1, kVoigtWingN - 1));
    e.row = i + sel(core, 0, kVoigtCoreN);
    e.f = t - (float)i;
    e.c = *reinterpret_cast<const float4 *>(T + 4 * e.row);
    return e;
}
__device__ __forceinline__ float voigt_value(const VoigtEntry &e, float xa) {
#pragma clang fp contract(off)
    const float G = fmaf(e.f, fmaf(e.f, fmaf(e.f, e.c.w, e.c.z), e.c.y), e.c.x);
    return sel(xa < 8.0f, G, G * e.w * e.w * (1.0f / 64.0f));
}
// H(a, |x|)
__device__ __forceinline__ float voigt_lds(const float *T, float xa) { return voigt_value(voigt_entry(T, xa), xa); }

// Analytic approximation of H(a, u) that blends the Doppler core exp(-u^2) and
// the damping wing a / (sqrt(pi) (u^2 + a^2)) with the switch
// w = (1 + tanh(2|u| - 2 u0)) / 2 centred at the crossing point u0 of the two
// asymptotes (Sec. 2.2.1, the third profile mode).  Accurate in the core and
// the wing, rough between them: offered to show why the opacity profile must
// be the one the redistribution sampler assumes, not for production runs.
__device__ __forceinline__ float voigt_analytic(float a, float u0, float ua) {
    const float core = f_exp(-ua * ua);
    const float wing = a * kInvSqrtPiF * f_rcp(fmaf(ua, ua, a * a));
    const float w = 0.5f * (1.0f + tanhf(2.0f * (ua - u0)));
    return fmaf(w, wing - core, core);
}

// Atom parallel velocity for gas-frame frequency x (Sec. 2.1.1): piece by r1
// against the cumulative piece probabilities, quantile by r2, bilinear in
// (row of |x|, quantile node).
// The piece probabilities (cumulative, first three) depend on |x| alone and can
// be read ahead of the draw.
struct UparMass {
    float4 m0, m1;
    float fm;
};
// Its grid is the Voigt core's, so the Voigt entry gives row and position
// (beyond |x| = 8 what is read is not used).
__device__ __forceinline__ UparMass upar_mass(const float *T, const VoigtEntry &e) {
    static_assert(kMassN == kVoigtCoreN && kOffMass + 4 * (kVoigtCoreN + kVoigtWingN) + 4 <= kTabFloats,
                  "one grid, and the wing's rows stay inside the table block");
    UparMass q;
    q.fm = e.f;
    q.m0 = *reinterpret_cast<const float4 *>(T + kOffMass + 4 * e.row);
    q.m1 = *reinterpret_cast<const float4 *>(T + kOffMass + 4 * e.row + 4);
    return q;
}
// the wing pieces' quantile coordinate: nodes at q = 4 xi^3 (xi < 1/2),
// 1 - 4 (1 - xi)^3 (xi >= 1/2)
__device__ __forceinline__ float wing_level(float r2) {
#pragma clang fp contract(off)
    const bool lo = r2 < 0.5f;
    const float cb = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(0.25f * sel(lo, r2, 1.0f - r2)) * (1.0f / 3.0f));
    return sel(lo, cb, 1.0f - cb);
}
// xw: wing_level(r2)
__device__ __forceinline__ float upar_from(const float *T, const UparMass &q, float x, float a, float thd, float r1,
                                           float r2, float xw) {
#pragma clang fp contract(off)
    const float xa = fabsf(x);
    const bool lin = xa < 8.0f;
    const float c1 = fmaf(q.fm, q.m1.x - q.m0.x, q.m0.x);
    const float c2 = fmaf(q.fm, q.m1.y - q.m0.y, q.m0.y);
    const float c3 = fmaf(q.fm, q.m1.z - q.m0.z, q.m0.z);
    // the first that holds names the piece; beyond the table every draw is the bump's
    const bool spike = lin & (r1 < c1), l1 = lin & (r1 < c2), l2 = !lin | (r1 < c3);
    const float p = sel(lin, xa * 6.0f, fminf(fmaf(f_log(xa * 0.125f), kRowInvLog, 48.0f), 63.0f));
    const int j = min((int)p, kRows - 2);
    const float fr = p - (float)j;
    const int off = sel(spike, kOffSpike, sel(l1, kOffL1, sel(l2, kOffL2, kOffRight)));
    const float xi = sel(spike, r2, xw);
    int nq = sel(spike, kQS, kQL1);  // kQL1 == kQL2 == kQR
    asm("" : "+v"(nq));              // one multiply-add below, not the shifts of a known power of two
    const float nq1 = sel(spike, (float)(kQS - 1), (float)(kQL1 - 1));
    const int k = min((int)(xi * nq1), nq - 2);
    const float fq = fmaf(xi, nq1, -(float)k);
    const float *r0 = T + ((int)__umul24((unsigned)j, (unsigned)nq) + off + k);
    const float *rn = r0 + nq;
    const float v0 = fmaf(fq, r0[1] - r0[0], r0[0]);
    const float v1 = fmaf(fq, rn[1] - rn[0], rn[0]);
    const float v = fmaf(fr, v1 - v0, v0);
    // spike: u = x + a tan(theta); wings: x -+ DELTA e^v; bump: v itself
    const float th = v * thd * (1.0f / (2.0f * kPiF));
    const float us = fmaf(a * sin_rev(th), f_rcp(cos_rev(th)), xa);
    const float s = (float)kDelta * f_exp(v);
    const float uw = xa + sel(l1, -s, s);
    const float u = sel(spike, us, sel(l2 & !l1, v, uw));
    // p(u | -x) = p(-u | x): u takes the sign of x.  A zero is +0 here: the
    // sources give no -0, and a difference or sum of a walk makes none.
    return __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(u), __float_as_uint(x), 0x80000000u, 0x78));
}

__device__ __forceinline__ float upar_lds(const float *T, float x, float a, float thd, float r1, float r2) {
    return upar_from(T, upar_mass(T, voigt_entry(T, fabsf(x))), x, a, thd, r1, r2, wing_level(r2));
}

// Dipole phase (3/8)(1 + g^2): g = 2 sinh(asinh(4u - 2)/3).
__device__ __forceinline__ float dipole_g(float u) {
    float q = 4.0f * u - 2.0f;
    float aq = fabsf(q);
    float t = f_log(aq + f_sqrt(fmaf(aq, aq, 1.0f))) * (1.0f / 3.0f);
    float e = f_exp(t);
    float g = e - f_rcp(e);
    return copysignf(g, q);
}

// ------------------------------------------------------------- scattering ---
// Draws of a scattering: the sampler's uniforms r1, r2 with the latter's
// wing_level, the two u_perp components (Box-Muller, N(0, 1/2) each), the cosine
// g of the scattering angle (isotropic or dipole) with sqrt(1 - g^2), cos, sin
// of the azimuth psi, and the u_perp component along the outgoing direction's
// transverse part.
struct SDraws {
    float r1, r2, xw, up1, up2, g, sg, cp, sp, kick;
};

__device__ __forceinline__ void scatter_draws(uint32_t w1, uint32_t w2, uint4 B, bool dipole, SDraws &d) {
#pragma clang fp contract(off)
    d.r1 = u01(w1);
    d.r2 = u01(w2);
    d.xw = wing_level(d.r2);
    const float rr = f_sqrt(-f_log(u01(B.x)));
    const float th = u01(B.y);
    d.up1 = rr * cos_rev(th);
    d.up2 = rr * sin_rev(th);
    d.g = dipole ? dipole_g(u01(B.z)) : fmaf(2.0f, u01(B.z), -1.0f);
    d.sg = f_sqrt(fmaxf(0.0f, fmaf(-d.g, d.g, 1.0f)));
    const float psi = u01(B.w);
    d.cp = cos_rev(psi);
    d.sp = sin_rev(psi);
    d.kick = fmaf(d.up1, d.cp, d.up2 * d.sp);
}

// ax bx + ay by + az bz in the one order every variant uses
__device__ __forceinline__ float dot3(float ax, float bx, float ay, float by, float az, float bz) {
    return fmaf(az, bz, fmaf(ax, bx, ay * by));
}

// Orthonormal basis (e1, e2) about n (Duff et al. 2017)
struct Basis {
    float e1x, e1y, e1z, e2x, e2y, e2z;
};
__device__ __forceinline__ Basis scatter_basis(float nx, float ny, float nz) {
#pragma clang fp contract(off)
    const float sgn = copysignf(1.0f, nz);
    const float A = -f_rcp(sgn + nz);
    Basis e;
    e.e2x = nx * ny * A;
    e.e2y = fmaf(ny * ny, A, sgn);
    e.e2z = -ny;
    e.e1x = fmaf(A, nx * (nx * sgn), 1.0f);
    e.e1y = sgn * e.e2x;
    e.e1z = -sgn * nx;
    return e;
}
// the outgoing direction
__device__ __forceinline__ void scatter_turn(float nx, float ny, float nz, const Basis &e, const SDraws &b, float &ox,
                                             float &oy, float &oz) {
#pragma clang fp contract(off)
    ox = fmaf(b.g, nx, b.sg * fmaf(b.cp, e.e1x, b.sp * e.e2x));
    oy = fmaf(b.g, ny, b.sg * fmaf(b.cp, e.e1y, b.sp * e.e2y));
    oz = fmaf(b.g, nz, b.sg * fmaf(b.cp, e.e1z, b.sp * e.e2z));
    const float rn = f_rsq(fmaf(oz, oz, fmaf(ox, ox, oy * oy)));
    ox *= rn; oy *= rn; oz *= rn;
}
// the outgoing gas-frame frequency (eq. riia-scatter)
__device__ __forceinline__ float scatter_shift(float x, float upar, const SDraws &b) {
#pragma clang fp contract(off)
    return fmaf(b.sg, b.kick, fmaf(upar, b.g - 1.0f, x));
}

// ----------------------------------------------------------------- waves ---
// Lane index of the k-th set bit (k counted from 0) of m; k < popcount(m).
__device__ __forceinline__ int nth_set_lane(uint64_t m, int k) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const uint64_t low = (w == 64) ? m : (m & ((1ull << w) - 1ull));
        const int c = __popcll(low);
        if (k >= c) { k -= c; m >>= w; pos += w; }
        else m = low;
    }
    return pos;
}

// x, y or z of the axis a crossing goes along; by value, since a conditional
// between captured variables would select between their addresses and hold the
// lane's state in memory
template <class V>
__device__ __forceinline__ V by_axis(bool ax0, bool ax1, V x, V y, V z) {
    return sel(ax0, x, sel(ax1, y, z));
}

// Packets a wave starts with, so that few packets use many SIMDs: up to two
// waves per SIMD (eight of a workgroup's) share them evenly, more packets fill
// those waves' lanes first and then further waves.  A lone wave leaves issue
// slots idle that a second one takes, a third and fourth only slow the first
// two (10,000 packets on a tau0 = 300 slab: 15.1 ms with one wave per SIMD,
// 14.9 with two, 15.0 with three, 15.5 with four; 130,000 on a 32^3 dipole
// sphere of tau0 = 1e3: 30.9, 30.2, 32.6, 33.5).
inline int first_lanes(uint64_t n, uint64_t waves, uint64_t grid) {
    const uint64_t w = std::min(waves, 8 * grid);
    return (int)std::min<uint64_t>(64, (n + w - 1) / w);
}

// A wave's share of a launch's work items [0, n): the first `lanes` of them
// fixed by its place, the rest from the launch's counter (zeroed by the caller).
// The counter is one address for the whole chip and serves about one request in
// 4.6 ns, so short items taken one refill at a time wait for it: in a Lambda
// cycle's transport 4096 waves asked once per iteration, 19 us apart.  A wave
// that comes back within kPoolSoon iterations therefore takes twice as many as
// the last time (at most kPoolChunk, and no more than its even share of what is
// left: the cap is between half of it and the whole), and one that comes back
// later takes what it needs: long items are never held in stock while another
// wave is idle.
constexpr uint32_t kPoolChunk = 256;
constexpr int kPoolSoon = 32;
// Idle lanes are refilled together: at kRefillLanes of them, or kRefillWait
// iterations after the first, or when no lane is live.  Starting a packet costs
// the wave more than an iteration, however many lanes start.
constexpr int kRefillLanes = 16, kRefillWait = 8;
struct WorkPool {
    uint64_t next;            // the stock's first item
    uint32_t left, chunk;     // items in stock; taken the last time
    bool dry;                 // the counter has passed n
    int waited, since;        // iterations since the first idle lane, since the last request

    __device__ __forceinline__ void init(int lanes) {
        // waves counted across the workgroups first, so that consecutive ones sit on different CUs
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)) * gridDim.x + blockIdx.x;
        next = (uint64_t)wave * (uint64_t)lanes;
        left = (uint32_t)lanes;
        chunk = 0;
        dry = lanes < 64;
        waited = 0;
        since = 0;
    }
    // whether the idle lanes (a wave-uniform mask) are refilled in this iteration
    __device__ __forceinline__ bool due(uint64_t idle, bool any_live) {
        ++since;
        if (idle == 0ull) return false;
        if (__popcll(idle) >= kRefillLanes || ++waited >= kRefillWait || !any_live || dry) {
            waited = 0;
            return true;
        }
        return false;
    }
    // the work item of this lane (n or more: none), for the lanes of `idle`
    __device__ __forceinline__ uint64_t take(uint64_t idle, int lane, uint64_t lanemask_lt, unsigned long long *counter,
                                             uint64_t n, int lanes) {
        const uint32_t cnt = (uint32_t)__popcll(idle), rank = (uint32_t)__popcll(idle & lanemask_lt);
        uint64_t mine = rank < left ? next + rank : ~0ull;
        if (cnt <= left) {
            next += cnt;
            left -= cnt;
        } else if (dry) {
            left = 0;
        } else {
            const uint32_t more = cnt - left, waves = (blockDim.x / 64) * gridDim.x;
            const uint64_t first = (uint64_t)waves * (uint64_t)lanes;  // those given out by place
            const uint64_t seen = max(next + left, first), rest = n > seen ? n - seen : 0;
            // rest >> share is between half and the whole of the even share
            const int share = 32 - __clz((int)waves);
            chunk = since < kPoolSoon ? min(2 * max(chunk, more), kPoolChunk) : 0u;
            chunk = max(more, (uint32_t)min(rest >> share, (uint64_t)chunk));
            since = 0;
            const int leader = __ffsll((long long)idle) - 1;
            uint64_t nb = 0;
            if (lane == leader) nb = first + atomicAdd(counter, (unsigned long long)chunk);
            nb = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(nb >> 32), leader) << 32) |
                 (uint32_t)__builtin_amdgcn_readlane((int)nb, leader);
            if (rank >= left) mine = nb + (rank - left);
            next = nb + more;
            left = chunk - more;
            dry = nb >= n;
        }
        return mine;
    }
};

}  // namespace krt
