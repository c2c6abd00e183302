// krt_transport.hip -- gfx950 kernels of the Monte Carlo line-transfer pass.
//
// One photon packet per lane in a persistent wavefront pool (Sec. 2.3.2 runs
// packets from a global work queue; here each wave refills its retired lanes
// from one wave-aggregated atomic, so lanes stay busy while packets of very
// different lengths finish).  Per loop iteration a lane does one flight
// segment (to its next interaction or to the next cell face) and, on an
// interaction, one resonant scattering.  Fields are SoA binary32 read once per
// cell entry; the per-line Voigt and atom-velocity tables live in LDS.
// Tallies are int64 fixed point: a window of channels per lane for the current
// cell, written back with one atomic per (cell, channel) met when the packet
// leaves.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "krt_internal.h"
#include "krt_kernels.h"
#include "krt_device.h"
#include "krt_mlp.h"

namespace krt {

// --------------------------------------------------------- tally helpers ---
// Integer tally atomics return nothing, so a wave never waits on them; sums
// past 2^62 are detected after the launch (finish_kernel).
__device__ __forceinline__ void tally_add_i64(int64_t *p, int64_t v) {
    atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}

// Emissivity tally of a packet's visit to one cell: a window of eight
// consecutive channels accumulates the scatterings; a channel outside it
// writes the window back (one atomic per channel met) and moves it.  Consecutive
// scatterings see camera frequencies within a few Doppler widths of the cell's,
// so the window rarely moves.
//
// Isotropic phase: every scattering adds the same 2^F, so the window counts
// scatterings, eight 8-bit counts in one register pair.  The wave writes all
// its windows back every kEmisTicks iterations, before a count can pass 255.
// Dipole phase: the contributions differ, so the window holds int64 sums, in
// LDS ([slot][thread], each thread its own), which stay until the packet leaves
// the window or the cell.
// Against four direct-mapped (channel, int64 sum) register slots with a
// four-way branch per scattering this takes 3 VGPRs instead of 12.
constexpr int kEmisSlots = 8;
constexpr int kEmisTicks = 255;

template <bool kSum>
struct EmisWindow {
    int w = 0;            // first channel of the window
    uint64_t cnt = 0;     // 8-bit counts of channels w .. w + 7 (kSum: bit s = slot s in use)
    int size;             // channels it spans: kEmisSlots, or all where there are fewer
    int64_t *acc;         // kSum: this thread's LDS sums
    int stride;           // ... and the distance between its slots

    // writes the window back to the tallies `cell` (of the window's cell)
    __device__ __forceinline__ void flush(int64_t *cell, int frac_bits) {
        while (cnt != 0) {
            if constexpr (kSum) {
                const int s = __ffs((unsigned)cnt) - 1;
                tally_add_i64(cell + (w + s), acc[s * stride]);
                acc[s * stride] = 0;
                cnt &= cnt - 1;
            } else {
                const int s = (__ffsll((long long)cnt) - 1) & ~7;
                const uint64_t n = (cnt >> s) & 255u;
                tally_add_i64(cell + (w + (s >> 3)), (int64_t)(n << frac_bits));
                cnt &= ~(255ull << s);
            }
        }
    }
    // One scattering of weight v (kSum; 2^frac_bits otherwise) into channel ch,
    // `unit` = 1, or nothing, `unit` = 0 (a lane without a packet; v is 0 too).
    // The caller has seen that the window holds the channel (or the lane adds
    // nothing).
    __device__ __forceinline__ void add(int ch, uint32_t unit, int64_t v) {
        const uint32_t d = (uint32_t)(ch - w);
        if constexpr (kSum) {
            const uint32_t s = min(d, (uint32_t)(kEmisSlots - 1));
            __hip_atomic_fetch_add(acc + s * stride, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            cnt |= (uint64_t)(unit << s);
        } else {
            cnt += (uint64_t)unit << ((8 * d) & 63);
        }
    }
    // moves the (written back) window to hold channel ch of nch
    __device__ __forceinline__ void move(int ch, int nch) { w = max(0, min(ch - (size / 2 - 1), nch - size)); }
};

// Counters a workgroup keeps in LDS until it ends: the outcomes 1..3 of retired
// packets first, then emissions and the retired packets' sums.
enum { kLcEscaped = 0, kLcDestroyed, kLcStuck, kLcEmit, kLcScat, kLcCross, kLcDrop, kNLdsCounters };

// wave-wide sum of a 64-bit value, then one atomic from the first active lane
__device__ __forceinline__ void wave_add_counter(int64_t *dst, int64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if (__lane_id() == 0 && v != 0) atomicAdd(reinterpret_cast<unsigned long long *>(dst), (unsigned long long)v);
}

// ------------------------------------------------------ learned escape ---
// Batched evaluation of the escape network for the lanes of the wave set in
// `ask` (wave-uniform control flow: every lane executes the MFMA).  The asking
// lanes are packed in rank order into blocks of 16 samples, so a call costs
// ceil(popcount(ask) / 16) block evaluations.  pk[] holds this lane's inputs
// as bf16 pairs; an asking lane receives the normalised outputs k set in the
// wave-uniform `want` (a subset of kMlpFetch) in out[k] (the others keep their
// values).
constexpr uint32_t kMlpFetch = 0x003F1FFFu;  // outputs 0-12 and 16-21: all the transport reads
__device__ __forceinline__ void mlp_eval_wave(const unsigned char *img, const float *bias, const uint32_t pk[kMlpPackDw],
                                              int lane, uint64_t ask, uint32_t want, float out[kMlpOut]) {
    const int nask = __popcll(ask);
    const int nblk = (nask + 15) >> 4;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int rank = __popcll(ask & lt);
    const bool mine = (ask >> lane) & 1ull;
    const int g = lane >> 4;
#pragma unroll 1
    for (int b = 0; b < nblk; ++b) {
        // block position p = lane & 15 holds the asker of rank 16 b + p (if any);
        // lane group g takes that asker's input dwords 4g .. 4g + 3
        const int r = 16 * b + (lane & 15);
        const int src = (r < nask) ? nth_set_lane(ask, r) : lane;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int d = 0; d < kMlpPackDw; ++d) {
            const uint32_t v = (uint32_t)__shfl((int)pk[d], src, 64);
            if ((d >> 2) == g) w[d & 3] = v;
        }
        const bool use = r < nask;
        const v4i16 lo = {(short)(use ? w[0] & 0xFFFFu : 0u), (short)(use ? w[0] >> 16 : 0u),
                          (short)(use ? w[1] & 0xFFFFu : 0u), (short)(use ? w[1] >> 16 : 0u)};
        const v4i16 hi = {(short)(use ? w[2] & 0xFFFFu : 0u), (short)(use ? w[2] >> 16 : 0u),
                          (short)(use ? w[3] & 0xFFFFu : 0u), (short)(use ? w[3] >> 16 : 0u)};
        v4f32 oa, ob;
        mlp_forward_block(img, bias, cat8(lo, hi), lane, oa, ob);
        // output k of block position p sits in lane 16 ((k % 16) / 4) + p,
        // component k % 4, of tile k / 16
        const bool take = mine && (rank >> 4) == b;
#pragma unroll
        for (int k = 0; k < kMlpOut; ++k) {
            if (!((kMlpFetch >> k) & 1u) || !((want >> k) & 1u)) continue;  // wave-uniform
            const v4f32 o = (k < 16) ? oa : ob;
            const float comp = (k % 4 == 0) ? o.x : (k % 4 == 1) ? o.y : (k % 4 == 2) ? o.z : o.w;
            const float v = __shfl(comp, 16 * ((k % 16) / 4) + (rank & 15), 64);
            if (take) out[k] = v;
        }
    }
}

// ------------------------------------------------------ network call ---
// The pieces of one learned whole-cell escape, shared by the transport kernel
// (calls batched inside it) and escape_call_kernel (parked calls), so both
// apply a call with the same arithmetic.

// Whether a scattering at the cell-frame position (fx, fy, fz) in [0, 1]^3 of a
// cell of line-centre opacity k0c, at gas-frame frequency xc, qualifies for a
// call: a cubic cell with tau_c = k0c half_dx in range, the point at least
// esc_depth_min below its nearest face, |xc| <= esc_x_max.  Returns the reduced
// frame and log10 tau_c, log10 depth.
__device__ __forceinline__ void call_frame(const RunParams &P, float k0c, float fx, float fy, float fz,
                                           CellFrame &CF, float &tc, float &dep) {
    tc = k0c * P.esc_half_dx;  // line-centre depth, centre to face
    cell_reduce(2.0f * fx - 1.0f, 2.0f * fy - 1.0f, 2.0f * fz - 1.0f, CF);
    dep = tc * (1.0f - CF.q[2]);
}
__device__ __forceinline__ bool call_eligible(const RunParams &P, float k0c, float fx, float fy, float fz, float xc,
                                              CellFrame &CF, float &ltc, float &ldep) {
    if (!P.esc_cubic) return false;
    float tc, dep;
    call_frame(P, k0c, fx, fy, fz, CF, tc, dep);
    if (tc >= P.esc_tc_min && tc <= P.esc_tc_max && dep >= P.esc_depth_min && fabsf(xc) <= P.esc_x_max) {
        ltc = __log10f(tc);
        ldep = __log10f(dep);
        return true;
    }
    return false;
}

// call_eligible's test without the frame: the transport kernel tests every
// scattering and reduces the frame only inside a call batch (same decisions:
// the largest |offset| is the last of the sorted three)
__device__ __forceinline__ bool call_ok(const RunParams &P, float k0c, float fx, float fy, float fz, float xc) {
    if (!P.esc_cubic) return false;
    const float tc = k0c * P.esc_half_dx;
    const float qm = fmaxf(fabsf(2.0f * fx - 1.0f), fmaxf(fabsf(2.0f * fy - 1.0f), fabsf(2.0f * fz - 1.0f)));
    const float dep = tc * (1.0f - qm);
    return tc >= P.esc_tc_min && tc <= P.esc_tc_max && dep >= P.esc_depth_min && fabsf(xc) <= P.esc_x_max;
}

// The two evaluations of a call for the lanes in `ask` (wave-uniform): the
// marginal one (exit face from the softmax at level u01(C.z), side of x_out
// from the learned P(x_out >= 0) at u01(C.w), |x_out| from the exit face's
// quantile at u_a = u01(C.x)), then the one conditional on the sampled face and
// x_out (offsets, cosine, alpha at the levels of D).  cnd: the raw condition
// (log10 tau_c, log10 a, |x_in|, q0, q1, q2, log10 depth, incoming direction in
// the reduced frame).  xo carries x_in's sign convention (reduced frame).
__device__ __forceinline__ void call_network(const unsigned char *mimg, const float *mbias, const float *mnorm,
                                             int lane, uint64_t ask, const float cnd[10], uint4 C, uint4 D,
                                             int &face, float &xo, float mo[kMlpOut]) {
    float in[kMlpIn];
    uint32_t pk[kMlpPackDw];
#pragma unroll
    for (int k = 0; k < kMlpOut; ++k) mo[k] = 0.0f;
    face = 5;
    xo = 0.0f;
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {
        if (e == 0) mlp_inputs(cnd, u01(C.x), u01(C.y), u01(D.z), u01(D.w), false, 0.0f, 0, in);
        else mlp_inputs(cnd, u01(D.x), u01(D.y), u01(D.z), u01(D.w), true, xo, face, in);
        pack_inputs(in, pk);
        mlp_eval_wave(mimg, mbias, pk, lane, ask, e == 0 ? 0x003F01FFu : 0x00001E00u, mo);
        if (e == 0) {
            float mx = mo[0];
#pragma unroll
            for (int f = 1; f < 6; ++f) mx = fmaxf(mx, mo[f]);
            float ef[6], se = 0.0f;
#pragma unroll
            for (int f = 0; f < 6; ++f) { ef[f] = __expf(mo[f] - mx); se += ef[f]; }
            const float uf = u01(C.z) * se;
            float c2 = 0.0f;
            bool found = false;
#pragma unroll
            for (int f = 0; f < 6; ++f) {
                c2 += ef[f];
                if (!found && uf < c2) { face = f; found = true; }
            }
            const bool pos = u01(C.w) < sigmoid_f(mo[kOutSide]);
            float ma = mo[kOutXAbs], mm = mnorm[kOutXAbs], ms = mnorm[kMlpOut + kOutXAbs];
#pragma unroll
            for (int f = 1; f < 6; ++f)
                if (face == f) {
                    ma = mo[kOutXAbs + f];
                    mm = mnorm[kOutXAbs + f];
                    ms = mnorm[kMlpOut + kOutXAbs + f];
                }
            const float mag = fmaxf(fmaf(ma, ms, mm), 0.0f);
            xo = pos ? mag : -mag;
        }
    }
}

// erf by the rational approximation of Abramowitz & Stegun (Handbook of
// Mathematical Functions, 7.1.26; absolute error at most 1.5e-7): one
// reciprocal and one exp instead of the library's longer evaluation.  It
// integrates the skipped scatterings' Gaussian over the channels, whose
// weights carry about 1e-7 of their own rounding.
__device__ __forceinline__ float erf_fast(float x) {
    const float ax = fabsf(x);
    const float t = f_rcp(fmaf(0.3275911f, ax, 1.0f));
    const float p = fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f),
                         0.254829592f);
    return copysignf(1.0f - t * p * f_exp(-ax * ax), x);
}

// The sampled exit applied to the packet: the exit point on the face (cell
// frame, fx, fy, fz in [0, 1]), the exit direction, the lab frequency
// x = sign(xc) xo + n.v, and the expected number of skipped scatterings
// E[N_s] (calibrated), whose emissivity -- thermalised core, camera frequency
// ~ N(n_cam.v, (<x^2> + 1)/3), integrated exactly over the whole channels that
// meet the central +-3 sd and renormalised to their share of it (the tails
// beyond hold 0.27%) -- goes to dep(channel, fixed-point weight); mass outside
// the channel grid is added to n_drop.  alpha takes its sign from the lowest
// bit of C.z.
template <class Dep>
__device__ __forceinline__ void call_apply(const RunParams &P, const float *mnorm, const float *cedges,
                                           const CellFrame &CF, const float mo[kMlpOut], int face, float xo,
                                           uint32_t cz, float ltc, float ldep, float xc, float vxc, float vyc,
                                           float vzc, float &fx, float &fy, float &fz, float &nx, float &ny,
                                           float &nz, float &x, int64_t &n_skip, int64_t &n_drop, Dep dep) {
    const float lns = mo[kOutLogN] * mnorm[kMlpOut + kOutLogN] + mnorm[kOutLogN] +
                      mnorm[kNormCal + cal_bin(ltc, ldep, fabsf(xc))];
    const float lx2 = mo[kOutLogX2] * mnorm[kMlpOut + kOutLogX2] + mnorm[kOutLogX2];
    // offsets learned as asinh, the cosine as mu^2
    auto sinh_f = [](float v) { const float ev = f_exp(v); return 0.5f * (ev - f_rcp(ev)); };
    const float ys = sinh_f(mo[kOutYS] * mnorm[kMlpOut + kOutYS] + mnorm[kOutYS]);
    const float yt = sinh_f(mo[kOutYT] * mnorm[kMlpOut + kOutYT] + mnorm[kOutYT]);
    const float mu = f_sqrt(fminf(fmaxf(mo[kOutMu2] * mnorm[kMlpOut + kOutMu2] + mnorm[kOutMu2], 1e-6f), 1.0f));
    const float al = fminf(fmaxf(mo[kOutAlpha] * mnorm[kMlpOut + kOutAlpha] + mnorm[kOutAlpha], 0.0f), 3.14159265f);
    // exit point and direction in the reduced frame: face axis k, outward side
    const int k = face >> 1;
    const float side = (face & 1) ? 1.0f : -1.0f;
    const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
    const float qk = pick3(CF.q[0], CF.q[1], CF.q[2], k);
    const float qa = pick3(CF.q[0], CF.q[1], CF.q[2], k1);
    const float qb = pick3(CF.q[0], CF.q[1], CF.q[2], k2);
    const float dpl = 1.0f - side * qk;
    const float es = fminf(fmaxf(qa + dpl * ys, -1.0f), 1.0f);
    const float et = fminf(fmaxf(qb + dpl * yt, -1.0f), 1.0f);
    // tangential direction at angle +-alpha from the offset (es - qa, et - qb)
    const float ds = es - qa, dt = et - qb;
    const float rr = f_sqrt(ds * ds + dt * dt);
    const float ir = (rr > 0.0f) ? f_rcp(rr) : 0.0f;
    const float c0 = (rr > 0.0f) ? ds * ir : 1.0f, s0 = dt * ir;
    const float arev = al * 0.159154943f * ((cz & 1u) ? -1.0f : 1.0f);
    const float ca = cos_rev(arev), sa = sin_rev(arev);
    const float sm = f_sqrt(fmaxf(0.0f, 1.0f - mu * mu));
    const float d1 = sm * (c0 * ca - s0 * sa), d2 = sm * (s0 * ca + c0 * sa);
    // back to the cell frame: reduced axis r is cell axis perm[r] with sign sg
    float pc[3] = {0.0f, 0.0f, 0.0f}, nc[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const float R_ = (r == k) ? side : ((r == k1) ? es : et);
        const float V_ = (r == k) ? side * mu : ((r == k1) ? d1 : d2);
        const int axc = CF.perm[r];
        const float sgc = pick3(CF.sg[0], CF.sg[1], CF.sg[2], axc);
#pragma unroll
        for (int a3 = 0; a3 < 3; ++a3)
            if (a3 == axc) { pc[a3] = sgc * R_; nc[a3] = sgc * V_; }
    }
    fx = fminf(fmaxf(0.5f * (pc[0] + 1.0f), 0.0f), 1.0f);
    fy = fminf(fmaxf(0.5f * (pc[1] + 1.0f), 0.0f), 1.0f);
    fz = fminf(fmaxf(0.5f * (pc[2] + 1.0f), 0.0f), 1.0f);
    nx = nc[0]; ny = nc[1]; nz = nc[2];
    const float Ns = fmaxf(f_exp(lns), 1.0f);  // E[N_s | condition]
    if (P.emis_raw) {
        const float sd = f_sqrt((f_exp(lx2) + 1.0f) * (1.0f / 3.0f));
        const float vc = P.n_cam[0] * vxc + P.n_cam[1] * vyc + P.n_cam[2] * vzc;
        const float isd = kInvSqrt2F * f_rcp(sd);
        auto cdf = [&](float e) { return 0.5f * (1.0f + erf_fast((e - vc) * isd)); };
        const float wlo = vc - 3.0f * sd, whi = vc + 3.0f * sd;
        const int kb0u = bin_index(wlo, cedges, P.emis_nch, P.ch_inv_w);
        const int kb1u = bin_index(whi, cedges, P.emis_nch, P.ch_inv_w);
        const int kb0 = max(kb0u, 1), kb1 = min(kb1u, P.emis_nch);
        float cdf_lo = cdf(cedges[kb0 - 1]);
        // the Gaussian's mass over the channels met (the window's own ends where
        // it leaves the grid): the deposits are scaled by its inverse
        const float c_first = (kb0u >= 1) ? cdf_lo : cdf(wlo);
        const float c_last = cdf((kb1u >= 0 && kb1u <= P.emis_nch) ? cedges[kb1] : whi);
        const float inv_cov = f_rcp(fmaxf(c_last - c_first, 0.5f));
        const float W = Ns * P.frac_scale * inv_cov;
        float inside = 0.0f;
        for (int kb = kb0; kb <= kb1; ++kb) {
            const float cdf_hi = 0.5f * (1.0f + erf_fast((cedges[kb] - vc) * isd));
            const float fr = cdf_hi - cdf_lo;
            cdf_lo = cdf_hi;
            inside += fr;
            const int64_t wq = (int64_t)__float2ll_rn(W * fr);
            if (wq != 0) dep(kb - 1, wq);
        }
        n_drop += (int64_t)__float2ll_rn(Ns * fmaxf(0.0f, 1.0f - inside * inv_cov));
    }
    const float sx = (xc < 0.0f) ? -1.0f : 1.0f;
    x = sx * xo + nx * vxc + ny * vyc + nz * vzc;
    n_skip += (int64_t)__float2ll_rn(Ns);
}

// raw condition of a call: (log10 tau_c, log10 a, |x_in|, q0, q1, q2, log10
// depth, incoming direction in the reduced frame)
__device__ __forceinline__ void call_condition(const RunParams &P, const CellFrame &CF, float ltc, float ldep,
                                               float xc, float nx, float ny, float nz, float cnd[10]) {
    cnd[0] = ltc;
    cnd[1] = P.esc_log10a;
    cnd[2] = fabsf(xc);
    cnd[3] = CF.q[0]; cnd[4] = CF.q[1]; cnd[5] = CF.q[2];
    cnd[6] = ldep;
#pragma unroll
    for (int r = 0; r < 3; ++r)
        cnd[7 + r] = pick3(CF.sg[0], CF.sg[1], CF.sg[2], CF.perm[r]) * pick3(nx, ny, nz, CF.perm[r]);
}

// ------------------------------------------------ continuous temperature ---
// A cell of Doppler width r b_ref: frequency scale sc = 1 / r (and back, isc),
// its damping ac = a / r, the Voigt blocks around ac with the weight of the
// upper one (linear in ln a), and the nearest sampler node (block offset, its
// damping and sampler threshold).
struct ContCell {
    float sc, isc, ac, tv, sa, sthd;
    int voff, toff;
};
__device__ __forceinline__ ContCell cont_cell(const RunParams &P, float a, float r) {
    ContCell c;
    c.isc = r;
    c.sc = 1.0f / r;
    c.ac = a * c.sc;
    const float s = logf(c.ac) - P.cv_lna0;
    const float uv = fminf(fmaxf(s * P.cv_inv_step, 0.0f), (float)(P.cv_n - 1));
    const int kv = min((int)uv, max(P.cv_n - 2, 0));
    c.tv = uv - (float)kv;
    c.voff = kv * kVoigtFloats;
    const int ks = min((int)(fmaxf(s * P.cs_inv_step, 0.0f) + 0.5f), P.cs_n - 1);
    c.toff = ks * kTabFloats;
    const float2 sp = P.cs_par[ks];
    c.sa = sp.x;
    c.sthd = sp.y;
    return c;
}
// H(ac, |x|) between the two Voigt blocks
__device__ __forceinline__ float cont_voigt(const RunParams &P, int voff, float tv, float xa) {
    const float h0 = voigt_lds(P.cv_tab + voff, xa);
    return fmaf(tv, voigt_lds(P.cv_tab + voff + kVoigtFloats, xa) - h0, h0);
}

// --------------------------------------------------------------- kernel ---
// Distance along one axis to the face ahead: n the direction's component, f the
// position in the cell, dx its width.  A zero component gives +inf, or NaN (0
// times inf) for a packet exactly on the face; the minimum over the axes
// ignores a NaN as it ignores +inf, and the direction has another component.
// A subnormal component counts as zero (its reciprocal is +inf).
__device__ __forceinline__ float face_dist(float n, float f, float dx) {
    const float up = fminf(fmaxf(n * 0x1p126f, 0.0f), 1.0f);  // 1 toward the upper face, 0 toward the lower
    return fabsf(f - up) * dx * f_rcp(fabsf(n));
}

// kProf: 0 tables in LDS (production); 1 the same tables read from global
// memory (the workgroup still stages them, so occupancy is unchanged and only
// the memory space of the lookups differs); 2 analytic opacity profile in the
// flights, tables for the redistribution; 3 per-cell temperature classes: in a
// cell of Doppler width b the gas-frame frequency is (x - n.v) b_ref / b, the
// damping a b_ref / b, and the class's own tables (global memory) serve the
// opacity and the redistribution; frequencies return to reference units on
// leaving the cell's frame.
// kDip: dipole phase (plain walk; the learned escape is isotropic).
// kRec: quads of the cell records (P.rec) that the fields are read from, 0 for
// the fields' own arrays.
//
// A lane's iteration has three parts: the flight of every live lane (opacity,
// distance to the face, position), then the cell change of the lanes that
// cross, then the scattering of the lanes that interact, which also draws the
// random words of their next event.  The walk is bound by instruction issue
// when the waves are full and by the latency of one lane's chain when few
// packets are left, so each part is written without branches: selects between
// the table pieces, one LDS read per lookup, the tally bin from its guess
// unless the frequency is within rounding of a bin edge.  Every product and sum
// is a fixed one (fmaf where it is fused, contraction off otherwise), so that
// all variants walk a packet through the same numbers.
// Measured against the walk of nested branches that scattered ahead of the
// flight: expanding 128^3 sphere, 4e6 packets (full waves) 5.4e10 to 1.0e11
// scatterings/s; the longest packet of a thick slab 1146 to 605 ns an event
// without an emissivity tally, 1708 to 718 with 32 channels.
// 1024 lanes (16 waves) share a workgroup's copy of the tables in LDS.
//
// The launch's parameters re-read where they are used: for the paths a packet
// takes rarely (crossings, refills, retirements).  Read through P the compiler
// keeps them all in scalar registers across the loop, which are too few, and
// every scattering then pays for moving its own constants in and out.
typedef const __attribute__((address_space(4))) RunParams *ColdParams;
__device__ __forceinline__ ColdParams cold_params() {
    ColdParams p = (ColdParams)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

template <int kMode, int kMaxThreads, int kProf = 0, bool kDip = false, int kRec = 0>
__global__ void __launch_bounds__(kMaxThreads) mc_transport_kernel(RunParams P) {
#pragma clang fp contract(off)
    constexpr bool kEsc = kMode == kModeFused, kPark = kMode == kModePark;
    constexpr bool kTemp = kProf == 3 || kProf == 4;  // per-cell temperature: classes or continuum
    extern __shared__ float4 lds4[];
    const float *T = (kProf == 1) ? P.tab : reinterpret_cast<const float *>(lds4);
    // bin edges after the tables: spectrum then channels; the network variant
    // reads the spectrum edges (once per escaped packet) from global memory, so
    // that its LDS holds the tables, the channel edges and the network image
    constexpr int kLdsSpec = kEsc ? 0 : (kMaxSpecBins + 1);
    constexpr int kLdsMlp = kTabFloats + kChanEdgeFloats;  // floats before the network image
    float *ledges = reinterpret_cast<float *>(lds4) + kTabFloats;
    const float *sedges = kEsc ? P.spec_edges : ledges;  // spectrum edges
    float *cedges = ledges + kLdsSpec;                    // channel edges
    // then the workgroup's counters, then the dipole windows
    unsigned long long *lcnt =
        reinterpret_cast<unsigned long long *>(lds4 + (kEsc ? kLdsMlp + kMlpFwdBytes / 4 : kTabFloats + kEdgeFloats) / 4);
    EmisWindow<kDip> E;
    E.size = min(kEmisSlots, P.emis_nch);
    {
        const float4 *src = reinterpret_cast<const float4 *>(P.tab);
        for (int i = threadIdx.x; i < kTabFloats / 4; i += blockDim.x) lds4[i] = src[i];
        if (!kEsc)
            for (int i = threadIdx.x; i <= P.spec_nb; i += blockDim.x) ledges[i] = P.spec_edges[i];
        for (int i = threadIdx.x; i <= P.emis_nch; i += blockDim.x) cedges[i] = P.ch_edges[i];
        if (kEsc) {
            const float4 *ms = reinterpret_cast<const float4 *>(P.mlp_img);
            float4 *md = lds4 + kLdsMlp / 4;
            for (int i = threadIdx.x; i < kMlpFwdBytes / 16; i += blockDim.x) md[i] = ms[i];
        }
        if (threadIdx.x < kNLdsCounters) lcnt[threadIdx.x] = 0ull;
        if constexpr (kDip) {
            E.stride = (int)blockDim.x;
            E.acc = reinterpret_cast<int64_t *>(lcnt + kNLdsCounters) + threadIdx.x;
            if (P.emis_raw)
                for (int k = 0; k < kEmisSlots; ++k) E.acc[k * E.stride] = 0;
        }
    }
    __syncthreads();
    const unsigned char *mimg = reinterpret_cast<const unsigned char *>(lds4 + kLdsMlp / 4);
    const float *mbias = reinterpret_cast<const float *>(mimg + kTilesFwd * kTileBytes);
    const float *mnorm = mbias + kBiasFloats;

    const int lane = __lane_id();
    const uint64_t lanemask_lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    float a = P.a, thd = P.thd;
    // what every iteration reads stays in vector registers: as scalars these
    // values are too many, and would be loaded again, with a wait, in each
    float dx0 = P.dx[0], dx1 = P.dx[1], dx2 = P.dx[2], idx0 = P.inv_dx[0], idx1 = P.inv_dx[1], idx2 = P.inv_dx[2];
    float cx = P.n_cam[0], cy = P.n_cam[1], cz = P.n_cam[2];
    float ch_off = P.ch_off, ch_inv_w = P.ch_inv_w, ch_safe = P.ch_safe;
    if constexpr (!kEsc) {
        asm volatile("" : "+v"(a), "+v"(thd), "+v"(dx0), "+v"(dx1), "+v"(dx2), "+v"(idx0), "+v"(idx1), "+v"(idx2));
        asm volatile("" : "+v"(cx), "+v"(cy), "+v"(cz), "+v"(ch_off), "+v"(ch_inv_w), "+v"(ch_safe));
    }

    // lane state
    float sc = 1.0f, isc = 1.0f, ac = a, thdc = thd;  // cell temperature (kProf 3, 4)
    float sac = a, tv = 0.0f;  // continuum (kProf 4): the sampler node's damping, upper Voigt weight
    int toff = 0, voff = 0;
    // kLive, kNeed (a packet), kDone (the pool is empty), or above kLive: retiring
    // with outcome state - kLive (1 escaped, 2 destroyed, 3 stuck)
    constexpr int kDone = -1, kNeed = 0, kLive = 1;
    int state = kNeed;
    uint64_t pid = 0;
    PhiloxPacket pk{};
    int ci = 0, cj = 0, ck = 0, cell = 0;
    float fx = 0.f, fy = 0.f, fz = 0.f;
    float nx = 0.f, ny = 0.f, nz = 1.f;
    float x = 0.f, tau = 0.f;
    uint32_t ev = 0, wa1 = 0, wa2 = 0, wa3 = 0;
    uint4 wb = make_uint4(0u, 0u, 0u, 0u);
    float k0c = 0.f, vxc = 0.f, vyc = 0.f, vzc = 0.f, epsc = 0.f, kabsc = 0.f;
    uint32_t nscat_pkt = 0, ncross_pkt = 0;
    uint32_t ndrop = 0;  // scatterings of the packet outside the channels, in this lane
    uint32_t seg = 0;  // plain scatterings of the packet in this launch (park mode)
    bool pend = false;   // fused mode: a qualifying scattering waits for its wave's next call batch
    uint32_t pwait = 0;  // ... for this many loop iterations so far
    int64_t jacc = 0;
    int64_t c_mlp = 0, c_skip = 0, c_drop = 0;  // network calls
    const float jscale = P.jbar_scale * kInvSqrtPiF;
    const bool emis_on = P.emis_raw != nullptr, jbar_on = P.jbar_raw != nullptr;
    const bool destroys = P.eps != nullptr || P.kabs != nullptr;  // uniform
    const uint32_t max_events = (uint32_t)P.max_events;
    auto count = [&](int slot, uint64_t v) __attribute__((always_inline)) { atomicAdd(&lcnt[slot], (unsigned long long)v); };

    // entering a cell: its fields, and with temperature classes or a continuum
    // of widths its frequency scale, damping, sampler threshold and table set
    struct CellFields {
        const float *k0, *vx, *vy, *vz, *eps, *kabs;
        const float4 *rec;
        __device__ __forceinline__ void load(ColdParams C) {
            if constexpr (kRec > 0) {
                rec = C->rec;
                return;
            }
            k0 = C->k0; vx = C->vx; vy = C->vy; vz = C->vz; eps = C->eps; kabs = C->kabs;
            asm volatile("" : "+s"(k0), "+s"(vx), "+s"(vy), "+s"(vz), "+s"(eps), "+s"(kabs));
        }
    };
    auto enter_cell = [&](const CellFields &F) __attribute__((always_inline)) {
        if constexpr (kRec > 0) {
            const float4 *r = F.rec + (int64_t)cell * kRec;
            const float4 q = r[0];
            k0c = q.x; vxc = q.y; vyc = q.z; vzc = q.w;
            if constexpr (kRec == 2) {
                const float2 e = *reinterpret_cast<const float2 *>(r + 1);
                epsc = e.x; kabsc = e.y;
            }
        } else {
            k0c = F.k0[cell];
            if (F.vx) { vxc = F.vx[cell]; vyc = F.vy[cell]; vzc = F.vz[cell]; }
            if (F.eps) epsc = F.eps[cell];
            if (F.kabs) kabsc = F.kabs[cell];
        }
        if constexpr (kProf == 3) {
            const int k = P.tclass[cell];
            const float4 cp = P.cls_par[k];
            sc = cp.x; ac = cp.y; thdc = cp.z; isc = cp.w;
            sac = ac;
            toff = k * kTabFloats;
        }
        if constexpr (kProf == 4) {
            const ContCell cc = cont_cell(P, a, P.bratio[cell]);
            sc = cc.sc; isc = cc.isc; ac = cc.ac; tv = cc.tv;
            sac = cc.sa; thdc = cc.sthd;
            voff = cc.voff; toff = cc.toff;
        }
    };
    auto locate = [&]() __attribute__((always_inline)) {
        const ColdParams C = cold_params();
        ci = cell % C->n[0];
        cj = (cell / C->n[0]) % C->n[1];
        ck = cell / (C->n[0] * C->n[1]);
    };
    auto gas_freq = [&]() __attribute__((always_inline)) {
#pragma clang fp contract(off)
        if constexpr (kTemp) return (x - dot3(ny, vyc, nx, vxc, nz, vzc)) * sc;
        else return x - dot3(nx, vxc, ny, vyc, nz, vzc);
    };
    // random words of event ev: optical depth, destruction, sampler; then the
    // second block's four
    auto draw_event = [&]() __attribute__((always_inline)) {
        uint4 A;
        philox_pair(pk, ev, P.key0, P.key1, A, wb);
        tau = -f_log(u01(A.x));
        wa1 = A.y; wa2 = A.z; wa3 = A.w;
    };
    auto flush_emis = [&]() __attribute__((always_inline)) {
        const ColdParams C = cold_params();
        E.flush(C->emis_raw + (int64_t)cell * C->emis_nch, C->emis_frac_bits);
    };
    auto flush_jbar = [&]() __attribute__((always_inline)) {
        if (jacc != 0) { tally_add_i64(cold_params()->jbar_raw + cell, jacc); jacc = 0; }
    };
    auto give_up = [&]() __attribute__((always_inline)) {
        atomicOr(cold_params()->status, (uint32_t)KRT_ST_STUCK_BIT);
        state = kLive + 3;
    };

    // the table entries a lane's gas-frame frequency selects, read together: the
    // sampler's wait for the flight's opacity costs it nothing then
    struct Lookup {
        float H;
        UparMass m;
    };
    auto look_up = [&](float xc) __attribute__((always_inline)) {
        Lookup q;
        const float xa = fabsf(xc);
        const float *TL = kTemp ? ((kProf == 4) ? P.cs_tab : P.cls_tab) + toff : T;
        const VoigtEntry e = voigt_entry(TL, xa);
        q.m = upar_mass(TL, e);
        if constexpr (kProf == 2) q.H = voigt_analytic(a, P.voigt_u0, xa);
        else if constexpr (kProf == 4) q.H = cont_voigt(P, voff, tv, xa);
        else q.H = voigt_value(e, xa);
        return q;
    };

    // one flight segment: to the next interaction, or to the face of the cell
    struct Segment {
        float kap, dtau, tx, ty, tm;
        bool hit;  // an interaction inside the cell
    };
    auto segment = [&](float H) __attribute__((always_inline)) {
#pragma clang fp contract(off)
        Segment q;
        H = (k0c > 0.0f) ? H : 0.0f;
        // line opacity plus the cell's grey absorption (exactly k0 H without one)
        q.kap = fmaf(k0c, H, kabsc);
        q.tx = face_dist(nx, fx, dx0);
        q.ty = face_dist(ny, fy, dx1);
        q.tm = fminf(fminf(q.tx, q.ty), face_dist(nz, fz, dx2));
        const float dmin = fmaxf(q.tm, 0.0f);
        q.dtau = q.kap * dmin;
        q.hit = (q.kap > 0.0f) & (q.dtau >= tau);
        const float l = sel(q.hit, tau * f_rcp(q.kap), dmin);
        fx = fminf(fmaxf(fmaf(l * nx, idx0, fx), 0.0f), 1.0f);
        fy = fminf(fmaxf(fmaf(l * ny, idx1, fy), 0.0f), 1.0f);
        fz = fminf(fmaxf(fmaf(l * nz, idx2, fz), 0.0f), 1.0f);
        if (jbar_on) {
            asm volatile("");  // a branch: not computed and dropped by every run without the tally
            jacc += (int64_t)__float2ll_rn(l * H * jscale);
        }
        return q;
    };
    // ... which the packet crosses: escape, periodic wrap or the next cell
    auto cross = [&](const Segment &q) __attribute__((always_inline)) {
        // every parameter of the crossing at once: one wait instead of one at each use
        const ColdParams C = cold_params();
        const int gn0 = C->n[0], gn1 = C->n[1], gn2 = C->n[2], b0 = C->bc[0], b1 = C->bc[1], b2 = C->bc[2];
        CellFields F;
        F.load(C);
        tau -= q.dtau;
        ncross_pkt += 1;
        // leaving the cell: flush its tallies
        if (jbar_on) flush_jbar();
        if (emis_on) flush_emis();
        const bool ax0 = q.tx == q.tm, ax1 = !ax0 && q.ty == q.tm;  // ties go to the lower axis
        const float na = by_axis(ax0, ax1, nx, ny, nz);
        const int st = na > 0.0f ? 1 : -1;
        const float fn = na > 0.0f ? 0.0f : 1.0f;
        const int na_n = by_axis(ax0, ax1, gn0, gn1, gn2);
        const bool periodic = by_axis(ax0, ax1, b0, b1, b2) != 0;
        int c = by_axis(ax0, ax1, ci, cj, ck) + st;
        const bool out = (unsigned)c >= (unsigned)na_n;
        c = out ? (st > 0 ? 0 : na_n - 1) : c;  // the wrapped cell of a periodic axis
        fx = ax0 ? fn : fx;
        fy = ax1 ? fn : fy;
        fz = (ax0 || ax1) ? fz : fn;
        if (out && !periodic) {
            const int b = bin_index(x, sedges, C->spec_nb, C->spec_inv_w);
            if (b < 0) atomicOr(C->status, (uint32_t)KRT_ST_NAN_BIT);
            else atomicAdd(reinterpret_cast<unsigned long long *>(C->spec_raw + b), 1ull);
            state = kLive + 1;
        } else if (ncross_pkt > kMaxCrossings) {
            give_up();
        } else {
            ci = ax0 ? c : ci;
            cj = ax1 ? c : cj;
            ck = (ax0 || ax1) ? ck : c;
            cell = (ck * gn1 + cj) * gn0 + ci;
            enter_cell(F);
        }
    };
    // an interaction is an absorption with probability p_d = kabs / kap, else a
    // line scattering destroyed with probability eps: one uniform decides both
    auto destroyed = [&](const Segment &q, float ue) __attribute__((always_inline)) {
#pragma clang fp contract(off)
        const float pd = (kabsc > 0.0f) ? kabsc * f_rcp(q.kap) : 0.0f;
        return ue < fmaf(1.0f - pd, epsc, pd);
    };

    // the resonant scattering of a live lane at gas-frame frequency xc with its
    // event's draws (eq. riia-scatter), and its emissivity tally
    // (unit = 1; a lane without a packet may pass through with unit = 0, tallying
    // nothing)
    auto scatter = [&](float xc, const UparMass &m, const SDraws &b, uint32_t unit) __attribute__((always_inline)) {
#pragma clang fp contract(off)
        const float upar = kTemp ? upar_from(((kProf == 4) ? P.cs_tab : P.cls_tab) + toff, m, xc, sac, thdc, b.r1, b.r2, b.xw)
                                 : upar_from(T, m, xc, a, thd, b.r1, b.r2, b.xw);
        const Basis e = scatter_basis(nx, ny, nz);
        float ox, oy, oz;
        scatter_turn(nx, ny, nz, e, b, ox, oy, oz);
        float xo = scatter_shift(xc, upar, b);
        if constexpr (kTemp) xo *= isc;  // back to reference units
        if (emis_on) {
            const float gc = dot3(nx, cx, ny, cy, nz, cz);
            const float upc = fmaf(b.up1, dot3(e.e1x, cx, e.e1y, cy, e.e1z, cz),
                                   b.up2 * dot3(e.e2x, cx, e.e2y, cy, e.e2z, cz));
            float xcam = fmaf(upar, gc - 1.0f, xc) + upc;
            const float vc = dot3(cx, vxc, cy, vyc, cz, vzc);
            xcam = kTemp ? fmaf(xcam, isc, vc) : xcam + vc;
            bool sure;
            int ch = channel_guess(xcam, ch_inv_w, ch_off, ch_safe, sure);
            const bool other = (unit != 0) & (!sure | ((unsigned)(ch - E.w) >= (unsigned)E.size));
            if (__ballot(other) != 0ull) {  // wave-uniform: rare
                if (other) {
                    const int nch = P.emis_nch;
                    if (!sure) ch = bin_index(xcam, cedges, nch, ch_inv_w) - 1;
                    if ((unsigned)ch >= (unsigned)nch) {
                        ndrop += 1;
                        unit = 0;
                    } else if ((unsigned)(ch - E.w) >= (unsigned)E.size) {
                        flush_emis();
                        E.move(ch, nch);
                    }
                }
            }
            int64_t wq = 0;
            if constexpr (kDip) {
                // contributions below 2^32 (F <= 30) convert through 32 bits
                const float wf = unit ? 0.75f * fmaf(gc, gc, 1.0f) * P.frac_scale : 0.0f;
                wq = P.emis_w32 ? (int64_t)__float2uint_rn(wf) : (int64_t)__float2ll_rn(wf);
            }
            E.add(ch, unit, wq);
        }
        nx = ox; ny = oy; nz = oz;
        x = fmaf(vzc, nz, fmaf(vyc, ny, fmaf(vxc, nx, xo)));
        nscat_pkt += 1;
    };

    // a retired packet: write back the tallies of its last cell, count and log it
    auto retire = [&]() __attribute__((always_inline)) {
        const int outcome = state - kLive;
        if (jbar_on) flush_jbar();
        if (emis_on) flush_emis();
        count(outcome - 1, 1);
        count(kLcScat, nscat_pkt);
        count(kLcCross, ncross_pkt);
        if (ndrop) { count(kLcDrop, ndrop); ndrop = 0; }
        const ColdParams C = cold_params();
        if (C->plog) {
            float *L = C->plog + 8 * (pid - C->packet_offset);
            L[0] = x; L[1] = (float)nscat_pkt; L[2] = (float)outcome;
            L[3] = nx; L[4] = ny; L[5] = nz;
            L[6] = (float)cell; L[7] = (float)ev;
        }
        state = kNeed;
    };

    // park mode: lanes with a qualifying scattering (kind 1), or past their
    // round's budget of plain scatterings (kind 0, after committing one), leave
    // as records (their cell's register tallies flushed first); one
    // wave-aggregated atomic takes the slots.  A parked lane is free for new
    // work, with no outcome.  The budget bounds a round by its slowest packet.
    auto park = [&](bool want, bool &scat, float xc, uint32_t kind) __attribute__((always_inline)) {
        const uint64_t pm = __ballot(want);
        if (pm == 0ull) return;
        const int leader = __ffsll((long long)pm) - 1;
        unsigned long long base = 0;
        if (lane == leader) base = atomicAdd(P.park_count, (unsigned long long)__popcll(pm));
        base = __shfl(base, leader, 64);
        if (want) {
            if (jbar_on) flush_jbar();
            if (emis_on) flush_emis();
            if (ndrop) { count(kLcDrop, ndrop); ndrop = 0; }
            const uint64_t slot = base + (uint64_t)__popcll(pm & lanemask_lt);
            if (slot < P.park_cap) {
                uint4 *r = P.park_out + kParkQuads * slot;
                r[0] = make_uint4((uint32_t)pid, (uint32_t)(pid >> 32), ev, (uint32_t)cell);
                r[1] = make_uint4(__float_as_uint(fx), __float_as_uint(fy), __float_as_uint(fz), __float_as_uint(x));
                r[2] = make_uint4(__float_as_uint(nx), __float_as_uint(ny), __float_as_uint(nz), nscat_pkt);
                r[3] = make_uint4(ncross_pkt, __float_as_uint(xc), kind, 0u);
            } else {
                atomicOr(P.status, (uint32_t)KRT_ST_STUCK_BIT);  // the host sizes the list; never expected
                count(kLcStuck, 1);
                count(kLcScat, nscat_pkt);
                count(kLcCross, ncross_pkt);
            }
            state = kNeed;
            scat = false;
        }
    };

    // the event of this lane is over (scattering walked, or a call): the next one's draws
    auto next_event = [&](auto draw) __attribute__((always_inline)) {
        ev += 1;
        draw();
    };
    // packets past their last event, and those that ended
    auto settle = [&]() __attribute__((always_inline)) {
        const bool over = ev > max_events;
        if (over || state > kLive) {
            if (over && state == kLive) give_up();
            if (state > kLive) retire();
        }
    };

    WorkPool pool;
    pool.init(P.first_lanes);
    int ticks = kEmisTicks;
    bool tail = false;
    for (;;) {
        // ---- refill idle lanes from the global queue -----------------------
        const uint64_t need_mask = __ballot(state == kNeed);
        if (pool.due(need_mask, __ballot(state == kLive) != 0ull)) {
            bool need = state == kNeed;
            const ColdParams C = cold_params();
            const uint64_t n_res = C->n_res, n_work = n_res + C->n_packets;
            const uint64_t idx = pool.take(need_mask, lane, lanemask_lt, C->work_counter, n_work, C->first_lanes);
            if (need && idx >= n_work) { state = kDone; need = false; }
            const bool fresh_pkt = need && idx >= n_res;
            const uint64_t fm = __ballot(fresh_pkt);
            if (fm && lane == __ffsll((long long)fm) - 1) count(kLcEmit, (uint64_t)__popcll(fm));
            if (need) {
                CellFields F;
                F.load(C);
                if (!fresh_pkt) {
                    // ---- a packet back from a network call: its next event ----
                    const uint4 *r = C->res_in + kParkQuads * idx;
                    const uint4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
                    pid = (uint64_t)r0.x | ((uint64_t)r0.y << 32);
                    ev = r0.z;
                    cell = (int)r0.w;
                    locate();
                    fx = __uint_as_float(r1.x); fy = __uint_as_float(r1.y); fz = __uint_as_float(r1.z);
                    x = __uint_as_float(r1.w);
                    nx = __uint_as_float(r2.x); ny = __uint_as_float(r2.y); nz = __uint_as_float(r2.z);
                    nscat_pkt = r2.w;
                    ncross_pkt = r3.x;
                    enter_cell(F);
                } else {
                    // ---- emission (event 0) ----------------------------------
                    pid = C->packet_offset + C->new_lo + (idx - n_res);
                    const uint32_t plo = (uint32_t)pid, phi = (uint32_t)(pid >> 32);
                    uint4 e0 = philox(make_uint4(0u, plo, phi, 0u), C->key0, C->key1);
                    if (C->source == KRT_SRC_BEAM_I) {
                        nx = C->src_dir[0]; ny = C->src_dir[1]; nz = C->src_dir[2];
                    } else {
                        float mu = fmaf(2.0f, u01(e0.x), -1.0f);
                        float st = f_sqrt(fmaxf(0.0f, fmaf(-mu, mu, 1.0f)));
                        float ph = u01(e0.y);
                        nx = st * cos_rev(ph); ny = st * sin_rev(ph); nz = mu;
                    }
                    if (C->source == KRT_SRC_VOLUME_I) {
                        uint4 e1 = philox(make_uint4(0u, plo, phi, 1u), C->key0, C->key1);
                        int col = (int)__umulhi(e0.z, (uint32_t)C->ncell);
                        cell = (u01(e0.w) < C->alias_prob[col]) ? col : C->alias_idx[col];
                        locate();
                        fx = u01(e1.x); fy = u01(e1.y); fz = u01(e1.z);
                    } else {
                        int c3[3]; float f3[3];
                        float nd[3] = {nx, ny, nz};
                        double u2[2] = {0.0, 0.0};
                        if (C->source == KRT_SRC_PLANE_I) {
                            uint4 e1 = philox(make_uint4(0u, plo, phi, 1u), C->key0, C->key1);
                            u2[0] = (double)u01(e1.x); u2[1] = (double)u01(e1.y);
                        }
#pragma unroll
                        for (int d = 0; d < 3; ++d) {
                            double X = C->src_pos[d];
                            if (C->source == KRT_SRC_PLANE_I && d < 2) X = fma(u2[d], C->hi[d] - C->lo[d], C->lo[d]);
                            double f = (X - C->lo[d]) / C->dxd[d];
                            double fl = floor(f);
                            int c = (int)fl;
                            float fr = (float)(f - fl);
                            if (fl == f && nd[d] < 0.0f) { c -= 1; fr = 1.0f; }
                            if (c < 0) { c = 0; fr = 0.0f; }
                            if (c >= C->n[d]) { c = C->n[d] - 1; fr = 1.0f; }
                            c3[d] = c; f3[d] = fr;
                        }
                        ci = c3[0]; cj = c3[1]; ck = c3[2];
                        fx = f3[0]; fy = f3[1]; fz = f3[2];
                        cell = (ck * C->n[1] + cj) * C->n[0] + ci;
                    }
                    enter_cell(F);
                    float xg = C->src_x0;
                    if (C->src_profile != KRT_PROF_DELTA_I) {
                        uint4 e2 = philox(make_uint4(0u, plo, phi, 2u), C->key0, C->key1);
                        float rr = f_sqrt(-f_log(u01(e2.x)));
                        float th = u01(e2.y);
                        xg = rr * cos_rev(th);
                        if (C->src_profile == KRT_PROF_VOIGT_I) {
                            float c = u01(e2.z) - 0.5f;  // Cauchy(a): a tan(pi c)
                            xg = fmaf((kTemp ? ac : a) * sin_rev(0.5f * c), f_rcp(cos_rev(0.5f * c)), xg);
                        }
                        if constexpr (kTemp) xg *= isc;  // the emitting cell's units -> reference
                    }
                    x = fmaf(nz, vzc, fmaf(ny, vyc, fmaf(nx, vxc, xg)));
                    ev = 0;
                    nscat_pkt = 0;
                    ncross_pkt = 0;
                }
                pk = philox_packet((uint32_t)pid, (uint32_t)(pid >> 32), P.key0, P.key1);
                seg = 0;
                jacc = 0;
                state = kLive;
                next_event(draw_event);
                if (ev > max_events) give_up();
            }
            // (a packet resumed past its last event is neither live nor done: it
            // retires below)
            if (__ballot(state != kDone) == 0ull) break;
            // pool exhausted and few live lanes: continue in tail mode
            if (!kEsc && P.tail_lanes > 0 && __ballot(state == kDone) != 0ull &&
                __popcll(__ballot(state == kLive)) <= P.tail_lanes) {
                tail = true;
                break;
            }
        }
        if constexpr (!kDip) {
            if (--ticks == 0) {
                asm volatile("");
                ticks = kEmisTicks;
                if (emis_on) flush_emis();
            }
        }

        // ---- one flight segment (divergent) --------------------------------
        const float xc = gas_freq();
        const Lookup tl = look_up(xc);
        const bool fly = (state == kLive) & !pend;
        Segment sg{};
        // (the position of a lane without a packet is of no use to anyone)
        if (!kEsc || fly) sg = segment(tl.H);
        bool scat = fly & sg.hit;
        if (fly & !sg.hit) cross(sg);
        if (!kEsc && destroys) {
            asm volatile("");
            if (scat && destroyed(sg, u01(wa1))) {
                state = kLive + 2;
                scat = false;
            }
        }

        // ---- learned whole-cell escape ---------------------------------------
        // At a scattering inside a thick cubic cell, at least esc_depth_min below
        // its nearest face and in the line core, one network sample replaces the
        // walk until the photon leaves the cell: exit face, point, direction and
        // frequency, and the expected number of scatterings skipped.  Fused mode
        // evaluates the network here, batched over the asking lanes of the wave
        // (wave-uniform); park mode writes the packet to the park list and frees
        // the lane, and escape_call_kernel applies the call.
        bool mlp = false, go = false;
        if (kPark) {
            CellFrame CF{};
            float ltc = 0.0f, ldep = 0.0f;
            if (scat) mlp = call_eligible(P, k0c, fx, fy, fz, xc, CF, ltc, ldep);
        }
        if (kEsc) {
            if (scat || pend) mlp = call_ok(P, k0c, fx, fy, fz, xc);
            // once the packet pool is exhausted (some lane of this wave is done) the
            // wave lives only as long as its slowest packet: fewer asking lanes suffice.
            // With waiting on (esc_wait > 0) a qualifying lane that finds too few
            // others holds its scattering (pend) instead of walking it, for at most
            // esc_wait iterations; the batch also goes when every live lane asks.
            // While the pool lasts and nothing forces the batch, it takes whole
            // 16-sample blocks only: the askers past them, in lane order, stay held.
            const uint64_t wm = __ballot(mlp);
            const bool tailw = __ballot(state == kDone) != 0ull;
            const int need_lanes = tailw ? P.esc_tail_lanes : P.esc_min_lanes;
            const bool forced = wm == __ballot(state == kLive) || __ballot(pend && pwait >= P.esc_wait) != 0ull;
            go = wm != 0ull && (__popcll(wm) >= need_lanes || forced);  // wave-uniform
            bool held = !go;
            if (go && !tailw && !forced && P.esc_wait > 0 && mlp && __popcll(wm) >= 16)
                held = __popcll(wm & lanemask_lt) >= (__popcll(wm) & ~15);
            if (held) {
                if (mlp && P.esc_wait > 0) {
                    pwait = pend ? pwait + 1 : 1;
                    pend = true;
                }
                mlp = false;
            }
        }

        // ---- resonant scattering (event ev), divergent -----------------------
        const bool walk = scat && !mlp && !pend;
        if (walk) {
            SDraws b;
            scatter_draws(wa2, wa3, wb, kDip, b);
            scatter(xc, tl.m, b, 1);
            if constexpr (!kEsc && !kPark) next_event(draw_event);
        }
        if (kPark) {
            const bool cont = walk && ++seg >= P.park_budget;
            bool go_on = walk;
            park(mlp || cont, go_on, xc, mlp ? 1u : 0u);
            if (go_on) next_event(draw_event);
        }
        if (kEsc) {
            if (go) {
                const uint64_t wm = __ballot(mlp);  // the lanes this batch serves
                CellFrame CF{};
                float ltc, ldep;
                {
                    float tc, dep;
                    call_frame(P, k0c, fx, fy, fz, CF, tc, dep);
                    ltc = __log10f(tc);
                    ldep = __log10f(dep);
                }
                const uint32_t plo = (uint32_t)pid, phi = (uint32_t)(pid >> 32);
                const uint4 C = philox(make_uint4(ev, plo, phi, 2u), P.key0, P.key1);
                const uint4 D = philox(make_uint4(ev, plo, phi, 3u), P.key0, P.key1);
                float cnd[10];
                call_condition(P, CF, ltc, ldep, xc, nx, ny, nz, cnd);
                int face;
                float xo, mo[kMlpOut];
                call_network(mimg, mbias, mnorm, lane, wm, cnd, C, D, face, xo, mo);
                if (mlp) {
                    int64_t *ebase = P.emis_raw ? P.emis_raw + (int64_t)cell * P.emis_nch : nullptr;
                    // the deposit spans consecutive channels, each once: direct atomics
                    call_apply(P, mnorm, cedges, CF, mo, face, xo, C.z, ltc, ldep, xc, vxc, vyc, vzc, fx, fy,
                               fz, nx, ny, nz, x, c_skip, c_drop,
                               [&](int ch, int64_t w) __attribute__((always_inline)) { tally_add_i64(ebase + ch, w); });
                    c_mlp += 1;
                    pend = false;
                }
            }
            // an event is consumed by a walked scattering or a call; a held one waits
            if (walk || mlp) next_event(draw_event);
        }
        settle();
    }
    // ---- tail mode ------------------------------------------------------------
    // The packet pool is exhausted and at most tail_lanes lanes are live, so the
    // wave lasts as long as its slowest packet.  The idle lanes precompute the
    // random draws of the live packets' coming events: with k live lanes, lane j
    // holds the draws of event ev0 + j / k of the live lane of rank j % k, and a
    // live lane fetches its event's draws by a cross-lane read.  The draws are
    // the same words mapped by the same functions as in the loop above, so the
    // tallies do not depend on where a packet switches mode.
    // Such a wave is bound by the latency of one packet's chain and issues an
    // instruction only every few cycles, a branch with its change of the lane
    // mask every ten or so.  What need not be looked at for each event (draws
    // used up, window counts, the event limit) is counted down together in a
    // scalar, and the lanes without a packet go along, so that while no lane
    // crosses a face an event is one straight piece of code.
    if (!kEsc && tail) {
        int left = 0;         // events until the next look
        int k = 1;            // live lanes when the bank was filled
        int at = 0;           // 4 x the lane that holds this lane's draws (bpermute's address)
        bool fresh = false;   // set after a scattering: tau of the new event comes from the draws
        uint32_t unit = 0;    // 1 for a live lane
        float pt = 0.f, pue = 0.f;
        SDraws pb{};
        for (;;) {
            if (left == 0) {
                settle();
                const uint64_t live = __ballot(state == kLive);
                if (live == 0ull) break;
                if constexpr (!kDip) {
                    if (ticks <= 64) {
                        ticks = kEmisTicks;
                        if (emis_on) flush_emis();
                    }
                }
                k = __popcll(live);
                left = 64 / k;  // each lane's share of the bank
                ticks -= left;
                if (__ballot(state == kLive && max_events - ev < 64u) != 0ull) left = 1;
                unit = state == kLive ? 1u : 0u;
                const int owner = nth_set_lane(live, lane % k);
                PhiloxPacket op;
                op.bk = __shfl(pk.bk, owner, 64);
                op.hk = __shfl(pk.hk, owner, 64);
                op.la = __shfl(pk.la, owner, 64);
                const uint32_t e = __shfl(ev, owner, 64) + (uint32_t)(lane / k);
                uint4 A, B;
                philox_pair(op, e, P.key0, P.key1, A, B);
                pt = -f_log(u01(A.x));
                pue = u01(A.y);
                scatter_draws(A.z, A.w, B, kDip, pb);
                at = 4 * __popcll(live & lanemask_lt);
            }
            --left;
            auto fetch = [&](float v) __attribute__((always_inline)) {
                return __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(v)));
            };
            const float dt = fetch(pt);
            SDraws db;
            db.r1 = fetch(pb.r1); db.r2 = fetch(pb.r2); db.xw = fetch(pb.xw);
            db.g = fetch(pb.g); db.sg = fetch(pb.sg);
            db.cp = fetch(pb.cp); db.sp = fetch(pb.sp);
            db.kick = fetch(pb.kick);
            db.up1 = fetch(pb.up1); db.up2 = fetch(pb.up2);
            tau = sel(fresh, dt, tau);
            fresh = false;
            const float xc = gas_freq();
            const Lookup tl = look_up(xc);
            const bool have = state == kLive;
            const Segment sg = segment(tl.H);
            if (!kPark && !destroys && __ballot(have & !sg.hit) == 0ull) {
                scatter(xc, tl.m, db, unit);
                next_event([&]() __attribute__((always_inline)) { fresh = true; at += 4 * k; });
                continue;
            }
            float due = 0.0f;
            if (destroys) due = fetch(pue);
            bool walk = have & sg.hit;
            if (have & !sg.hit) cross(sg);
            if (destroys && walk && destroyed(sg, due)) {
                state = kLive + 2;
                walk = false;
            }
            bool called = false;
            if (kPark) {
                CellFrame CF{};
                float ltc = 0.0f, ldep = 0.0f;
                called = walk && call_eligible(P, k0c, fx, fy, fz, xc, CF, ltc, ldep);
                walk = walk && !called;
            }
            if (walk) scatter(xc, tl.m, db, 1);
            if (kPark) {
                const bool cont = walk && ++seg >= P.park_budget;
                park(called || cont, walk, xc, called ? 1u : 0u);
            }
            if (walk) next_event([&]() __attribute__((always_inline)) { fresh = true; at += 4 * k; });
            if (__ballot(have & (state != kLive)) != 0ull) {
                settle();
                unit = state == kLive ? 1u : 0u;
                if (__ballot(state == kLive) == 0ull) break;
            }
        }
    }

    if (kEsc) {
        wave_add_counter(P.counters + KRT_C_EMIS_DROP, c_drop);
        wave_add_counter(P.counters + KRT_C_MLP_I, c_mlp);
        wave_add_counter(P.counters + KRT_C_SKIPPED_I, c_skip);
    }
    __syncthreads();
    if (threadIdx.x < kNLdsCounters && lcnt[threadIdx.x] != 0ull) {
        constexpr int slot[kNLdsCounters] = {KRT_C_ESCAPED, KRT_C_DESTROYED, KRT_C_STUCK, KRT_C_EMITTED,
                                             KRT_C_SCATTER, KRT_C_CROSS, KRT_C_EMIS_DROP};
        int to = slot[0];
#pragma unroll
        for (int i = 1; i < kNLdsCounters; ++i) to = (int)threadIdx.x == i ? slot[i] : to;
        atomicAdd(reinterpret_cast<unsigned long long *>(P.counters + to), lcnt[threadIdx.x]);
    }
}

// -------------------------------------------------------------- finalise ---
// One pass over a raw tally after the transport: sets the saturation bit if a
// sum left [0, 2^62] (the transport's atomics return nothing), and with kOut
// writes its FP32 form (FP64 scaling).  A stream bound by memory, so the check
// and the scaling share one read.  kStream: past the 256 MB last-level cache
// the accesses are marked as not to be kept.  128^3 x 64 sums, 1.6 GB: check and
// scaling apart 237 + 264 us, together 267, streaming 244 (6.6 TB/s; 16 bytes a
// lane 257 to 324 with the launch's shape).
template <bool kOut, bool kStream>
__global__ void __launch_bounds__(256) finish_kernel(const int64_t *raw, float *out, int64_t n, double scale,
                                                     uint32_t *status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int64_t v = kStream ? __builtin_nontemporal_load(raw + i) : raw[i];
        bad |= (v < 0) | (v > (int64_t(1) << 62));
        if constexpr (kOut) {
            const float o = (float)((double)v * scale);
            if (kStream) __builtin_nontemporal_store(o, out + i);
            else out[i] = o;
        }
    }
    if (__ballot(bad) != 0ull && __lane_id() == 0) atomicOr(status, (uint32_t)KRT_ST_SATURATE_BIT);
}

// One record per cell of the fields a packet needs on entering it: (k0, v) and,
// with quads = 2, (eps, kabs, 0, 0).
__global__ void pack_fields_kernel(const float *k0, const float *vx, const float *vy, const float *vz, const float *eps,
                                   const float *kabs, float4 *rec, int quads, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        rec[i * quads] = make_float4(k0[i], vx ? vx[i] : 0.0f, vx ? vy[i] : 0.0f, vx ? vz[i] : 0.0f);
        if (quads == 2) rec[2 * i + 1] = make_float4(eps ? eps[i] : 0.0f, kabs ? kabs[i] : 0.0f, 0.0f, 0.0f);
    }
}

__global__ void zero_i64_kernel(int64_t *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0;
}

// ----------------------------------------------------------- diagnostics ---
__global__ void debug_philox_kernel(const uint32_t *ctr, const uint32_t *key, uint32_t *out, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint4 c = make_uint4(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]);
    uint4 r = philox(c, key[2 * i], key[2 * i + 1]);
    out[4 * i] = r.x; out[4 * i + 1] = r.y; out[4 * i + 2] = r.z; out[4 * i + 3] = r.w;
}

__global__ void debug_bins_kernel(const float *x, int64_t n, int nb, const float *edges, float inv_w,
                                  int32_t *out) {
    __shared__ float e[kMaxSpecBins + 1];
    for (int i = threadIdx.x; i <= nb; i += blockDim.x) e[i] = edges[i];
    __syncthreads();
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = bin_index(x[i], e, nb, inv_w);
}

// H(a / r, |x|) for the widths r[i] as the continuum transport evaluates it
__global__ void debug_voigt_cont_kernel(RunParams P, float a, const float *r, const float *x, int64_t n, float *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const ContCell cc = cont_cell(P, a, r[i]);
    out[i] = cont_voigt(P, cc.voff, cc.tv, fabsf(x[i]));
}

__global__ void debug_voigt_kernel(const float *tab, const float *x, int64_t n, float *out) {
    extern __shared__ float4 lds4[];
    float *T = reinterpret_cast<float *>(lds4);
    const float4 *src = reinterpret_cast<const float4 *>(tab);
    for (int i = threadIdx.x; i < kTabFloats / 4; i += blockDim.x) lds4[i] = src[i];
    __syncthreads();
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = voigt_lds(T, fabsf(x[i]));
}

__global__ void debug_voigt_analytic_kernel(float a, float u0, const float *x, int64_t n, float *out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = voigt_analytic(a, u0, fabsf(x[i]));
}

__global__ void debug_upar_kernel(const float *tab, float a, float thd, float x, uint32_t k0, uint32_t k1,
                                  uint64_t packet, uint32_t ev0, int64_t n, float *out) {
    extern __shared__ float4 lds4[];
    float *T = reinterpret_cast<float *>(lds4);
    const float4 *src = reinterpret_cast<const float4 *>(tab);
    for (int i = threadIdx.x; i < kTabFloats / 4; i += blockDim.x) lds4[i] = src[i];
    __syncthreads();
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint4 A = philox(make_uint4(ev0 + (uint32_t)i, (uint32_t)packet, (uint32_t)(packet >> 32), 0u), k0, k1);
    out[i] = upar_lds(T, x + 0.0f, a, thd, u01(A.z), u01(A.w));  // -0 as 0, as a walk's sources give it
}

// ---------------------------------------------------------------- launch ---
// dynamic LDS of a transport launch: at most the tables, the edges and the
// dipole windows of 1024 threads, or the tables and the network image
constexpr int kPlainLds = sizeof(float) * (kTabFloats + kEdgeFloats) + sizeof(int64_t) * kNLdsCounters;
constexpr int kFusedLds =
    (int)sizeof(float) * (kTabFloats + kChanEdgeFloats) + kMlpFwdBytes + (int)sizeof(int64_t) * kNLdsCounters;
constexpr int kMaxTransportLds = std::max(kPlainLds + (int)sizeof(int64_t) * kEmisSlots * 1024, kFusedLds);
static_assert(kMaxTransportLds <= 160 * 1024, "a workgroup's LDS fits one CU (160 KiB)");
static_assert((kTabFloats + kEdgeFloats) % 4 == 0 && (kTabFloats + kChanEdgeFloats + kMlpFwdBytes / 4) % 4 == 0,
              "the counters are aligned");

// A persistent walk takes no more workgroups than are resident at once: packets
// are first given out by place, and those of a workgroup that waits for another
// to end would wait with it (64 workgroups of 1024 lanes asked for per compute
// unit, one resident, 600,000 packets of a tau0 = 500 sphere: 306 ms, 30 with the
// one).
template <int kMode, int kMaxThreads, int kProf, bool kDip, int kRec = 0>
static hipError_t launch_transport_t(RunParams P, WalkGrid g, size_t lds, hipStream_t s) {
    auto fn = mc_transport_kernel<kMode, kMaxThreads, kProf, kDip, kRec>;
    static std::atomic<bool> attr_set{false};  // the most any launch of this variant asks for
    if (!attr_set.load()) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kMaxTransportLds);
        if (e != hipSuccess) return e;
        attr_set.store(true);
    }
    if (g.per_cu > 1) {
        int resident = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, fn, g.block, lds);
        if (e != hipSuccess) return e;
        g.per_cu = std::min(g.per_cu, std::max(resident, 1));
    }
    const int grid = g.cus * g.per_cu;
    P.first_lanes = first_lanes(P.n_res + P.n_packets, (uint64_t)grid * (uint64_t)(g.block / 64), (uint64_t)grid);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(g.block), lds, s, P);
    return hipGetLastError();
}

template <int kProf, int kRec = 0>
static hipError_t launch_plain(const RunParams &P, const WalkGrid &g, hipStream_t s) {
    // tables and both edge sets; with dipole phase the emissivity windows' sums
    if (P.phase == KRT_PHASE_DIPOLE_I)
        return launch_transport_t<kModePlain, 1024, kProf, true, kRec>(
            P, g, kPlainLds + (P.emis_raw ? sizeof(int64_t) * kEmisSlots * (size_t)g.block : 0), s);
    return launch_transport_t<kModePlain, 1024, kProf, false, kRec>(P, g, kPlainLds, s);
}

hipError_t launch_transport(const RunParams &P, int mode, const WalkGrid &g, hipStream_t s) {
    if (mode == kModeFused) {
        // compiled for the block size: up to 512 lanes 256 VGPRs (2 waves per SIMD;
        // the default), up to 768 lanes 168 VGPRs (spills, 3 waves), above that
        // 128 (4 waves, heavy spills)
        if (g.block <= 512 && P.rec) return launch_transport_t<kModeFused, 512, 0, false, 1>(P, g, kFusedLds, s);
        if (g.block <= 512) return launch_transport_t<kModeFused, 512, 0, false>(P, g, kFusedLds, s);
        if (g.block <= 768) return launch_transport_t<kModeFused, 768, 0, false>(P, g, kFusedLds, s);
        return launch_transport_t<kModeFused, 1024, 0, false>(P, g, kFusedLds, s);
    }
    if (mode == kModePark) return launch_transport_t<kModePark, 1024, 0, false>(P, g, kPlainLds, s);
    // temperature and the profile modes exist for the plain walk only
    if (P.bratio) return launch_plain<4>(P, g, s);
    if (P.tclass) return launch_plain<3>(P, g, s);
    if (P.profile_mode == 1) return launch_plain<1>(P, g, s);
    if (P.profile_mode == 2) return launch_plain<2>(P, g, s);
    return P.rec ? launch_plain<0, 2>(P, g, s) : launch_plain<0>(P, g, s);
}

// ------------------------------------------------------------ call kernel ---
// The network calls of parked packets, in place.  Every lane takes one record
// (wave-strided over the list), so each evaluation runs on full 16-sample
// blocks and no transport state is live around it.  The condition, the two
// evaluations and the applied exit are the transport's own (call_eligible,
// call_condition, call_network, call_apply); the skipped scatterings'
// emissivity goes straight to the int64 tallies.
constexpr int kCallThreads = 512;
__global__ void __launch_bounds__(kCallThreads) escape_call_kernel(RunParams P, uint4 *rec, uint64_t n) {
    extern __shared__ float4 lds4[];
    float *cedges = reinterpret_cast<float *>(lds4);
    {
        for (int i = threadIdx.x; i <= P.emis_nch; i += blockDim.x) cedges[i] = P.ch_edges[i];
        const float4 *ms = reinterpret_cast<const float4 *>(P.mlp_img);
        float4 *md = lds4 + kChanEdgeFloats / 4;
        for (int i = threadIdx.x; i < kMlpFwdBytes / 16; i += blockDim.x) md[i] = ms[i];
    }
    __syncthreads();
    const unsigned char *mimg = reinterpret_cast<const unsigned char *>(lds4 + kChanEdgeFloats / 4);
    const float *mbias = reinterpret_cast<const float *>(mimg + kTilesFwd * kTileBytes);
    const float *mnorm = mbias + kBiasFloats;
    const int lane = __lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / 64);
    int64_t c_mlp = 0, c_skip = 0, c_drop = 0;
    for (uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64) * 64; base < n;
         base += waves * 64) {  // wave-uniform
        const uint64_t i = base + (uint64_t)lane;
        const bool live = i < n;
        uint4 r0 = make_uint4(0u, 0u, 0u, 0u), r1 = r0, r2 = r0, r3 = r0;
        if (live) {
            const uint4 *r = rec + kParkQuads * i;
            r0 = r[0]; r1 = r[1]; r2 = r[2]; r3 = r[3];
        }
        const int cell = (int)r0.w;
        float fx = __uint_as_float(r1.x), fy = __uint_as_float(r1.y), fz = __uint_as_float(r1.z);
        float x = __uint_as_float(r1.w);
        float nx = __uint_as_float(r2.x), ny = __uint_as_float(r2.y), nz = __uint_as_float(r2.z);
        float k0c = 0.0f, vxc = 0.0f, vyc = 0.0f, vzc = 0.0f;
        if (live) {
            k0c = P.k0[cell];
            if (P.vx) { vxc = P.vx[cell]; vyc = P.vy[cell]; vzc = P.vz[cell]; }
        }
        // every record qualified when it was parked (the gas-frame frequency the
        // transport tested is in the record): only the frame and depths are rebuilt
        const float xc = __uint_as_float(r3.y);
        CellFrame CF{};
        float tc = 1.0f, dep = 1.0f;
        if (live) call_frame(P, k0c, fx, fy, fz, CF, tc, dep);
        const float ltc = __log10f(tc), ldep = __log10f(dep);
        const bool ask = live && r3.z == 1u;  // kind 0: parked to continue, no call
        const uint64_t am = __ballot(ask);
        if (am == 0ull) continue;
        const uint4 C = philox(make_uint4(r0.z, r0.x, r0.y, 2u), P.key0, P.key1);
        const uint4 D = philox(make_uint4(r0.z, r0.x, r0.y, 3u), P.key0, P.key1);
        float cnd[10];
        call_condition(P, CF, ltc, ldep, xc, nx, ny, nz, cnd);
        int face;
        float xo, mo[kMlpOut];
        call_network(mimg, mbias, mnorm, lane, am, cnd, C, D, face, xo, mo);
        if (ask) {
            int64_t *ebase = P.emis_raw ? P.emis_raw + (int64_t)cell * P.emis_nch : nullptr;
            call_apply(P, mnorm, cedges, CF, mo, face, xo, C.z, ltc, ldep, xc, vxc, vyc, vzc, fx, fy, fz, nx, ny, nz,
                       x, c_skip, c_drop, [&](int ch, int64_t w) __attribute__((always_inline)) { tally_add_i64(ebase + ch, w); });
            c_mlp += 1;
            uint4 *r = rec + kParkQuads * i;
            r[1] = make_uint4(__float_as_uint(fx), __float_as_uint(fy), __float_as_uint(fz), __float_as_uint(x));
            r[2] = make_uint4(__float_as_uint(nx), __float_as_uint(ny), __float_as_uint(nz), r2.w);
        }
    }
    wave_add_counter(P.counters + KRT_C_MLP_I, c_mlp);
    wave_add_counter(P.counters + KRT_C_SKIPPED_I, c_skip);
    wave_add_counter(P.counters + KRT_C_EMIS_DROP, c_drop);
}

hipError_t launch_escape_call(const RunParams &P, uint4 *rec, uint64_t n, int grid, hipStream_t s) {
    static_assert(sizeof(float) * kChanEdgeFloats + kMlpFwdBytes <= 160 * 1024, "the call kernel's LDS fits one CU");
    const size_t lds = sizeof(float) * kChanEdgeFloats + (size_t)kMlpFwdBytes;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(escape_call_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL(escape_call_kernel, dim3(grid), dim3(kCallThreads), lds, s, P, rec, n);
    return hipGetLastError();
}

hipError_t launch_finish(const int64_t *raw, float *out, int64_t n, double scale, uint32_t *status, hipStream_t s) {
    if (n <= 0 || !raw) return hipSuccess;
    const int grid = (int)std::min<int64_t>((n + 255) / 256, 65536);
    const bool stream = n > (int64_t(1) << 25);  // 256 MB of sums
    auto fn = out ? (stream ? finish_kernel<true, true> : finish_kernel<true, false>)
                  : (stream ? finish_kernel<false, true> : finish_kernel<false, false>);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, s, raw, out, n, scale, status);
    return hipGetLastError();
}

hipError_t launch_pack_fields(const RunParams &P, float4 *rec, int quads, hipStream_t s) {
    const int grid = (int)std::min<int64_t>(((int64_t)P.ncell + 255) / 256, 16384);
    hipLaunchKernelGGL(pack_fields_kernel, dim3(grid), dim3(256), 0, s, P.k0, P.vx, P.vy, P.vz, P.eps, P.kabs, rec,
                       quads, (int64_t)P.ncell);
    return hipGetLastError();
}

hipError_t launch_debug_voigt_analytic(float a, float u0, const float *x, int64_t n, float *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(debug_voigt_analytic_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, u0, x, n,
                       out);
    return hipGetLastError();
}

hipError_t launch_zero_i64(int64_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int grid = (int)std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(zero_i64_kernel, dim3(grid), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_debug_philox(const uint32_t *ctr, const uint32_t *key, uint32_t *out, int64_t n, hipStream_t s) {
    int grid = (int)((n + 255) / 256);
    hipLaunchKernelGGL(debug_philox_kernel, dim3(grid), dim3(256), 0, s, ctr, key, out, n);
    return hipGetLastError();
}

hipError_t launch_debug_bins(const float *x, int64_t n, int nb, const float *edges, float inv_w, int32_t *out,
                             hipStream_t s) {
    int grid = (int)((n + 255) / 256);
    hipLaunchKernelGGL(debug_bins_kernel, dim3(grid), dim3(256), 0, s, x, n, nb, edges, inv_w, out);
    return hipGetLastError();
}

hipError_t launch_debug_voigt_cont(const RunParams &P, float a, const float *r, const float *x, int64_t n, float *out,
                                   hipStream_t s) {
    hipLaunchKernelGGL(debug_voigt_cont_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, P, a, r, x, n, out);
    return hipGetLastError();
}

hipError_t launch_debug_voigt(const float *tab, const float *x, int64_t n, float *out, hipStream_t s) {
    size_t lds = sizeof(float) * kTabFloats;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(debug_voigt_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int grid = (int)((n + 255) / 256);
    hipLaunchKernelGGL(debug_voigt_kernel, dim3(grid), dim3(256), lds, s, tab, x, n, out);
    return hipGetLastError();
}

hipError_t launch_debug_upar(const float *tab, float a, float thd, float x, uint32_t k0, uint32_t k1,
                             uint64_t packet, uint32_t ev0, int64_t n, float *out, hipStream_t s) {
    size_t lds = sizeof(float) * kTabFloats;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(debug_upar_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int grid = (int)((n + 255) / 256);
    hipLaunchKernelGGL(debug_upar_kernel, dim3(grid), dim3(256), lds, s, tab, a, thd, x, k0, k1, packet, ev0, n, out);
    return hipGetLastError();
}

}  // namespace krt
