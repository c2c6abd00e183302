// krt_escape.hip -- learned whole-cell escape: training data from single-cell
// walks run with the plain transport arithmetic, BF16-MFMA training (forward
// and backward per 32-sample chunk, weight gradients as a split-K product over
// the stored activations, Adam) and batched inference for tests.
//
// Whole-cell walk (training data): a homogeneous static cube [-1, 1]^3 (units
// of its half-width) of line-centre opacity tau_c per unit length; a photon of
// gas-frame frequency x_in >= 0 arriving along n_in scatters at a start point
// q in the reduced frame (0 <= q0 <= q1 <= q2 < 1), then takes the transport's
// flights and resonant scatterings (isotropic phase) until it leaves.  The
// record is the condition and the exit (face, offsets, cosine, alpha, x_out),
// the number of scatterings N_s and the mean x^2 over them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "krt_internal.h"
#include "krt_kernels.h"
#include "krt_mlp.h"
#include "krt_device.h"

namespace krt {

// ------------------------------------------------------------- recording ---
// Persistent pool as in the transport: records spread over the waves first,
// then each lane takes an index from one wave-aggregated atomic on `counter`
// (zeroed by the caller); one event per loop iteration, so records of very
// different lengths share waves without idling; once the pool is empty a wave
// with few walks left draws their coming events ahead with its idle lanes and
// runs an event as one straight piece of code while no walk leaves the cell.
// A launch lasts as long as its longest walk, so the chain of one event bounds
// it, and the bulk the instruction issue.  300,000 records of log10 tau_c up to
// 4: 178 ms with the walk in nested branches and 256-lane workgroups, 80 ms now.
constexpr int kRecThreads = 1024;
constexpr int kRecTailLanes = 32;
__global__ void __launch_bounds__(kRecThreads) cell_record_kernel(RecordParams R) {
#pragma clang fp contract(off)
    extern __shared__ float4 lds4[];
    float *T = reinterpret_cast<float *>(lds4);
    const float4 *src = reinterpret_cast<const float4 *>(R.tab);
    for (int i = threadIdx.x; i < kTabFloats / 4; i += blockDim.x) lds4[i] = src[i];
    __syncthreads();
    const int lane = __lane_id();
    const uint64_t lanemask_lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    constexpr int kDone = -1, kNeed = 0, kLive = 1;
    int state = kNeed;
    uint64_t idx = 0;
    PhiloxPacket pk{};
    uint4 wb = make_uint4(0u, 0u, 0u, 0u);
    uint32_t w1 = 0, w2 = 0;
    float lt = 0.f, tauc = 0.f, xin = 0.f, q0 = 0.f, q1 = 0.f, q2 = 0.f;
    float m0 = 0.f, m1 = 0.f, m2 = 1.f;
    float px = 0.f, py = 0.f, pz = 0.f, nx = 0.f, ny = 0.f, nz = 1.f, x = 0.f, sx2 = 0.f, tau = 0.f;
    uint32_t ns = 0;  // scatterings so far; the next event is ns + 1
    auto draw_event = [&]() __attribute__((always_inline)) {
        uint4 A;
        philox_pair(pk, ns + 1, R.k0, R.k1, A, wb);
        tau = -f_log(u01(A.x));
        w1 = A.z; w2 = A.w;
    };
    // one event of a walk: the flight from the last interaction point (none
    // before the first event), then the scattering unless it left the cell
    struct Flight {
        float tx, ty, tm;
        bool inside;
        UparMass m;
    };
    auto fly = [&]() __attribute__((always_inline)) {
        Flight f;
        const float xa = fabsf(x);
        const VoigtEntry e = voigt_entry(T, xa);
        f.m = upar_mass(T, e);
        const float kap = tauc * voigt_value(e, xa);
        // a zero component gives +inf or NaN, which the minimum ignores
        f.tx = fabsf(px - copysignf(1.0f, nx)) * f_rcp(fabsf(nx));
        f.ty = fabsf(py - copysignf(1.0f, ny)) * f_rcp(fabsf(ny));
        f.tm = fminf(fminf(f.tx, f.ty), fabsf(pz - copysignf(1.0f, nz)) * f_rcp(fabsf(nz)));
        const float dm = fmaxf(f.tm, 0.0f);
        const bool first = ns == 0;
        f.inside = first | !(kap * dm < tau);
        const float l = sel(f.inside, sel(first, 0.0f, tau * f_rcp(kap)), dm);
        px = fminf(fmaxf(fmaf(l, nx, px), -1.f), 1.f);
        py = fminf(fmaxf(fmaf(l, ny, py), -1.f), 1.f);
        pz = fminf(fmaxf(fmaf(l, nz, pz), -1.f), 1.f);
        return f;
    };
    auto scatter = [&](const UparMass &m, const SDraws &b) __attribute__((always_inline)) {
        const float upar = upar_from(T, m, x, R.a, R.thd, b.r1, b.r2, b.xw);
        const Basis e = scatter_basis(nx, ny, nz);
        float ox, oy, oz;
        scatter_turn(nx, ny, nz, e, b, ox, oy, oz);
        sx2 = fmaf(x, x, sx2);
        x = scatter_shift(x, upar, b);
        nx = ox; ny = oy; nz = oz;
        ns += 1;
    };
    // a walk that left the cell (or passed max_scat: stored invalid)
    auto store = [&](const Flight &f, bool exited) __attribute__((always_inline)) {
        float *o = R.out + (int64_t)kRec * idx;
        o[kRecLT] = lt;
        o[kRecLA] = __log10f(R.a);
        o[kRecX] = xin;
        o[kRecQ0] = q0; o[kRecQ0 + 1] = q1; o[kRecQ0 + 2] = q2;
        o[kRecLD] = lt + __log10f(fmaxf(1.0f - q2, 1e-30f));
        o[kRecN0] = m0; o[kRecN0 + 1] = m1; o[kRecN0 + 2] = m2;
        if (exited) {
            const bool ax0 = f.tx == f.tm, ax1 = !ax0 && f.ty == f.tm;  // ties go to the lower axis
            // the face's axis, and the two that follow it cyclically
            const float nn = by_axis(ax0, ax1, nx, ny, nz), n1 = by_axis(ax0, ax1, ny, nz, nx),
                        n2 = by_axis(ax0, ax1, nz, nx, ny);
            const float qk = by_axis(ax0, ax1, q0, q1, q2), qa = by_axis(ax0, ax1, q1, q2, q0),
                        qb = by_axis(ax0, ax1, q2, q0, q1);
            const float side = nn > 0.f ? 1.f : -1.f;
            const float dpl = fmaf(-side, qk, 1.f);
            const float ds = by_axis(ax0, ax1, py, pz, px) - qa, dt = by_axis(ax0, ax1, pz, px, py) - qb;
            o[kRecFace] = (float)(2 * by_axis(ax0, ax1, 0, 1, 2) + (side > 0.f ? 1 : 0));
            o[kRecYS] = ds / dpl;
            o[kRecYT] = dt / dpl;
            o[kRecMu] = fabsf(nn);
            o[kRecAlpha] = atan2f(fabsf(fmaf(ds, n2, -(dt * n1))), fmaf(ds, n1, dt * n2));
            o[kRecXOut] = x;
            o[kRecLogN] = logf((float)ns);
            o[kRecLogX2] = logf(fmaxf(sx2 / (float)ns, 1e-6f));
            o[kRecValid] = 1.0f;
        } else {
            for (int k = kRecFace; k <= kRecValid; ++k) o[k] = 0.0f;
        }
        o[kRec - 1] = 0.0f;
        state = kNeed;
    };
    WorkPool pool;
    pool.init(R.first_lanes);
    for (;;) {
        const uint64_t need_mask = __ballot(state == kNeed);
        if (pool.due(need_mask, __ballot(state == kLive) != 0ull)) {
            const uint64_t mine = pool.take(need_mask, lane, lanemask_lt, R.counter, R.n, R.first_lanes);
            if (state == kNeed) {
                idx = mine;
                if (idx >= R.n) {
                    state = kDone;
                } else {
                    const uint64_t pid = R.offset + idx;
                    const uint32_t plo = (uint32_t)pid, phi = (uint32_t)(pid >> 32);
                    const uint4 c = philox(make_uint4(0u, plo, phi, 3u), R.k0, R.k1);
                    const uint4 d = philox(make_uint4(0u, plo, phi, 4u), R.k0, R.k1);
                    const uint4 e = philox(make_uint4(0u, plo, phi, 5u), R.k0, R.k1);
                    lt = fmaf(R.lt_hi - R.lt_lo, u01(c.x), R.lt_lo);
                    tauc = f_exp(lt * 2.302585093f);
                    if (R.fixed) {
                        xin = R.x_in;
                        q0 = R.q[0]; q1 = R.q[1]; q2 = R.q[2];
                    } else {
                        // |x_in| from 1/2 N(0, 1/2) + 1/2 U[-3, 3]
                        if (u01(c.y) < 0.5f) xin = fabsf(f_sqrt(-f_log(u01(c.z))) * cos_rev(u01(c.w)));
                        else xin = kRecXMax * u01(c.z);
                        // depth to the nearest face log-uniform in [depth_lo, tau_c]
                        const float l0 = fminf(R.ld_lo, lt);
                        const float ld = fmaf(lt - l0, u01(e.x), l0);
                        q2 = fminf(fmaxf(1.0f - f_exp((ld - lt) * 2.302585093f), 0.0f), 0.99999f);
                        const float a0 = q2 * u01(e.y), a1 = q2 * u01(e.z);
                        q0 = fminf(a0, a1);
                        q1 = fmaxf(a0, a1);
                    }
                    if (R.fixed && !R.iso_dir) {
                        m0 = R.n_in[0]; m1 = R.n_in[1]; m2 = R.n_in[2];
                    } else {
                        const float mu0 = fmaf(2.0f, u01(d.x), -1.0f), st0 = f_sqrt(fmaxf(0.0f, fmaf(-mu0, mu0, 1.0f)));
                        const float ph0 = u01(d.y);
                        m0 = st0 * cos_rev(ph0); m1 = st0 * sin_rev(ph0); m2 = mu0;
                    }
                    px = q0; py = q1; pz = q2;
                    nx = m0; ny = m1; nz = m2;
                    x = xin + 0.0f;  // -0 as 0: the sampler takes the sign of the frequency
                    sx2 = 0.0f;
                    ns = 0;
                    state = kLive;
                    pk = philox_packet(plo, phi, R.k0, R.k1);
                    draw_event();
                }
            }
            const uint64_t live = __ballot(state == kLive);
            if (live == 0ull) break;  // the pool is empty: every lane is done
            if (__ballot(state == kDone) != 0ull && __popcll(live) <= kRecTailLanes) break;
        }
        const Flight f = fly();  // (a done lane's position is of no use to anyone)
        const bool live = state == kLive;
        bool over = false;
        if (live & f.inside) {
            SDraws b;
            scatter_draws(w1, w2, wb, false, b);
            scatter(f.m, b);
            draw_event();
            over = ns > R.max_scat;
        }
        if (live & (!f.inside | over)) store(f, !f.inside);
    }
    // ---- tail (none left: the first look ends it)
    int left = 0;        // events until the next look
    int k = 1;           // live lanes when the bank was filled
    int at = 0;          // 4 x the lane that holds this lane's draws
    bool fresh = false;  // tau of the event comes from the draws
    float pt = 0.f;
    SDraws pb{};
    for (;;) {
        if (left == 0) {
            const uint64_t live = __ballot(state == kLive);
            if (live == 0ull) break;
            k = __popcll(live);
            left = 64 / k;
            if (__ballot(state == kLive && R.max_scat - ns < 64u) != 0ull) left = 1;
            const int owner = nth_set_lane(live, lane % k);
            PhiloxPacket op;
            op.bk = __shfl(pk.bk, owner, 64);
            op.hk = __shfl(pk.hk, owner, 64);
            op.la = __shfl(pk.la, owner, 64);
            const uint32_t e = __shfl(ns, owner, 64) + 1u + (uint32_t)(lane / k);
            uint4 A, B;
            philox_pair(op, e, R.k0, R.k1, A, B);
            pt = -f_log(u01(A.x));
            scatter_draws(A.z, A.w, B, false, pb);
            at = 4 * __popcll(live & lanemask_lt);
        }
        --left;
        auto fetch = [&](float v) __attribute__((always_inline)) {
            return __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(v)));
        };
        const float dt = fetch(pt);
        SDraws db;
        db.up1 = db.up2 = 0.0f;
        db.r1 = fetch(pb.r1); db.r2 = fetch(pb.r2); db.xw = fetch(pb.xw);
        db.g = fetch(pb.g); db.sg = fetch(pb.sg);
        db.cp = fetch(pb.cp); db.sp = fetch(pb.sp);
        db.kick = fetch(pb.kick);
        tau = sel(fresh, dt, tau);
        const Flight f = fly();
        const bool live = state == kLive;
        if (__ballot(live & !f.inside) == 0ull && left != 0) {
            scatter(f.m, db);
            fresh = true;
            at += 4 * k;
            continue;
        }
        bool over = false;
        if (live & f.inside) {
            scatter(f.m, db);
            at += 4 * k;
            over = ns > R.max_scat;
        }
        fresh = true;
        if (live & (!f.inside | over)) store(f, !f.inside);
    }
}

// ---------------------------------------------------------- parameters ---
// He-uniform initialisation from Philox (counter = (param index, 0, 0, 7))
__global__ void mlp_init_kernel(float *p, uint32_t k0, uint32_t k1) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    uint4 r = philox(make_uint4((uint32_t)i, 0u, 0u, 7u), k0, k1);
    float u = 2.0f * u01(r.x) - 1.0f;
    float fan_in = 0.0f;
    bool bias = false;
    if (i < kPB1) fan_in = kMlpIn;
    else if (i < kPW2) bias = true;
    else if (i < kPB2) fan_in = kMlpHid;
    else if (i < kPW3) bias = true;
    else if (i < kPB3) fan_in = kMlpHid;
    else if (i < kPW4) bias = true;
    else if (i < kPB4) fan_in = kMlpHid;
    else bias = true;
    p[i] = bias ? 0.0f : u * sqrtf(6.0f / fan_in);
}

// Operand slot 8g + j (lane group g, entry j) of feature f of a 32-wide chunk.
__device__ __forceinline__ int slot_of(int f) { return f < 16 ? 8 * (f >> 2) + (f & 3) : 8 * ((f - 16) >> 2) + 4 + (f & 3); }

// Parameter i's value into every place the packed blob holds it: a weight's
// bfloat16 slot in its forward tile and (layers 2-4) in its backward tile, a
// quantile level's weight of layer 1 also in the slot of that level's
// residual, a bias in FP32 behind the tiles.
__device__ __forceinline__ void pack_param(unsigned char *blob, int i, float v) {
    uint16_t *tiles = reinterpret_cast<uint16_t *>(blob);
    float *bias = reinterpret_cast<float *>(blob + kTilesAll * kTileBytes);
    auto put = [&](int tile, int row, int slot) {
        tiles[tile * (kTileBytes / 2) + (16 * (slot >> 3) + row) * 8 + (slot & 7)] = f2bf(v);
    };
    if (i < kPB1) {
        const int in = i / kMlpHid, out = i % kMlpHid;
        put(kTileFwdL1 + out / 16, out % 16, in);
        if (in >= kMlpLevelIn && in < kMlpLevelIn + kMlpOperandIn - kMlpResIn)
            put(kTileFwdL1 + out / 16, out % 16, kMlpResIn + in - kMlpLevelIn);
    } else if (i < kPW2) {
        bias[i - kPB1] = v;
    } else if (i < kPB3) {  // layers 2 and 3
        const bool l3 = i >= kPW3;
        const int k = i - (l3 ? kPW3 : kPW2);
        if (k >= kMlpHid * kMlpHid) {
            bias[(l3 ? 2 : 1) * kMlpHid + k - kMlpHid * kMlpHid] = v;
        } else {
            const int in = k / kMlpHid, out = k % kMlpHid;
            put((l3 ? kTileFwdL3 : kTileFwdL2) + (out / 16) * 4 + in / 32, out % 16, slot_of(in % 32));
            put((l3 ? kTileBwdL3 : kTileBwdL2) + (in / 16) * 4 + out / 32, in % 16, slot_of(out % 32));
        }
    } else if (i < kPW4) {
        bias[2 * kMlpHid + i - kPB3] = v;
    } else if (i < kPB4) {
        const int in = (i - kPW4) / kMlpOut, out = (i - kPW4) % kMlpOut;
        put(kTileFwdL4 + 4 * (out / 16) + in / 32, out % 16, slot_of(in % 32));
        put(kTileBwdL4 + in / 16, in % 16, slot_of(out));
    } else {
        bias[3 * kMlpHid + i - kPB4] = v;
    }
}

// The whole blob from the FP32 master parameters: the parameters, the unused
// operand slots of layer 1 (28-31, zero) and the normalisation.
__global__ void mlp_pack_kernel(const float *p, const float *norm, unsigned char *blob) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kNParams) pack_param(blob, i, p[i]);
    if (i < kMlpHid)
        *reinterpret_cast<uint2 *>(blob + (kTileFwdL1 + i / 16) * kTileBytes + (48 + i % 16) * 16 + 8) = make_uint2(0u, 0u);
    if (i < kNNorm) reinterpret_cast<float *>(blob + kTilesAll * kTileBytes)[kBiasFloats + i] = norm[i];
}

// Copy of the forward part (tiles + biases + norm) into one contiguous image,
// the layout staged into LDS by the transport kernel.
__global__ void mlp_fwd_image_kernel(const unsigned char *blob, unsigned char *img) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int tiles_b = kTilesFwd * kTileBytes;
    const int tail_b = (kBiasFloats + kNNorm) * 4;
    if (i < tiles_b) img[i] = blob[i];
    else if (i < tiles_b + tail_b) img[i] = blob[kTilesAll * kTileBytes + (i - tiles_b)];
}

// Regression target of output k on record r, in the output's own variable
// (|x_out| only for the record's exit face, asinh of the offsets, the cosine
// squared); false where the output has none (faces, side, unused outputs,
// another face's |x_out|).
__device__ __forceinline__ bool target_value(const float *r, int k, float &y) {
#pragma clang fp contract(off)  // the square is rounded before the mean is taken off: one rule for sums and losses
    if (k >= kOutXAbs && k < kOutXAbs + 6) {
        if ((int)r[kRecFace] != k - kOutXAbs) return false;
        y = fabsf(r[kRecXOut]);
        return true;
    }
    switch (k) {
        case kOutLogN: y = r[kRecLogN]; return true;
        case kOutLogX2: y = r[kRecLogX2]; return true;
        case kOutYS: y = asinhf(r[kRecYS]); return true;
        case kOutYT: y = asinhf(r[kRecYT]); return true;
        case kOutMu2: y = r[kRecMu] * r[kRecMu]; return true;
        case kOutAlpha: y = r[kRecAlpha]; return true;
        default: return false;
    }
}

// ----------------------------------------------------------- batch rows ---
// Training quantile levels are uniform, clamped to the encoded range [1e-4, 1 - 1e-4]
// (the pinball loss uses the clamped level too).
__device__ __forceinline__ float train_level(uint32_t w) {
    return fminf(fmaxf(u01(w), kLevelMin), 1.0f - kLevelMin);
}

// One row of a batch as the gradient pass reads it: 32 dwords, the layer-1
// operand (28 bfloat16 slots, four zero), then what the losses need.  Made
// ahead of the pass, one thread a row, so the pass starts with one contiguous
// load instead of an index, a scattered record, logarithms and inverse
// hyperbolic sines in a chain (all zero past the batch and for invalid
// records: no input and no gradient).
constexpr int kRowFlags = 16;   // 1 live, 2 conditional, 4 x_out >= 0
constexpr int kRowFace = 17;
constexpr int kRowY = 18;       // normalised targets: ln N_s, ln <x^2>, the four conditional ones, |x_out|
constexpr int kRowU = 25;       // the four quantile levels
static_assert(kRowU + 4 <= kRowDw, "a row holds its levels");

__device__ __forceinline__ void make_row(const float *r, float ua, float ub, float uc, float ud, bool cond,
                                         const float *norm, uint32_t *row) {
    uint32_t d[kRowDw] = {};
    if (r[kRecValid] > 0.5f) {
        const float xo = r[kRecXOut];
        const int face = (int)r[kRecFace];
        float in[kMlpIn];
        mlp_inputs(r, ua, ub, uc, ud, cond, xo, face, in);
        pack_inputs(in, d);
        d[kRowFlags] = 1u | (cond ? 2u : 0u) | (xo >= 0.0f ? 4u : 0u);
        d[kRowFace] = (uint32_t)face;
        auto target = [&](int slot, int k) {
            float raw = 0.0f;
            (void)target_value(r, k, raw);
            d[kRowY + slot] = __float_as_uint((raw - norm[k]) / norm[kMlpOut + k]);
        };
        if (cond) {
#pragma unroll
            for (int k = kOutYS; k <= kOutAlpha; ++k) target(2 + k - kOutYS, k);
        } else {
            target(0, kOutLogN);
            target(1, kOutLogX2);
            if (face >= 0 && face < 6) target(6, kOutXAbs + face);
        }
        d[kRowU] = __float_as_uint(ua);
        d[kRowU + 1] = __float_as_uint(ub);
        d[kRowU + 2] = __float_as_uint(uc);
        d[kRowU + 3] = __float_as_uint(ud);
    }
    uint4 *o = reinterpret_cast<uint4 *>(row);
#pragma unroll
    for (int k = 0; k < kRowDw / 4; ++k) o[k] = make_uint4(d[4 * k], d[4 * k + 1], d[4 * k + 2], d[4 * k + 3]);
}

// Row i of a random batch: a record uniform over the set, four quantile levels
// and the row kind (conditional with probability 1/3).
__device__ __forceinline__ void draw_row(const RowDraw &D, int i) {
    uint32_t *row = D.rows + (int64_t)kRowDw * i;
    if (i >= D.batch) {
        for (int k = 0; k < kRowDw; ++k) row[k] = 0u;
        return;
    }
    const uint4 r = philox(make_uint4(D.step, (uint32_t)i, 0u, 9u), D.k0, D.k1);
    const uint4 e = philox(make_uint4(D.step, (uint32_t)i, 1u, 9u), D.k0, D.k1);
    const int32_t idx = (int32_t)__umulhi(r.x, (uint32_t)D.n);
    make_row(D.rec + (int64_t)kRec * idx, train_level(r.y), train_level(r.z), train_level(r.w), train_level(e.y),
             u01(e.x) < (1.0f / 3.0f), D.norm, row);
}

// Rows of a given batch: row i uses record idx[i] and uq[5 i ..] = (u_a, u_b,
// u_c, u_d, 1 for a conditional row).
__global__ void __launch_bounds__(64) mlp_rows_kernel(const float *rec, const int32_t *idx, const float *uq,
                                                      int batch, const float *norm, uint32_t *rows) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 32 * ((batch + 31) / 32)) return;
    uint32_t *row = rows + (int64_t)kRowDw * i;
    if (i >= batch) {
        for (int k = 0; k < kRowDw; ++k) row[k] = 0u;
        return;
    }
    const float *q = uq + 5 * (int64_t)i;
    make_row(rec + (int64_t)kRec * idx[i], q[0], q[1], q[2], q[3], q[4] > 0.5f, norm, row);
}

__global__ void __launch_bounds__(64) mlp_draw_kernel(RowDraw D) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 32 * ((D.batch + 31) / 32)) draw_row(D, i);
}

// ----------------------------------------------------- forward + backward ---
// Activation store of a training step: per chunk of 32 samples 52 tiles of
// 16 features x 32 samples in the operand order of the weight-gradient product
// (lane l holds feature l%16, samples 8(l/16)..8(l/16)+7): H0 2 tiles (inputs,
// row 24 = 1 for the bias), H1..H3 8 each, dZ1..dZ3 8 each, dZ4 2.
constexpr int kActH0 = 0, kActH1 = 2, kActH2 = kActH1 + 8, kActH3 = kActH2 + 8, kActZ1 = kActH3 + 8,
              kActZ2 = kActZ1 + 8, kActZ3 = kActZ2 + 8, kActZ4 = kActZ3 + 8;
static_assert(kActZ4 + 2 == kActTiles, "activation store layout");

// Forward and backward pass of one chunk of 32 samples by one workgroup of
// eight waves.  Losses (each averaged over the batch): softmax cross-entropy
// for the exit face, logistic for the side of x_out, pinball for the quantiles
// at their own levels (|x_out| of face F only on records leaving through F),
// log-deviance for ln N_s.  Marginal rows train outputs 0-8 and 16-21,
// conditional rows 9-12.
//
// A batch of 8192 is 256 chunks, one workgroup per compute unit and two waves
// per SIMD: the chain of layers bounds it, so the chain is cut short.  Wave w
// owns row tile w of every layer for both 16-sample blocks (two products per
// weight tile) and passes its activations to the others through LDS as the
// next layer's operand: accumulators of tiles 2c, 2c + 1 side by side are
// operand chunk c.  Weight tiles are asked for two layers before their
// products (asked for all at once, the compute unit's 280 KB of loads held up
// the first layer's: it ended after 3.2 of 6.8 us).  Each hidden product is
// taken a second time with its operands exchanged: the same sums, with lane l
// holding feature l%16 of four consecutive samples, the weight-gradient
// product's order, for eight more matrix instructions a layer and wave instead
// of a transpose through LDS and 2-byte stores.  The activations are written
// through the L2 (agent scope), so the launch does not end with the write-back
// of 13.6 MB: 11.9 us and 6.6 us for the product that reads them, against 14.2
// and 6.7 with plain stores and 12.3 and 9.0 with nontemporal ones, which the
// memory-side cache does not keep.  8192 samples: 28 us before (16 samples a
// wave, rows of the store written 2 bytes at a time), 11.9 us now.
//
// kPair, for more chunks than compute units: tiles are asked for one layer
// ahead only, so that two workgroups share a compute unit (128 registers) and
// one's chain covers the other's waits.  A step of 8704 samples 25.7 us without
// / 24.6 with, 16384: 36.3 / 31.4, 100000: 128 / 112; up to a workgroup per unit
// there is nothing to cover (8192: 19.2 / 19.4).
template <bool kPair>
__global__ void __launch_bounds__(512, kPair ? 4 : 2) mlp_fwdbwd_kernel(const unsigned char *blob, const uint32_t *rows, int batch,
                                                         unsigned char *act, float *loss) {
    __shared__ __align__(16) v4i16 ex[2][4][2][64][2];  // operand chunks between layers, double-buffered
    __shared__ __align__(16) uint16_t tr[32][40];       // 32 features x 32 samples, turned (inputs, then dZ4)
    __shared__ __align__(16) v4i16 dos[2][64][2];       // dZ4 as the output layer's operand
    __shared__ float lsums[4];
    const int lane = __lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int s = lane % 16, g = lane / 16;
    const float *bias = reinterpret_cast<const float *>(blob + kTilesAll * kTileBytes);
    const float *norm = bias + kBiasFloats;
    const uint32_t *crow = rows + (int64_t)kRowDw * 32 * blockIdx.x;
    unsigned char *ca = act + (int64_t)blockIdx.x * (kActTiles * kTileBytes);
    const int ot = w & 1, ob = (w >> 1) & 1;  // output tile and block of waves 0-3

    v8i16 x[4][2];  // operand chunks x blocks
#pragma unroll
    for (int b = 0; b < 2; ++b) x[0][b] = *reinterpret_cast<const v8i16 *>(crow + kRowDw * (16 * b + s) + 4 * g);
    const v8i16 xt = *reinterpret_cast<const v8i16 *>(crow + kRowDw * (16 * (w & 1) + s) + 4 * g);
    v4f32 bs[3];
    float bt[3];
    auto biases = [&](int l) {
        bs[l] = ld4(bias + l * kMlpHid + 16 * w + 4 * g);
        bt[l] = bias[l * kMlpHid + 16 * w + s];
    };
    v8i16 w1 = tileA(blob, kTileFwdL1 + w, lane), w2[4], w3[4], w4[4], v4, v3[4], v2[4];
    auto tiles = [&](v8i16(&wt)[4], int tile) {
#pragma unroll
        for (int c = 0; c < 4; ++c) wt[c] = tileA(blob, tile + c, lane);
    };
    biases(0);
    __builtin_amdgcn_sched_barrier(0);
    tiles(w2, kTileFwdL2 + 4 * w);
    biases(1);
    __builtin_amdgcn_sched_barrier(0);
    auto third = [&]() {
        tiles(w3, kTileFwdL3 + 4 * w);
        biases(2);
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (!kPair) third();

    // the inputs' tiles of the store, turned by waves 0 and 1
    if (w < 2) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            tr[8 * g + j][16 * w + s] = g < 3 ? (uint16_t)xt[j] : (uint16_t)(j == 0 ? 0x3F80 : 0);
    }
    auto put_turned = [&](int tile) {
        *reinterpret_cast<v8i16 *>(ca + tile * kTileBytes + lane * 16) =
            *reinterpret_cast<const v8i16 *>(&tr[16 * w + s][8 * g]);
    };
    // four samples 4g.. of block b of feature s: half of a lane's 16 bytes
    unsigned char *cq = ca + ((g >> 1) * 16 + s) * 16 + (g & 1) * 8;
    auto put_quad = [&](int tile, int b, v4i16 v) {
        __hip_atomic_store(reinterpret_cast<uint64_t *>(cq + tile * kTileBytes + b * 512), __builtin_bit_cast(uint64_t, v),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto swap_ops = [&](int buf, v4i16 h0, v4i16 h1) {  // this wave's half chunks out, all chunks in
        ex[buf][w >> 1][0][lane][w & 1] = h0;
        ex[buf][w >> 1][1][lane][w & 1] = h1;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int k = 0; k < 2; ++k) x[c][k] = *reinterpret_cast<const v8i16 *>(&ex[buf][c][k][lane][0]);
    };
    auto act4 = [](const v4f32 &z) { return pack4(leaky(z.x), leaky(z.y), leaky(z.z), leaky(z.w)); };
    auto signs = [](const v4f32 &z) {
        return (z.x > 0.0f ? 1u : 0u) | (z.y > 0.0f ? 2u : 0u) | (z.z > 0.0f ? 4u : 0u) | (z.w > 0.0f ? 8u : 0u);
    };
    // signs of the pre-activations, all the backward pass needs of them: bit
    // 4 b + r in the operand order, 16 + 4 b + r turned
    uint32_t pos[3] = {0u, 0u, 0u};
    v4f32 acc[2], at[2];
    auto layer_out = [&](int l, int tile0) {
        v4i16 h[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            pos[l] |= (signs(acc[b]) | (signs(at[b]) << 16)) << (4 * b);
            h[b] = act4(acc[b]);
        }
        swap_ops(l & 1, h[0], h[1]);
#pragma unroll
        for (int b = 0; b < 2; ++b) put_quad(tile0 + w, b, act4(at[b]));
    };
    auto start = [&](int l) {
        acc[0] = acc[1] = bs[l];
        at[0] = at[1] = (v4f32){bt[l], bt[l], bt[l], bt[l]};
    };
    auto product = [&](const v8i16 &wt, int c) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            acc[b] = mfma32(wt, x[c][b], acc[b]);
            at[b] = mfma32(x[c][b], wt, at[b]);
        }
    };
    auto hidden = [&](const v8i16(&wt)[4], int l) {
        start(l);
#pragma unroll
        for (int c = 0; c < 4; ++c) product(wt[c], c);
    };
    start(0);
    product(w1, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kPair) third();
    layer_out(0, kActH1);
    if (w < 2) put_turned(kActH0 + w);
    if constexpr (kPair) {
        hidden(w2, 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    tiles(w4, kTileFwdL4 + 4 * ot);
    const v4f32 bo = ld4(bias + 3 * kMlpHid + 16 * ot + 4 * g);
    // this lane's row of the losses
    const uint4 *tq = reinterpret_cast<const uint4 *>(crow + kRowDw * (16 * ob + s) + kRowFlags);
    const uint4 q0 = tq[0], q1 = tq[1], q2 = tq[2], q3 = tq[3];
    const float scn = norm[kMlpOut + kOutLogN];
    v4 = tileA(blob, kTileBwdL4 + w, lane);
    __builtin_amdgcn_sched_barrier(0);
    auto back3 = [&]() {
        tiles(v3, kTileBwdL3 + 4 * w);
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (!kPair) {
        hidden(w2, 1);
        __builtin_amdgcn_sched_barrier(0);
        back3();
    }
    layer_out(1, kActH2);
    hidden(w3, 2);
    __builtin_amdgcn_sched_barrier(0);
    auto back2 = [&]() {
        tiles(v2, kTileBwdL2 + 4 * w);
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (kPair) back3();
    else back2();
    layer_out(2, kActH3);
    // gradients of outputs 16 ot + 4g + j of sample s of block ob, the choice of
    // formula by selects: a branch per lane group would run them one after the other
    static_assert(kOutSide == 6 && kOutLogN == 7 && kOutLogX2 == 8 && kOutYS == 9 && kOutYT == 10 && kOutMu2 == 11 &&
                      kOutAlpha == 12 && kOutXAbs == 16, "outputs by lane group");
    const float invB = 1.0f / (float)batch;
    const bool live = q0.x & 1u, cond = q0.x & 2u;
    const float side = (q0.x & 4u) ? 1.0f : 0.0f;
    const int face = (int)q0.y;
    const float ua = __uint_as_float(q2.y), ub = __uint_as_float(q2.z), uc = __uint_as_float(q2.w),
                ud = __uint_as_float(q3.x);
    const float ylog = __uint_as_float(q0.z);
    v4f32 o = bo;
    float yq[4] = {}, uq[4] = {ua, ua, ua, ua}, mx = 0.0f, se = 1.0f, flf = 0.0f;
    bool pin[4] = {};
    if (w < 4) {  // the outputs
#pragma unroll
        for (int c = 0; c < 4; ++c)
            o = mfma32(w4[c], *reinterpret_cast<const v8i16 *>(&ex[0][c][ob][lane][0]), o);
        const float ov[4] = {o.x, o.y, o.z, o.w};
        float dO[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (ot == 0) {  // wave-uniform
            // the six face logits of this lane's sample (lanes s and s + 16)
            float fl[6];
            fl[0] = __shfl(o.x, s, 64); fl[1] = __shfl(o.y, s, 64); fl[2] = __shfl(o.z, s, 64); fl[3] = __shfl(o.w, s, 64);
            fl[4] = __shfl(o.x, s + 16, 64); fl[5] = __shfl(o.y, s + 16, 64);
            mx = fl[0];
#pragma unroll
            for (int f = 1; f < 6; ++f) mx = fmaxf(mx, fl[f]);
            float sm[6];
            se = 0.0f;
#pragma unroll
            for (int f = 0; f < 6; ++f) { sm[f] = __expf(fl[f] - mx); se += sm[f]; }
            const float ise = 1.0f / se;
#pragma unroll
            for (int f = 0; f < 6; ++f) flf = sel(f == face, fl[f], flf);
            float soft[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float smk = j < 2 ? sel(g == 0, sm[j], sm[4 + (j & 1)]) : sm[j];
                soft[j] = (smk * ise - (4 * g + j == face ? 1.0f : 0.0f)) * invB;
            }
            const float dside = (sigmoid_f(o.z) - side) * invB;
            // weighted, scaled log-deviance w f(d) / s, d = s (y - o), f(d) = e^d - 1 - d,
            // continued linearly beyond d = kDevClamp
            const float ed = __expf(fminf(scn * (ylog - o.w), kDevClamp));
            const float dlog = kDevWeight * (1.0f - ed) * invB;
            const bool m = live && !cond, c = live && cond;
            dO[0] = sel(m && g < 2, soft[0], 0.0f);
            dO[1] = sel(m && g < 2, soft[1], 0.0f);
            dO[2] = sel(m && g < 2, sel(g == 0, soft[2], dside), 0.0f);
            dO[3] = sel(m && g < 2, sel(g == 0, soft[3], dlog), 0.0f);
            yq[0] = sel(cond, __uint_as_float(q1.w), __uint_as_float(q0.w));
            uq[0] = sel(cond, ud, ub);
            pin[0] = (m && g == 2) || (c && g == 3);
            yq[1] = __uint_as_float(q1.x);
            yq[2] = __uint_as_float(q1.y);
            uq[2] = ub;
            yq[3] = __uint_as_float(q1.z);
            uq[3] = uc;
            pin[1] = pin[2] = pin[3] = c && g == 2;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                yq[j] = __uint_as_float(q2.x);
                pin[j] = live && !cond && 4 * g + j < 6 && 4 * g + j == face;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) dO[j] = sel(pin[j], (((yq[j] < ov[j]) ? 1.0f : 0.0f) - uq[j]) * invB, dO[j]);
        dos[ob][lane][ot] = pack4(dO[0], dO[1], dO[2], dO[3]);
#pragma unroll
        for (int j = 0; j < 4; ++j) tr[16 * ot + 4 * g + j][16 * ob + s] = f2bf(dO[j]);
    }
    __syncthreads();
    if (w < 2) put_turned(kActZ4 + w);

    // ---- backward through the layers (dZ4 = dO): slots 8g + j of the output
    // layer's operand hold outputs 4g + j and 16 + 4g + j
    const v4f32 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 2; ++b) x[0][b] = *reinterpret_cast<const v8i16 *>(&dos[b][lane][0]);
    // times the leaky ReLU's derivative, by the pre-activation's sign
    auto slope = [](const v4f32 &z, uint32_t m) {
        return pack4(z.x * ((m & 1u) ? 1.0f : kLeak), z.y * ((m & 2u) ? 1.0f : kLeak), z.z * ((m & 4u) ? 1.0f : kLeak),
                     z.w * ((m & 8u) ? 1.0f : kLeak));
    };
    auto grad_store = [&](int l, int tile0) {
#pragma unroll
        for (int b = 0; b < 2; ++b) put_quad(tile0 + w, b, slope(at[b], pos[l] >> (16 + 4 * b)));
    };
    auto grad_ops = [&](int l, int buf) { swap_ops(buf, slope(acc[0], pos[l]), slope(acc[1], pos[l] >> 4)); };
    acc[0] = acc[1] = at[0] = at[1] = zero;
    product(v4, 0);
    if constexpr (kPair) back2();
    grad_ops(2, 1);
    grad_store(2, kActZ3);
    // layer 3 -> dZ2, layer 2 -> dZ1
    acc[0] = acc[1] = at[0] = at[1] = zero;
#pragma unroll
    for (int c = 0; c < 4; ++c) product(v3[c], c);
    grad_ops(1, 0);
    grad_store(1, kActZ2);
    at[0] = at[1] = zero;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b) at[b] = mfma32(x[c][b], v2[c], at[b]);
    grad_store(0, kActZ1);

    // the loss itself, while the stores drain
    if (!loss) return;
    if (w < 4) {
        const float ov[4] = {o.x, o.y, o.z, o.w};
        float lsum = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (pin[j]) lsum += (yq[j] - ov[j]) * (uq[j] - ((yq[j] < ov[j]) ? 1.0f : 0.0f));
        if (ot == 0 && live && !cond) {
            if (g == 0) {
                lsum += mx + __logf(se) - flf;
            } else if (g == 1) {
                lsum += fmaxf(o.z, 0.0f) + __logf(1.0f + __expf(-fabsf(o.z))) - side * o.z;
                const float d = scn * (ylog - o.w);
                const float dc = fminf(d, kDevClamp);
                lsum += kDevWeight * (__expf(dc) - 1.0f - dc + (__expf(kDevClamp) - 1.0f) * fmaxf(d - kDevClamp, 0.0f)) / scn;
            }
        }
        for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
        if (lane == 0) lsums[w] = lsum;
    }
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(loss, (lsums[0] + lsums[1] + lsums[2] + lsums[3]) * invB);
}

// Weight gradients as products over the stored activations: dW_l[in][out] =
// sum_s H_{l-1}[in][s] dZ_l[out][s], the bias from a row of ones.  One wave
// per (layer, 16-row tile, pair of 16-column tiles, sample split): the H
// operand of a chunk feeds both tiles' products.  Results go to
// part[split][param] (every parameter is written by exactly one wave per
// split, so the sum over splits in fixed order is deterministic).
//
// A batch of 8192 gives 712 waves of 32 chunks, 96 KB each, less than one wave
// per SIMD: the wait for memory bounds it.  Each tile is one contiguous 1 KB
// load, eight chunks (24 KB a wave) are on their way at any time, and a split's
// workgroups sit on one XCD (workgroups go round the eight), whose L2 then
// holds that split's eighth of the store.  8192 samples: 14.5 us before (rows
// of 2-byte columns, one chunk at a time), 6.6 us now (16 chunks on their way:
// no faster).
constexpr int kGradJobsL1 = 2 * 4, kGradJobsL2 = 9 * 4, kGradJobsL3 = 9 * 4, kGradJobsL4 = 9 * 1;
constexpr int kGradJobs = kGradJobsL1 + kGradJobsL2 + kGradJobsL3 + kGradJobsL4;   // 89
constexpr int kGradAhead = 8;

__global__ void __launch_bounds__(64) mlp_wgrad_kernel(const unsigned char *act, int nchunk, float *part,
                                                       RowDraw D) {
    const int lane = __lane_id();
    if (blockIdx.x >= kGradJobs * kGradSplits) {
        const int i = (blockIdx.x - kGradJobs * kGradSplits) * 64 + lane;
        if (i < 32 * ((D.batch + 31) / 32)) draw_row(D, i);
        return;
    }
    const int split = blockIdx.x % kGradSplits;
    int jj = blockIdx.x / kGradSplits;
    int htile, ztile, it, jp, nin, ldw, pw, pb;
    if (jj < kGradJobsL1) {
        it = jj / 4; jp = jj % 4; htile = kActH0; ztile = kActZ1; nin = kMlpIn; ldw = kMlpHid; pw = kPW1; pb = kPB1;
    } else if ((jj -= kGradJobsL1) < kGradJobsL2) {
        it = jj / 4; jp = jj % 4; htile = kActH1; ztile = kActZ2; nin = kMlpHid; ldw = kMlpHid; pw = kPW2; pb = kPB2;
    } else if ((jj -= kGradJobsL2) < kGradJobsL3) {
        it = jj / 4; jp = jj % 4; htile = kActH2; ztile = kActZ3; nin = kMlpHid; ldw = kMlpHid; pw = kPW3; pb = kPB3;
    } else {
        jj -= kGradJobsL3;
        it = jj; jp = 0; htile = kActH3; ztile = kActZ4; nin = kMlpHid; ldw = kMlpOut; pw = kPW4; pb = kPB4;
    }
    const int s = lane % 16, g = lane / 16;
    // row tile 8 of a hidden layer is the ones row alone: no load
    const bool ones = 16 * it >= kMlpHid;
    const short one = (short)(s == 0 ? 0x3F80 : 0);
    const v8i16 onesA = {one, one, one, one, one, one, one, one};
    // this split's columns: chunks of 32 samples
    const int c0 = (int)((int64_t)nchunk * split / kGradSplits), c1 = (int)((int64_t)nchunk * (split + 1) / kGradSplits);
    const unsigned char *zt = act + (ztile + 2 * jp) * kTileBytes + lane * 16;
    const unsigned char *ht = ones ? zt : act + (htile + it) * kTileBytes + lane * 16;
    v8i16 a[kGradAhead], b0[kGradAhead], b1[kGradAhead];
    auto fetch = [&](int k, int c) {
        const int64_t o = (int64_t)min(c, nchunk - 1) * (kActTiles * kTileBytes);
        a[k] = *reinterpret_cast<const v8i16 *>(ht + o);
        b0[k] = *reinterpret_cast<const v8i16 *>(zt + o);
        b1[k] = *reinterpret_cast<const v8i16 *>(zt + o + kTileBytes);
    };
#pragma unroll
    for (int k = 0; k < kGradAhead; ++k) fetch(k, c0 + k);
    v4f32 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    for (int c = c0; c < c1; c += kGradAhead) {
#pragma unroll
        for (int k = 0; k < kGradAhead; ++k) {
            if (c + k < c1) {  // wave-uniform
                const v8i16 h = ones ? onesA : a[k];
                acc0 = mfma32(h, b0[k], acc0);
                acc1 = mfma32(h, b1[k], acc1);
            }
            fetch(k, c + kGradAhead + k);
        }
    }
    float *dst = part + (int64_t)split * kNParams;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const v4f32 acc = t ? acc1 : acc0;
        const float v[4] = {acc.x, acc.y, acc.z, acc.w};
        const int out = 16 * (2 * jp + t) + s;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int in = 16 * it + 4 * g + r;
            if (in < nin) dst[pw + in * ldw + out] = v[r];
            else if (in == nin) dst[pb + out] = v[r];  // the row of ones: bias gradient
        }
    }
}

// sum of the split partial gradients (fixed order)
__global__ void mlp_gsum_kernel(const float *part, float *grad) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    float gsum = 0.0f;
    for (int sp = 0; sp < kGradSplits; ++sp) gsum += part[(int64_t)sp * kNParams + i];
    grad[i] = gsum;
}

// Adam (FP32 master, bias-corrected) on the summed split gradients; the new
// value goes straight to its places in the packed blob (a launch of 4 us saved).
constexpr int kAdamThreads = 128;
__global__ void __launch_bounds__(kAdamThreads) mlp_adam_kernel(float *p, float *m, float *v, const float *part,
                                                                float lr, float b1, float b2, float eps, float c1,
                                                                float c2, unsigned char *blob) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    float gi = 0.0f;
#pragma unroll
    for (int sp = 0; sp < kGradSplits; ++sp) gi += part[(int64_t)sp * kNParams + i];
    float mi = b1 * m[i] + (1.0f - b1) * gi;
    float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    pack_param(blob, i, pi);
}

// Normalisation of the targets: mean and standard deviation over the valid
// records of each output's own target (|x_out| of face F over the records
// leaving through F; the face and side logits and the unused outputs keep
// mean 0, scale 1), and the ranges of log10 a and log10 tau_c and the smallest
// log10 depth of the valid records (where the network may then be used).
//
// FP64 sums in a fixed order: chain t of 256 takes records t, t + 256, ...,
// and the chains are combined as a tree.  A workgroup takes four neighbouring
// chains: its threads read 512 records at a time, once for all outputs, and
// leave the targets in LDS, and its first wave carries the chains on, one lane
// per chain and target.  The next records are read meanwhile, so the additions
// bound it.  200,000 records: 562 us before (one workgroup per output reading
// every record, one load at a time), 84 us now.
constexpr int kNormChains = 256, kNormStride = 4, kNormThreads = 512, kNormRoles = 16;
constexpr int kNormSteps = kNormThreads / kNormStride;
// roles: 0-5 outputs 7-12, 6-11 |x_out| of face 0-5, 12-14 log10 a, tau_c, depth
constexpr int kNormCols = 10;  // six targets, |x_out|, log10 a, tau_c, depth
__device__ __forceinline__ int norm_role(int k) {  // role of output (or range) k, -1: none
    return (k >= kOutLogN && k <= kOutAlpha) ? k - kOutLogN
           : (k >= kOutXAbs && k < kOutXAbs + 6) ? 6 + k - kOutXAbs
           : k >= kMlpOut ? 12 + k - kMlpOut : -1;
}
static_assert(3 * kNormRoles * kNormChains * sizeof(double) <= sizeof(float) * kNParams * kGradSplits,
              "the sums fit the buffer of the split gradients");

__global__ void __launch_bounds__(kNormThreads) mlp_norm_sums_kernel(const float *rec, int64_t n, double *sums) {
    __shared__ float val[2][kNormCols][kNormThreads];
    __shared__ signed char who[2][kNormThreads];  // exit face of a valid record (7: another value), -1: no record
    const int t = threadIdx.x;
    const int chain = kNormStride * blockIdx.x + t % kNormStride;
    const int64_t batches = (n + (int64_t)kNormChains * kNormSteps - 1) / ((int64_t)kNormChains * kNormSteps);
    float v[12];
    auto read = [&](int64_t b) {
        const int64_t i = (b * kNormSteps + t / kNormStride) * kNormChains + chain;
        const float *r = rec + kRec * (i < n ? i : 0);
        const int cols[12] = {kRecValid, kRecFace, kRecLogN, kRecLogX2, kRecYS, kRecYT,
                              kRecMu, kRecAlpha, kRecXOut, kRecLA, kRecLT, kRecLD};
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = r[cols[k]];
        if (i >= n) v[0] = 0.0f;
    };
    auto leave = [&](int buf) {
        const int f = (int)v[1];
        who[buf][t] = v[0] < 0.5f ? (signed char)-1 : (signed char)((f >= 0 && f < 6) ? f : 7);
        val[buf][0][t] = v[2];
        val[buf][1][t] = v[3];
        val[buf][2][t] = asinhf(v[4]);
        val[buf][3][t] = asinhf(v[5]);
        val[buf][4][t] = v[6] * v[6];
        val[buf][5][t] = v[7];
        val[buf][6][t] = fabsf(v[8]);
        val[buf][7][t] = v[9];
        val[buf][8][t] = v[10];
        val[buf][9][t] = v[11];
    };
    // wave 0: lane = 4 role + chain
    const int role = t / kNormStride;
    const int col = role < 6 ? role : (role < 12 ? 6 : min(role - 5, kNormCols - 1));
    double a = 0.0, q = 0.0, c = 0.0;
    float lo = 1e30f, hi = -1e30f;
    read(0);
    for (int64_t b = 0; b < batches; ++b) {
        const int buf = (int)(b & 1);
        leave(buf);
        __syncthreads();
        if (b + 1 < batches) read(b + 1);
        if (t < 64) {
#pragma unroll 8
            for (int j = 0; j < kNormSteps; ++j) {
                const int e = kNormStride * j + t % kNormStride;
                const float yf = val[buf][col][e];
                const int f = who[buf][e];
                const bool in = f >= 0 && (role < 6 || role >= 12 || f == role - 6);
                const double y = yf;
                a = in ? a + y : a;
                q = in ? q + y * y : q;
                c = in ? c + 1.0 : c;
                lo = in ? fminf(lo, yf) : lo;
                hi = in ? fmaxf(hi, yf) : hi;
            }
        }
    }
    if (t < 64) {
        double *o = sums + (int64_t)role * kNormChains + chain;
        const bool range = role >= 12;
        o[0] = range ? (double)lo : a;
        o[kNormRoles * kNormChains] = range ? (double)hi : q;
        o[2 * kNormRoles * kNormChains] = c;
    }
}

// The chains' tree and the normalisation of output k (one workgroup of 256
// threads per output, three more for the ranges).
__global__ void __launch_bounds__(kNormChains) mlp_norm_kernel(const double *sums, float *norm) {
    __shared__ double s0[kNormChains], s1[kNormChains], s2[kNormChains];
    const int k = blockIdx.x, t = threadIdx.x, role = norm_role(k);
    const bool range = k >= kMlpOut;
    if (role < 0) {  // no target
        if (t == 0) {
            norm[k] = 0.0f;
            norm[kMlpOut + k] = 1.0f;
        }
        return;
    }
    s1[t] = sums[role * kNormChains + t];
    s2[t] = sums[(kNormRoles + role) * kNormChains + t];
    s0[t] = sums[(2 * kNormRoles + role) * kNormChains + t];
    __syncthreads();
    for (int st = kNormChains / 2; st >= 1; st >>= 1) {
        if (t < st) {
            s1[t] = range ? fmin(s1[t], s1[t + st]) : s1[t] + s1[t + st];
            s2[t] = range ? fmax(s2[t], s2[t + st]) : s2[t] + s2[t + st];
            s0[t] += s0[t + st];
        }
        __syncthreads();
    }
    if (t != 0) return;
    if (range) {
        const int o = kNormARange + 2 * (k - kMlpOut);
        norm[o] = (float)s1[0];
        norm[o + 1] = k < kMlpOut + 2 ? (float)s2[0] : 0.0f;  // padding after the depth minimum
    } else if (s0[0] < 1.0) {
        norm[k] = 0.0f;
        norm[kMlpOut + k] = 1.0f;
    } else {
        const double mean = s1[0] / s0[0];
        const double var = s2[0] / s0[0] - mean * mean;
        norm[k] = (float)mean;
        norm[kMlpOut + k] = (float)sqrt(var > 1e-12 ? var : 1e-12);
    }
}

// Forward for a list of raw rows in[n][kFwdRaw] = (log10 tau_c, log10 a, |x_in|,
// q0, q1, q2, log10 depth, m0, m1, m2, u_a, u_b, u_c, u_d, flag, x_out, face):
// out[n][32] normalised outputs back in their own variables (face and side
// logits as logits; ln E[N_s] with its calibration term; asinh of the offsets
// and mu^2 as learned).
__global__ void __launch_bounds__(256) mlp_forward_kernel(const unsigned char *blob, const float *inp,
                                                          int64_t n, float *out) {
    const int lane = __lane_id(), w = threadIdx.x / 64;
    const int64_t block = (int64_t)blockIdx.x * (blockDim.x / 64) + w;
    const int s = lane % 16, g = lane / 16;
    const int64_t si = block * 16 + s;
    if (block * 16 >= n) return;
    const bool live = si < n;
    const float *bias = reinterpret_cast<const float *>(blob + kTilesAll * kTileBytes);
    const float *norm = bias + kBiasFloats;
    const float *r = inp + (int64_t)kFwdRaw * (live ? si : 0);
    float in[kMlpIn];
    mlp_inputs(r, r[10], r[11], r[12], r[13], r[14] > 0.5f, r[15], (int)r[16], in);
    v4f32 o, ob;
    mlp_forward_block(blob, bias, xin_operand(in, lane), lane, o, ob);
    if (!live) return;
    const float v[8] = {o.x, o.y, o.z, o.w, ob.x, ob.y, ob.z, ob.w};
    for (int j = 0; j < 8; ++j) {
        const int k = (j < 4) ? 4 * g + j : 16 + 4 * g + (j - 4);
        out[kMlpOut * si + k] = v[j] * norm[kMlpOut + k] + norm[k] +
                                ((k == kOutLogN) ? norm[kNormCal + cal_bin(r[0], r[6], r[2])] : 0.0f);
    }
}

// Calibration sums over valid records with |x_in| <= kEscXMax (the range where
// the network is asked): per bin of (log10 tau_c, log10 depth, |x_in|), the
// number of records, sum N_s and sum exp(network ln E[N_s]) (without
// calibration), FP64.  One wave per 16-record block; block partial sums in LDS,
// then global atomics.
__global__ void __launch_bounds__(256) mlp_calib_kernel(const unsigned char *blob, const float *rec, int64_t n,
                                                        double *sums) {
    __shared__ double ls[3 * kNCal];
    for (int i = threadIdx.x; i < 3 * kNCal; i += blockDim.x) ls[i] = 0.0;
    __syncthreads();
    const int lane = __lane_id(), w = threadIdx.x / 64;
    const int64_t block = (int64_t)blockIdx.x * (blockDim.x / 64) + w;
    const int s = lane % 16, g = lane / 16;
    const int64_t si = block * 16 + s;
    if (block * 16 < n) {  // wave-uniform
        const float *r = rec + (int64_t)kRec * (si < n ? si : 0);
        const bool live = si < n && r[kRecValid] > 0.5f;
        const float *bias = reinterpret_cast<const float *>(blob + kTilesAll * kTileBytes);
        const float *norm = bias + kBiasFloats;
        // marginal row with quantile levels as the transport draws them: uniform,
        // from Philox(record index)
        const uint4 q = philox(make_uint4((uint32_t)si, (uint32_t)(si >> 32), 0u, 9u), 0x6C1Bu, 0x5EEDu);
        float in[kMlpIn];
        mlp_inputs(r, u01(q.x), u01(q.y), u01(q.z), u01(q.w), false, 0.0f, 0, in);
        v4f32 o, ob;
        mlp_forward_block(blob, bias, xin_operand(in, lane), lane, o, ob);
        static_assert(kOutLogN == 7, "ln E[N_s] sits in lane group 1, component 3");
        if (live && g == 1 && r[kRecX] <= kEscXMax) {
            const int b = cal_bin(r[kRecLT], r[kRecLD], r[kRecX]);
            const double pred = exp((double)(o.w * norm[kMlpOut + kOutLogN] + norm[kOutLogN]));
            atomicAdd(&ls[b], 1.0);
            atomicAdd(&ls[kNCal + b], exp((double)r[kRecLogN]));
            atomicAdd(&ls[2 * kNCal + b], pred);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * kNCal; i += blockDim.x)
        if (ls[i] != 0.0) atomicAdd(&sums[i], ls[i]);
}

// cal[b] = ln(sum N_s / sum predicted) for bins with at least 100 records, else 0
__global__ void mlp_calib_finish_kernel(const double *sums, float *norm) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= kNCal) return;
    const double cnt = sums[b], sn = sums[kNCal + b], sp = sums[2 * kNCal + b];
    norm[kNormCal + b] = (cnt >= 100.0 && sn > 0.0 && sp > 0.0) ? (float)log(sn / sp) : 0.0f;
}

// --------------------------------------------------------------- launch ---
hipError_t launch_cell_record(const RecordParams &R0, int cus, hipStream_t s) {
    const size_t lds = sizeof(float) * kTabFloats;
    static std::atomic<bool> attr{false};
    if (!attr.load()) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(cell_record_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr.store(true);
    }
    RecordParams R = R0;
    R.first_lanes = first_lanes(R.n, (uint64_t)cus * (kRecThreads / 64), (uint64_t)cus);
    hipLaunchKernelGGL(cell_record_kernel, dim3(cus), dim3(kRecThreads), lds, s, R);
    return hipGetLastError();
}

hipError_t launch_mlp_init(float *p, uint32_t k0, uint32_t k1, hipStream_t s) {
    hipLaunchKernelGGL(mlp_init_kernel, dim3((kNParams + 255) / 256), dim3(256), 0, s, p, k0, k1);
    return hipGetLastError();
}

static hipError_t launch_mlp_image(const unsigned char *blob, unsigned char *img, hipStream_t s) {
    hipLaunchKernelGGL(mlp_fwd_image_kernel, dim3((kMlpFwdBytes + 255) / 256), dim3(256), 0, s, blob, img);
    return hipGetLastError();
}

hipError_t launch_mlp_pack(const float *p, const float *norm, unsigned char *blob, unsigned char *img,
                           hipStream_t s) {
    hipLaunchKernelGGL(mlp_pack_kernel, dim3((kNParams + 255) / 256), dim3(256), 0, s, p, norm, blob);
    hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_mlp_image(blob, img, s);
}

hipError_t launch_mlp_rows(const float *rec, const int32_t *idx, const float *uq, int batch, const float *norm,
                           uint32_t *rows, hipStream_t s) {
    hipLaunchKernelGGL(mlp_rows_kernel, dim3((batch + 63) / 64), dim3(64), 0, s, rec, idx, uq, batch, norm, rows);
    return hipGetLastError();
}

hipError_t launch_mlp_draw(const RowDraw &D, hipStream_t s) {
    hipLaunchKernelGGL(mlp_draw_kernel, dim3((D.batch + 63) / 64), dim3(64), 0, s, D);
    return hipGetLastError();
}

// Gradient of the mean loss over a batch of rows into the split partials
// `part`; `next` (if any) draws the rows of the step after it.
hipError_t launch_mlp_grad(const unsigned char *blob, const uint32_t *rows, int batch, unsigned char *act, float *part,
                           float *loss, const RowDraw *next, int cus, hipStream_t s) {
    const int nchunk = (batch + 31) / 32;
    if (nchunk > cus)
        hipLaunchKernelGGL(mlp_fwdbwd_kernel<true>, dim3(nchunk), dim3(512), 0, s, blob, rows, batch, act, loss);
    else
        hipLaunchKernelGGL(mlp_fwdbwd_kernel<false>, dim3(nchunk), dim3(512), 0, s, blob, rows, batch, act, loss);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(kGradJobs * kGradSplits + (next ? (next->batch + 63) / 64 : 0)), dim3(64), 0,
                       s, act, nchunk, part, next ? *next : RowDraw{});
    return hipGetLastError();
}

hipError_t launch_mlp_gsum(const float *part, float *grad, hipStream_t s) {
    hipLaunchKernelGGL(mlp_gsum_kernel, dim3((kNParams + 255) / 256), dim3(256), 0, s, part, grad);
    return hipGetLastError();
}

// One Adam step into the master parameters and the packed blob, and (img not
// null, a training's last step) the inference image.
hipError_t launch_mlp_adam(float *p, float *m, float *v, const float *part, float lr, int step, unsigned char *blob,
                           unsigned char *img, hipStream_t s) {
    const float b1 = 0.9f, b2 = 0.999f;
    float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((kNParams + kAdamThreads - 1) / kAdamThreads), dim3(kAdamThreads), 0, s, p,
                       m, v, part, lr, b1, b2, 1e-8f, c1, c2, blob);
    hipError_t e = hipGetLastError();
    return (e != hipSuccess || !img) ? e : launch_mlp_image(blob, img, s);
}

hipError_t launch_mlp_calib(const unsigned char *blob, const float *rec, int64_t n, double *sums, float *norm,
                            hipStream_t s) {
    int64_t blocks = (n + 63) / 64;  // 4 waves of 16 records per block
    hipLaunchKernelGGL(mlp_calib_kernel, dim3((unsigned)blocks), dim3(256), 0, s, blob, rec, n, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_calib_finish_kernel, dim3((kNCal + 255) / 256), dim3(256), 0, s, sums, norm);
    return hipGetLastError();
}

hipError_t launch_mlp_norm(const float *rec, int64_t n, double *scratch, float *norm, hipStream_t s) {
    hipLaunchKernelGGL(mlp_norm_sums_kernel, dim3(kNormChains / kNormStride), dim3(kNormThreads), 0, s, rec, n, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_norm_kernel, dim3(kMlpOut + 3), dim3(kNormChains), 0, s, scratch, norm);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const unsigned char *blob, const float *inp, int64_t n, float *out, hipStream_t s) {
    int64_t nblocks = (n + 15) / 16;
    int grid = (int)((nblocks + 3) / 4);
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(grid), dim3(256), 0, s, blob, inp, n, out);
    return hipGetLastError();
}

}  // namespace krt
