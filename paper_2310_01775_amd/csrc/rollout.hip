// Relaxed block-pushing rollout and its adjoint on gfx950.
//
// Model (Sec. III-B: semi-implicit Euler with spring-based penalty contacts;
// Sec. IV-A and Appendix E: pushing from the N/E/S/W faces of block 0).
// Push phase k runs once per side s from the shared phase-start state S_k; the
// next phase starts from S_{k+1} = sum_s softmax(a_k)_s X_s(t_{k+1}).
//
// Lanes: one per (particle i, side s, block b).  The SL = 1, 2 or 4 block
// slots of a (particle, side) sub-rollout sit in one DPP quad (SL = B rounded
// up; slots b >= B are idle copies), so a lane integrates one block and reads
// the other blocks' positions (and, in the reverse, force adjoints) by
// quad_perm moves each step; the sides of a particle meet only at phase
// boundaries.  A step thus costs one block's friction and integration, B-1
// pair terms and the pusher per lane, instead of all blocks' work.
//
// The adjoint is the exact reverse of the forward arithmetic (Sec. III-B:
// gradients back-propagated through the whole trajectory), either from a full
// tape of pre-step states or by replaying checkpointed segments of <= K steps
// into a scratch buffer and reversing each.
#include "common.h"
#include "internal.h"

namespace stamp {

// One wave per workgroup: a small particle set spreads over as many CUs as it
// has waves instead of stacking four waves on one CU.
constexpr int kRolloutBlock = 64;

// Block slots per (particle, side) sub-rollout, and lanes per particle.
template <int B>
struct Slots {
    static constexpr int SL = B == 1 ? 1 : (B == 2 ? 2 : 4);
    static constexpr int LANES = 4 * SL;
};

// State of one block: position, angle, velocities.
struct Blk {
    float x, y, ph, vx, vy, om;
};

// Fixed data of one lane during one push phase.  The pusher of side s sits at
// A + R(A)[(h0 + standoff) n_s + o t_s - D sig n_s] (anchor A = block-0 pose at
// the phase start), i.e. at P0 + sig V with P0 = A + R(A)((h0 + standoff) n_s
// + o t_s) and V = -D R(A) n_s, both fixed over the phase.
struct Push {
    float nx, ny, tx, ty;  // face normal n_s and tangent t_s (block frame)
    float P0x, P0y;        // pusher position at sig = 0 (world frame)
    float Vx, Vy;          // pusher travel over the phase (world frame)
};

// Anchor-frame quantities of a phase, kept for the adjoint.
struct Anchor {
    float cA, sA;          // rotation of the anchor
    float q0x, q0y;        // (h0 + standoff) n_s + o t_s (block frame)
};

// sin and cos by Cody-Waite reduction x = r + k pi/2 (pi/2 in two parts,
// fused multiply-adds), |r| <= pi/4, and Taylor polynomials in r^2 (sin to
// r^9, cos to r^10: truncation below 3e-9 on the reduced range); about one
// FP32 ulp over the block angles a push produces.
__device__ __forceinline__ void sincos_rd(float x, float& s, float& c) {
    const float k = rintf(x * 0.636619772f);  // 2/pi
    float r = fmaf(-k, 1.57079637f, x);       // pi/2 rounded to FP32
    r = fmaf(-k, -4.37113883e-8f, r);         // pi/2 minus that
    const float r2 = r * r;
    float ps = fmaf(r2, 2.75573192e-6f, -1.98412698e-4f);  // 1/9!, -1/7!
    ps = fmaf(r2, ps, 8.33333333e-3f);                     // 1/5!
    ps = fmaf(r2, ps, -1.66666667e-1f);                    // -1/3!
    const float sr = fmaf(r * r2, ps, r);
    float pc = fmaf(r2, -2.75573192e-7f, 2.48015873e-5f);  // -1/10!, 1/8!
    pc = fmaf(r2, pc, -1.38888889e-3f);                    // -1/6!
    pc = fmaf(r2, pc, 4.16666667e-2f);                     // 1/4!
    pc = fmaf(r2, pc, -0.5f);
    const float cr = fmaf(r2, pc, 1.0f);
    const int q = (int)k & 3;  // sin(r + q pi/2), cos(r + q pi/2)
    const float ss = (q & 1) ? cr : sr;
    const float cc = (q & 1) ? sr : cr;
    s = (q & 2) ? -ss : ss;
    c = ((q + 1) & 2) ? -cc : cc;
}

// The phase's pusher data from the anchor pose (Ax, Ay, Aph) and (o, D); the
// forward pass and the adjoint both build it here, so replays match bit for bit.
__device__ __forceinline__ void phase_push(const SimConst& c, float Ax, float Ay, float Aph, float o, float D,
                                           Push& p, Anchor& a) {
    sincos_rd(Aph, a.sA, a.cA);
    a.q0x = fmaf(c.h0d, p.nx, o * p.tx);
    a.q0y = fmaf(c.h0d, p.ny, o * p.ty);
    p.P0x = Ax + fmaf(a.cA, a.q0x, -(a.sA * a.q0y));
    p.P0y = Ay + fmaf(a.sA, a.q0x, a.cA * a.q0y);
    p.Vx = -D * fmaf(a.cA, p.nx, -(a.sA * p.ny));
    p.Vy = -D * fmaf(a.sA, p.nx, a.cA * p.ny);
}


// Tape entries hold, per (particle, side) sub-rollout, its blocks' states one
// after another: block b of sub-rollout 4i+s is slot (4i+s)B+b, 6 floats
// (x, y, phi, vx, vy, omega).
// They are read and written at a 32-bit float offset from a wave-uniform entry
// pointer (a scalar base plus a vector offset in the memory instruction).
__device__ __forceinline__ void load_blk_at(Blk& X, const float* __restrict__ entry, uint32_t off) {
    const float2* p = reinterpret_cast<const float2*>(entry + off);
    const float2 a = p[0], c = p[1], e = p[2];
    X.x = a.x;
    X.y = a.y;
    X.ph = c.x;
    X.vx = c.y;
    X.vy = e.x;
    X.om = e.y;
}

__device__ __forceinline__ void store_blk_at(const Blk& X, float* __restrict__ entry, uint32_t off) {
    float2* p = reinterpret_cast<float2*>(entry + off);
    p[0] = make_float2(X.x, X.y);
    p[1] = make_float2(X.ph, X.vx);
    p[2] = make_float2(X.vy, X.om);
}

// Push profile s((j + 1) / L) of step j of a phase: the wave evaluates 64
// consecutive steps at once (one per lane) and each step reads its value back
// with readlane, so a step costs one instruction instead of the polynomial.
// Every pass (forward, replay, reverse) takes the same per-lane expression.
__device__ __forceinline__ float profile_block(int j, float invL) {
    return push_profile((float)((j & ~63) + 1 + (int)__lane_id()) * invL);
}
__device__ __forceinline__ float profile_lane(float v, int j) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), j & 63));
}
struct Profile {
    float invL;
    int base;
    float v;
    __device__ __forceinline__ void reset(float inv) {
        invL = inv;
        base = -1;
    }
    __device__ __forceinline__ float at(int j) {
        const int b0 = j & ~63;
        if (b0 != base) {
            base = b0;
            v = profile_block(j, invL);
        }
        return profile_lane(v, j);
    }
};

// f(j, s((j + 1) / L)) for the steps j0 <= j < j1 of a phase.  A step of a
// rollout that has its SIMD to itself costs its instructions' issue and its
// branches (no other wave fills the fetch after a taken branch), so the loop
// over a block of 64 steps holds no profile check and no masked store.
// Forward at N = 1024, B = 3, T = 200: 74 us with the check, the mask and the
// per-phase inputs read at each phase start; 60 us without the check and with
// the inputs read once (phase_table); 55 us with the stores unmasked.
template <class F>
__device__ __forceinline__ void for_steps(int j0, int j1, float invL, F&& f) {
    for (int j = j0; j < j1;) {
        const float v = profile_block(j, invL);
        const int je = min(j1, (j & ~63) + 64);
#pragma unroll 1
        for (; j < je; ++j) f(j, profile_lane(v, j));
    }
}

// Index of the K-th block other than b (increasing order).
__host__ __device__ constexpr int other_block(int K, int b) { return K < b ? K : K + 1; }

// quad_perm control that hands lane slot b the value of slot other_block(K, b)
// of its own group of SL slots (an idle slot takes what block B - 1 takes).
template <int B, int K>
constexpr int other_sel() {
    constexpr int SL = Slots<B>::SL;
    int sel = 0;
    for (int p = 0; p < 4; ++p) {
        const int b = p % SL, base = p - b;
        int q = other_block(K, b < B ? b : B - 1);
        if (q >= SL) q = 0;
        sel |= (base + q) << (2 * p);
    }
    return sel;
}

template <int B, int K>
__device__ __forceinline__ float from_other_k(float v) {
    constexpr int sel = other_sel<B, K>();
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), sel, 0xF, 0xF, false));
}

// K is a constant of an unrolled loop (0..2).
template <int B>
__device__ __forceinline__ float from_other(float v, int K) {
    if (K == 0) return from_other_k<B, 0>(v);
    if (K == 1) return from_other_k<B, 1>(v);
    return from_other_k<B, 2>(v);
}

// Sum over the four sides of a particle (lanes SL apart): (v0+v1)+(v2+v3) on
// every lane, bit-identical.
template <int SL>
__device__ __forceinline__ float side_sum(float v) {
    if constexpr (SL == 1) {
        return quad_sum(v);
    } else {
        v = v + __shfl_xor(v, SL);
        return v + __shfl_xor(v, 2 * SL);
    }
}

// Sum over the block slots of a sub-rollout.
template <int SL>
__device__ __forceinline__ float slot_sum(float v) {
    if constexpr (SL >= 2) v = v + quad_xor1(v);
    if constexpr (SL == 4) v = v + quad_xor2(v);
    return v;
}

// Constants of this lane's block b (an idle slot duplicates block B - 1).
template <int B>
struct BlkConst {
    float cf, cr, ev2, ew2, dtm, dtI, crw2;
    float hs[B > 1 ? B - 1 : 1];  // h_b + h_q of the other blocks, increasing q
    float x0, y0, ph0;            // initial pose
};

template <int B>
__device__ __forceinline__ float pick(const float* a, int b) {
    float v = a[0];
#pragma unroll
    for (int q = 1; q < B; ++q) v = (b == q) ? a[q] : v;
    return v;
}

template <int B>
__device__ __forceinline__ BlkConst<B> blk_const(const SimConst& c, int b) {
    BlkConst<B> k;
    k.cf = pick<B>(c.cf, b);
    k.cr = pick<B>(c.cr, b);
    k.ev2 = pick<B>(c.ev2, b);
    k.ew2 = pick<B>(c.ew2, b);
    k.dtm = pick<B>(c.dtm, b);
    k.dtI = pick<B>(c.dtI, b);
    k.crw2 = pick<B>(c.crw2, b);
    float px[kMaxBlocks], py[kMaxBlocks], pp[kMaxBlocks];
#pragma unroll
    for (int q = 0; q < kMaxBlocks; ++q) {
        px[q] = c.pose0[q][0];
        py[q] = c.pose0[q][1];
        pp[q] = c.pose0[q][2];
    }
    k.x0 = pick<B>(px, b);
    k.y0 = pick<B>(py, b);
    k.ph0 = pick<B>(pp, b);
#pragma unroll
    for (int K = 0; K < (B > 1 ? B - 1 : 1); ++K) {
        float v = 0.0f;
#pragma unroll
        for (int bb = 0; bb < B; ++bb) v = (b == bb && B > 1 && K < B - 1) ? c.hsum[bb][other_block(K, bb)] : v;
        k.hs[K] = v;
    }
    return k;
}

// One semi-implicit Euler step of block b of the sub-rollout (pusher of this
// lane's side on block 0).  Products that feed a sum are fused (fmaf); the
// reverse below differentiates the same expressions.  Forces on a block sum in
// the order friction, pairs by increasing partner, pusher.
template <int B>
__device__ __forceinline__ void step_forward(const SimConst& c, const BlkConst<B>& k, int b, Blk& X, const Push& p,
                                             float sig) {
    constexpr int NO = B - 1;
    float ox[NO > 0 ? NO : 1], oy[NO > 0 ? NO : 1];
#pragma unroll
    for (int K = 0; K < NO; ++K) {
        ox[K] = from_other<B>(X.x, K);
        oy[K] = from_other<B>(X.y, K);
    }
    // regularised Coulomb friction
    const float inv = hw_rsq(fmaf(X.vx, X.vx, fmaf(X.vy, X.vy, k.ev2)));
    const float kf = k.cf * inv;
    float Fx = -kf * X.vx;
    float Fy = -kf * X.vy;
    const float invw = hw_rsq(fmaf(X.om, X.om, k.ew2));
    float Tq = -(k.cr * invw) * X.om;
    // block-block penalty on the inscribed disks, central force
#pragma unroll
    for (int K = 0; K < NO; ++K) {
        const float dx = X.x - ox[K], dy = X.y - oy[K];
        const float d2 = fmaf(dx, dx, fmaf(dy, dy, c.er2));
        const float rinv = hw_rsq(d2);
        const float pen = fmaf(-d2, rinv, k.hs[K]);  // h_b + h_q - r
        const float fr = c.kb * softplus(pen, c.beta_log2e, c.ln2_over_beta) * rinv;
        Fx = fmaf(fr, dx, Fx);
        Fy = fmaf(fr, dy, Fy);
    }
    // the virtual pusher of this side, on block 0: contact normal e = R(phi0) n
    {
        const float relx = fmaf(sig, p.Vx, p.P0x) - X.x;
        const float rely = fmaf(sig, p.Vy, p.P0y) - X.y;
        float s0, c0;
        sincos_rd(X.ph, s0, c0);
        const float ex = fmaf(c0, p.nx, -(s0 * p.ny)), ey = fmaf(s0, p.nx, c0 * p.ny);
        const float pen = c.h0 - fmaf(ex, relx, ey * rely);
        const float f = c.kp * softplus(pen, c.beta_log2e, c.ln2_over_beta);
        if (b == 0) {
            Fx = fmaf(-f, ex, Fx);
            Fy = fmaf(-f, ey, Fy);
            Tq = fmaf(-f, fmaf(relx, ey, -(rely * ex)), Tq);  // rel x (-f e)
        }
    }
    // semi-implicit Euler: velocities, then positions with the new velocities
    X.vx = fmaf(k.dtm, Fx, X.vx);
    X.vy = fmaf(k.dtm, Fy, X.vy);
    X.om = fmaf(k.dtI, Tq, X.om);
    X.x = fmaf(c.dt, X.vx, X.x);
    X.y = fmaf(c.dt, X.vy, X.y);
    X.ph = fmaf(c.dt, X.om, X.ph);
}

// The reverse of step_forward splits in two: what depends on the pre-step
// state X alone (linearise: the trigonometry, the contacts' forces and their
// derivatives) and the adjoint's own recursion (step_adjoint: products of
// these with the adjoint).  Only the second is a serial chain over the steps,
// so another wave may compute the first ahead of it.
// The values, in order: pusher relx rely ex ey s0 c0 cross f spg; friction vx
// vy kf q w; per other block dx dy rinv fr fs.
template <int B>
struct Lin {
    static constexpr int N = 14 + 5 * (B - 1);
    static constexpr int N4 = (N + 3) / 4;
    float v[4 * N4];
};

template <int B>
__device__ __forceinline__ void linearise(const SimConst& c, const BlkConst<B>& k, const Blk& X, const Push& p,
                                          float sig, Lin<B>& t) {
    constexpr int NO = B - 1;
    {
        const float relx = fmaf(sig, p.Vx, p.P0x) - X.x;
        const float rely = fmaf(sig, p.Vy, p.P0y) - X.y;
        float s0, c0;
        sincos_rd(X.ph, s0, c0);
        const float ex = fmaf(c0, p.nx, -(s0 * p.ny)), ey = fmaf(s0, p.nx, c0 * p.ny);
        const float pen = c.h0 - fmaf(ex, relx, ey * rely);
        const float u = softplus_u(pen, c.beta_log2e);
        const float rr = hw_rcp(1.0f + u);
        t.v[0] = relx;
        t.v[1] = rely;
        t.v[2] = ex;
        t.v[3] = ey;
        t.v[4] = s0;
        t.v[5] = c0;
        t.v[6] = fmaf(relx, ey, -(rely * ex));                                             // cross
        t.v[7] = c.kp * fmaf(hw_log2(1.0f + u), c.ln2_over_beta, fmaxf(pen, 0.0f));  // f
        t.v[8] = pen >= 0.0f ? rr : u * rr;                                                // sp'(pen)
    }
    {
        const float inv = hw_rsq(fmaf(X.vx, X.vx, fmaf(X.vy, X.vy, k.ev2)));
        const float kf = k.cf * inv;
        const float invw = hw_rsq(fmaf(X.om, X.om, k.ew2));
        t.v[9] = X.vx;
        t.v[10] = X.vy;
        t.v[11] = kf;
        t.v[12] = kf * inv * inv;
        t.v[13] = -(k.crw2 * (invw * invw * invw));
    }
#pragma unroll
    for (int K = 0; K < NO; ++K) {
        const float dx = X.x - from_other<B>(X.x, K), dy = X.y - from_other<B>(X.y, K);
        const float d2 = fmaf(dx, dx, fmaf(dy, dy, c.er2));
        const float rinv = hw_rsq(d2);
        const float pen = fmaf(-d2, rinv, k.hs[K]);
        const float u = softplus_u(pen, c.beta_log2e);
        const float fr = c.kb * fmaf(hw_log2(1.0f + u), c.ln2_over_beta, fmaxf(pen, 0.0f)) * rinv;
        const float rr = hw_rcp(1.0f + u);
        const float fp = c.kb * (pen >= 0.0f ? rr : u * rr);  // f'(pen)
        float* q = t.v + 14 + 5 * K;
        q[0] = dx;
        q[1] = dy;
        q[2] = rinv;
        q[3] = fr;
        q[4] = fr + fp;
    }
}

// On entry L is the adjoint of the block's post-step state; on exit that of
// its pre-step state.  Adjoints of the phase's pusher data (P0, V) are
// accumulated on block 0.
template <int B>
__device__ __forceinline__ void step_adjoint(const SimConst& c, const BlkConst<B>& k, int b, const Lin<B>& t, Blk& L,
                                             const Push& p, float sig, float& P0xb, float& P0yb, float& Vxb,
                                             float& Vyb) {
    constexpr int NO = B - 1;
    // integrator: x' = x + dt v', v' = v + (dt/m) F
    L.vx = fmaf(c.dt, L.x, L.vx);
    L.vy = fmaf(c.dt, L.y, L.vy);
    L.om = fmaf(c.dt, L.ph, L.om);
    const float Fxb = k.dtm * L.vx;
    const float Fyb = k.dtm * L.vy;
    const float Tqb = k.dtI * L.om;
    float ofx[NO > 0 ? NO : 1], ofy[NO > 0 ? NO : 1];
#pragma unroll
    for (int K = 0; K < NO; ++K) {
        ofx[K] = from_other<B>(Fxb, K);
        ofy[K] = from_other<B>(Fyb, K);
    }
    // pusher
    {
        const float relx = t.v[0], rely = t.v[1], ex = t.v[2], ey = t.v[3], s0 = t.v[4], c0 = t.v[5];
        const float cross = t.v[6], f = t.v[7], spg = t.v[8];
        // F0 += -f e, T0 += -f cross
        const float fb = -fmaf(cross, Tqb, fmaf(ex, Fxb, ey * Fyb));
        const float crossb = -f * Tqb;
        const float penb = fb * c.kp * spg;
        // cross = relx ey - rely ex, pen = h0 - (ex relx + ey rely)
        const float exb = fmaf(-f, Fxb, -fmaf(crossb, rely, penb * relx));
        const float eyb = fmaf(-f, Fyb, fmaf(crossb, relx, -(penb * rely)));
        const float relxb = fmaf(crossb, ey, -(penb * ex));
        const float relyb = -fmaf(crossb, ex, penb * ey);
        // e = (c0 nx - s0 ny, s0 nx + c0 ny)
        const float c0b = fmaf(exb, p.nx, eyb * p.ny);
        const float s0b = fmaf(eyb, p.nx, -(exb * p.ny));
        if (b == 0) {
            L.ph += fmaf(c0, s0b, -(s0 * c0b));
            // rel = P0 + sig V - x0
            L.x -= relxb;
            L.y -= relyb;
            P0xb += relxb;
            P0yb += relyb;
            Vxb = fmaf(sig, relxb, Vxb);
            Vyb = fmaf(sig, relyb, Vyb);
        }
    }
    // block-block contacts: F_b += f u with u = Delta / r, Delta = x_b - x_q
#pragma unroll
    for (int K = 0; K < NO; ++K) {
        const float* q = t.v + 14 + 5 * K;
        const float dx = q[0], dy = q[1], rinv = q[2], fr = q[3];
        const float gx = Fxb - ofx[K], gy = Fyb - ofy[K];
        const float gu = fmaf(gx, dx, gy * dy) * rinv;  // adjoint of f
        // d(f u)/dDelta = f/r (I - u u^T) + f'(pen)(-u) u^T
        const float k2 = q[4] * gu * rinv;  // coefficient of Delta
        L.x += fmaf(fr, gx, -(k2 * dx));
        L.y += fmaf(fr, gy, -(k2 * dy));
    }
    // friction
    const float vx = t.v[9], vy = t.v[10], kf = t.v[11];
    const float kd = t.v[12] * fmaf(Fxb, vx, Fyb * vy);
    L.vx = fmaf(kd, vx, fmaf(-kf, Fxb, L.vx));
    L.vy = fmaf(kd, vy, fmaf(-kf, Fyb, L.vy));
    L.om = fmaf(t.v[13], Tqb, L.om);
}

template <int B>
__device__ __forceinline__ void step_reverse(const SimConst& c, const BlkConst<B>& k, int b, const Blk& X, Blk& L,
                                             const Push& p, float sig, float& P0xb, float& P0yb, float& Vxb,
                                             float& Vyb) {
    Lin<B> t;
    linearise<B>(c, k, X, p, sig, t);
    step_adjoint<B>(c, k, b, t, L, p, sig, P0xb, P0yb, Vxb, Vyb);
}

__device__ __forceinline__ void side_frame(int s, Push& p) {
    p.nx = (s == 1) ? 1.0f : ((s == 3) ? -1.0f : 0.0f);
    p.ny = (s == 0) ? 1.0f : ((s == 2) ? -1.0f : 0.0f);
    p.tx = -p.ny;
    p.ty = p.nx;
}

// softmax(a)_s of this lane's side (max-subtracted, Eq. 5's relaxation)
__device__ __forceinline__ float side_weight(float a0, float a1, float a2, float a3, int s) {
    float m = fmaxf(fmaxf(a0, a1), fmaxf(a2, a3));
    float e0 = expf(a0 - m), e1 = expf(a1 - m), e2 = expf(a2 - m), e3 = expf(a3 - m);
    float es = (s == 0) ? e0 : (s == 1) ? e1 : (s == 2) ? e2 : e3;
    return es / (((e0 + e1) + e2) + e3);
}

// A lane's inputs of every phase -- its side's weight z, the offset o and the
// depth D -- read once before the time loop into the wave's LDS table
// [H][3][64].  Read at each phase start instead, they waited behind the tape
// stores in flight (memory operations complete in order), a drain of the
// store queue per phase.
constexpr int kPhaseFloats = 3 * 64;  // one phase of the table
__device__ __forceinline__ void phase_table(const float* __restrict__ theta, int N, int i, int s, int H, float* tab,
                                            int lw) {
    float a[kMaxPushes][6];
#pragma unroll
    for (int k = 0; k < kMaxPushes; ++k)
        if (k < H)
#pragma unroll
            for (int c = 0; c < 6; ++c) a[k][c] = theta[(int64_t)(6 * k + c) * N + i];
#pragma unroll
    for (int k = 0; k < kMaxPushes; ++k)
        if (k < H) {
            float* t = tab + k * kPhaseFloats + lw;
            t[0] = side_weight(a[k][0], a[k][1], a[k][2], a[k][3], s);
            t[64] = a[k][4];
            t[128] = a[k][5];
        }
}

__device__ __forceinline__ float smooth_abs(float u, float ea2) { return sqrtf(u * u + ea2); }

// ---------------------------------------------------------------------------
// Forward rollout of one lane: particle i, side s, block slot b.  Every lane of
// the wave runs it (cross-lane moves and readlane need all lanes): lanes past
// the last particle repeat particle N-1 and idle slots block B-1: they store
// the same values to the same places of the tape, so no store of the time loop
// is masked.  tab: the wave's phase table in LDS.
template <int B>
__device__ __forceinline__ void rollout_fwd_lane(const SimConst& c, int N, const float* __restrict__ theta,
                                                 float* __restrict__ cost, float* __restrict__ tape,
                                                 const TapeGeom& g, uint32_t* status, int64_t lane, float* tab) {
    constexpr int SL = Slots<B>::SL;
    const int64_t iw = lane / (4 * SL);
    const bool live = iw < N;
    const int i = live ? (int)iw : N - 1;
    const int r = (int)(lane % (4 * SL));
    const int s = r / SL, b = min(r % SL, B - 1);
    const int64_t slot = ((int64_t)4 * i + s) * B + b;
    const uint32_t off = (uint32_t)(slot * 6);  // within an entry (< 2^32 floats)
    const int64_t stride = 6 * B * g.lanes;  // floats per tape entry
    const int H = c.H, T = c.T;
    const int lw = (int)(lane & 63);
    phase_table(theta, N, i, s, H, tab, lw);
    const BlkConst<B> k = blk_const<B>(c, b);

    Blk S;
    S.x = k.x0;
    S.y = k.y0;
    S.ph = k.ph0;
    S.vx = S.vy = S.om = 0.0f;
    float Px[kMaxPushes + 1], Py[kMaxPushes + 1];  // block 0's, on slot 0
    float Lbound = 0.0f;
    Push p;
    side_frame(s, p);
    int64_t entry = 0;
    for (int kk = 0; kk < H; ++kk) {
        const int tk = phase_start(kk, T, H), tk1 = phase_start(kk + 1, T, H);
        const float invL = 1.0f / (float)(tk1 - tk);
        Px[kk] = S.x;
        Py[kk] = S.y;
        const float* ph = tab + kk * kPhaseFloats + lw;
        const float z = ph[0], o = ph[64], D = ph[128];
        Anchor an;
        phase_push(c, S.x, S.y, S.ph, o, D, p, an);  // block 0's anchor on slot 0
        Lbound += relu(fabsf(o) - c.omax) * relu(fabsf(o) - c.omax) + relu(-D) * relu(-D) +
                  relu(D - c.dmax) * relu(D - c.dmax);
        Blk X = S;
        const int nst = tk1 - tk;
        if (tape && g.ckpt == 0) {
            float* e = tape + (int64_t)tk * stride;
            for_steps(0, nst, invL, [&](int, float sig) {
                store_blk_at(X, e, off);
                e += stride;
                step_forward<B>(c, k, b, X, p, sig);
            });
        } else if (tape) {
            for (int js = 0; js < nst; js += g.ckpt, ++entry) {  // a checkpoint, then its segment
                store_blk_at(X, tape + entry * stride, off);
                for_steps(js, min(js + g.ckpt, nst), invL,
                          [&](int, float sig) { step_forward<B>(c, k, b, X, p, sig); });
            }
        } else {
            for_steps(0, nst, invL, [&](int, float sig) { step_forward<B>(c, k, b, X, p, sig); });
        }
        if (tape) store_blk_at(X, tape + g.ends_off + (int64_t)kk * stride, off);
        // phase mixture over the sides
        S.x = side_sum<SL>(z * X.x);
        S.y = side_sum<SL>(z * X.y);
        S.ph = side_sum<SL>(z * X.ph);
        S.vx = side_sum<SL>(z * X.vx);
        S.vy = side_sum<SL>(z * X.vy);
        S.om = side_sum<SL>(z * X.om);
    }
    Px[H] = S.x;
    Py[H] = S.y;
    if (r != 0 || !live) return;
    // cost (Appendix E-B), on slot 0 of side 0
    const float dxg = fabsf(Px[H] - c.goal[0]) - c.tol, dyg = fabsf(Py[H] - c.goal[1]) - c.tol;
    const float Ltarget = relu(dxg) * relu(dxg) + relu(dyg) * relu(dyg);
    const float Lrot = 1.0f - cosf(S.ph - c.goal[2]);
    float Ltraj = 0.0f;
    for (int kk = 1; kk <= H; ++kk) {
        Ltraj += smooth_abs(Px[kk - 1] - Px[kk], c.ea2) + smooth_abs(Py[kk - 1] - Py[kk], c.ea2);
        Ltraj += smooth_abs(Px[kk] - Px[H], c.ea2) + smooth_abs(Py[kk] - Py[H], c.ea2);
        Ltraj -= smooth_abs(Px[kk - 1] - Px[H], c.ea2) + smooth_abs(Py[kk - 1] - Py[H], c.ea2);
    }
    const float C = c.wt * Ltarget + c.wr * Lrot + c.wtr * Ltraj + c.wb * Lbound;
    cost[i] = C;
    if (status && !isfinite(C)) atomicOr(status, STAMP_STATUS_NONFINITE_COST);
}

// ---------------------------------------------------------------------------
// A wave's LDS table in the reverse sweep: the phase inputs [H][3][64]
// (phase_table), then the cost's adjoints of the phase starts [H][2][64].
constexpr int kSeedFloats = 2 * 64;
__host__ __device__ constexpr int adj_table_floats(int H) { return H * (kPhaseFloats + kSeedFloats); }

// dC/dP_k of the phase-start positions (times cost_bar) into the table, and
// the adjoint of the final block-0 pose in xb, yb, phb.  pos(k): P_k.
template <class F>
__device__ __forceinline__ void cost_seeds(const SimConst& c, int H, float cb, F&& pos, float PHx, float PHy, float phT,
                                           float* seeds, int lw, float& xb, float& yb, float& phb) {
    float Px[kMaxPushes], Py[kMaxPushes], Pxb[kMaxPushes], Pyb[kMaxPushes];
#pragma unroll
    for (int k = 0; k < kMaxPushes; ++k) {
        Pxb[k] = Pyb[k] = 0.0f;
        if (k < H) pos(k, Px[k], Py[k]);
    }
    xb = yb = 0.0f;
    {
        const float ux = PHx - c.goal[0], uy = PHy - c.goal[1];
        xb += cb * c.wt * 2.0f * relu(fabsf(ux) - c.tol) * copysignf(1.0f, ux);
        yb += cb * c.wt * 2.0f * relu(fabsf(uy) - c.tol) * copysignf(1.0f, uy);
    }
    phb = cb * c.wr * sinf(phT - c.goal[2]);
    const float wtr = cb * c.wtr;
    if (!c.per_phase) {
#pragma unroll
        for (int k = 1; k <= kMaxPushes; ++k) {
            float u, dd;
            if (k < H) {
                u = Px[k - 1] - Px[k];  dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k - 1] += dd;  Pxb[k] -= dd;
                u = Py[k - 1] - Py[k];  dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k - 1] += dd;  Pyb[k] -= dd;
                u = Px[k] - PHx;        dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k] += dd;      xb -= dd;
                u = Py[k] - PHy;        dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k] += dd;      yb -= dd;
                u = Px[k - 1] - PHx;    dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k - 1] -= dd;  xb += dd;
                u = Py[k - 1] - PHy;    dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k - 1] -= dd;  yb += dd;
            } else if (k == H) {  // P_k is P_H itself: its own term MH(P_H, P_H) has no gradient
                u = Px[k - 1] - PHx;    dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k - 1] += dd;  xb -= dd;
                u = Py[k - 1] - PHy;    dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k - 1] += dd;  yb -= dd;
                u = PHx - PHx;          dd = wtr * u / smooth_abs(u, c.ea2);  xb += dd;          xb -= dd;
                u = PHy - PHy;          dd = wtr * u / smooth_abs(u, c.ea2);  yb += dd;          yb -= dd;
                u = Px[k - 1] - PHx;    dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k - 1] -= dd;  xb += dd;
                u = Py[k - 1] - PHy;    dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k - 1] -= dd;  yb += dd;
            }
        }
    } else {
        // Per-phase split: term k of L_traj is phase k-1's and reaches only
        // that phase's end P_k (its start P_{k-1} and the final P_H are other
        // phases' constants); the last term, MH(P_H, P_H) = 2 eps_a, has no
        // gradient.  The target and rotation terms stay on the last phase.
#pragma unroll
        for (int k = 1; k < kMaxPushes; ++k) {
            if (k < H) {
                float u, dd;
                u = Px[k - 1] - Px[k];  dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k] -= dd;
                u = Py[k - 1] - Py[k];  dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k] -= dd;
                u = Px[k] - PHx;        dd = wtr * u / smooth_abs(u, c.ea2);  Pxb[k] += dd;
                u = Py[k] - PHy;        dd = wtr * u / smooth_abs(u, c.ea2);  Pyb[k] += dd;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kMaxPushes; ++k)
        if (k < H) {
            seeds[k * kSeedFloats + lw] = Pxb[k];
            seeds[k * kSeedFloats + 64 + lw] = Pyb[k];
        }
}

// Checkpoints of phase k (K > 0), and the tape entry its states start at.
__device__ __forceinline__ int phase_segments(int k, int T, int H, int K) {
    return (phase_start(k + 1, T, H) - phase_start(k, T, H) + K - 1) / K;
}
__device__ __forceinline__ int phase_entry(const TapeGeom& g, int k, int T, int H) {
    if (g.ckpt == 0) return phase_start(k, T, H);
    int e = 0;
    for (int q = 0; q < k; ++q) e += phase_segments(q, T, H, g.ckpt);
    return e;
}

// One lane of the block-per-lane layout in the reverse sweep.
template <int B>
struct AdjLane {
    int i, s, b, lw;
    bool live;  // lanes past the last particle repeat particle N-1: the same scratch values, no results
    bool blk;   // a block slot (an idle one duplicates block B - 1)
    int64_t slot0, stride;
    uint32_t off;
    __device__ __forceinline__ AdjLane(int N, int64_t lane, const TapeGeom& g) {
        constexpr int SL = Slots<B>::SL;
        const int64_t iw = lane / (4 * SL);
        live = iw < N;
        i = live ? (int)iw : N - 1;
        const int r = (int)(lane % (4 * SL));
        s = r / SL;
        b = min(r % SL, B - 1);
        blk = r % SL < B;
        lw = (int)(lane & 63);
        slot0 = ((int64_t)4 * i + s) * B;
        off = (uint32_t)((slot0 + b) * 6);
        stride = 6 * B * g.lanes;  // floats per tape entry
    }
};

// Reverse sweep of one lane; cost_bar (or cb_scalar when null) scales dC/dtheta.
// rev(k, entry, p, L, P0xb, P0yb, Vxb, Vyb) takes the adjoint L back through
// the steps of phase k, whose first tape entry is `entry`.  The phase's end
// states and anchor are read a phase ahead.
template <int B, class F>
__device__ __forceinline__ void reverse_sweep(const SimConst& c, int N, const AdjLane<B>& a,
                                              const float* __restrict__ tape, const TapeGeom& g,
                                              const float* __restrict__ cost_bar, float cb_scalar,
                                              float* __restrict__ grad, uint32_t* status, float* tab, F&& rev) {
    constexpr int SL = Slots<B>::SL;
    const int H = c.H, T = c.T, i = a.i, s = a.s, b = a.b, lw = a.lw;
    const int64_t stride = a.stride;
    float* seeds = tab + H * kPhaseFloats;
    int entry = phase_entry(g, H - 1, T, H);
    Blk Xe, A;  // the phase's end states and its start (block 0's pose: the anchor, on slot 0)
    load_blk_at(Xe, tape + g.ends_off + (int64_t)(H - 1) * stride, a.off);
    load_blk_at(A, tape + (int64_t)entry * stride, a.off);
    const float cb = cost_bar ? cost_bar[i] : cb_scalar;
    float PHx, PHy, phT;
    {
        const float z = tab[(H - 1) * kPhaseFloats + lw];
        const float* e = tape + g.ends_off + (int64_t)(H - 1) * stride + a.slot0 * 6;
        PHx = side_sum<SL>(z * e[0]);
        PHy = side_sum<SL>(z * e[1]);
        phT = side_sum<SL>(z * e[2]);
    }
    // adjoint of S_H (block 0 carries the cost's terms)
    float xb, yb, phb;
    cost_seeds(
        c, H, cb,
        [&](int k, float& x, float& y) {
            const float* e = tape + (int64_t)phase_entry(g, k, T, H) * stride + a.slot0 * 6;
            x = e[0];
            y = e[1];
        },
        PHx, PHy, phT, seeds, lw, xb, yb, phb);
    Blk Ls;
    Ls.x = Ls.y = Ls.ph = Ls.vx = Ls.vy = Ls.om = 0.0f;
    if (b == 0) {
        Ls.x = xb;
        Ls.y = yb;
        Ls.ph = phb;
    }

    Push p;
    side_frame(s, p);
    bool bad = false;
    for (int kk = H - 1; kk >= 0; --kk) {
        const float* pt = tab + kk * kPhaseFloats + lw;
        const float z = pt[0], o = pt[64], D = pt[128];
        // phase end: S_{k+1} = sum_s z_s X_s
        Blk L;
        const float zp = Ls.x * Xe.x + Ls.y * Xe.y + Ls.ph * Xe.ph + Ls.vx * Xe.vx + Ls.vy * Xe.vy + Ls.om * Xe.om;
        const float zb = slot_sum<SL>(a.blk ? zp : 0.0f);
        L.x = z * Ls.x;
        L.y = z * Ls.y;
        L.ph = z * Ls.ph;
        L.vx = z * Ls.vx;
        L.vy = z * Ls.vy;
        L.om = z * Ls.om;
        const float ab = z * (zb - side_sum<SL>(z * zb));  // softmax VJP
        Anchor an;
        phase_push(c, A.x, A.y, A.ph, o, D, p, an);
        const int here = entry;
        if (kk > 0) {
            entry -= g.ckpt == 0 ? phase_start(kk, T, H) - phase_start(kk - 1, T, H)
                                 : phase_segments(kk - 1, T, H, g.ckpt);
            load_blk_at(Xe, tape + g.ends_off + (int64_t)(kk - 1) * stride, a.off);
            load_blk_at(A, tape + (int64_t)entry * stride, a.off);
        }
        float P0xb = 0.0f, P0yb = 0.0f, Vxb = 0.0f, Vyb = 0.0f;
        rev(kk, here, p, L, P0xb, P0yb, Vxb, Vyb);
        // back to the anchor and (o, D): P0 = A + R(A) q0, q0 = (h0 + standoff) n + o t,
        // V = -D e_A, e_A = R(A) n (meaningful on slot 0, zero elsewhere)
        const float eAx = fmaf(an.cA, p.nx, -(an.sA * p.ny)), eAy = fmaf(an.sA, p.nx, an.cA * p.ny);
        const float Db = -fmaf(Vxb, eAx, Vyb * eAy);
        const float eAxb = -D * Vxb, eAyb = -D * Vyb;
        const float cAb = fmaf(eAxb, p.nx, eAyb * p.ny) + fmaf(P0xb, an.q0x, P0yb * an.q0y);
        const float sAb = fmaf(eAyb, p.nx, -(eAxb * p.ny)) + fmaf(P0yb, an.q0x, -(P0xb * an.q0y));
        const float q0xb = fmaf(an.cA, P0xb, an.sA * P0yb), q0yb = fmaf(an.cA, P0yb, -(an.sA * P0xb));
        const float ob = fmaf(q0xb, p.tx, q0yb * p.ty);
        const float Aphb = fmaf(an.cA, sAb, -(an.sA * cAb));
        // adjoint of S_k: the four sub-rollouts share it
        Ls.x = side_sum<SL>(L.x);
        Ls.y = side_sum<SL>(L.y);
        Ls.ph = side_sum<SL>(L.ph);
        Ls.vx = side_sum<SL>(L.vx);
        Ls.vy = side_sum<SL>(L.vy);
        Ls.om = side_sum<SL>(L.om);
        const float Axs = side_sum<SL>(P0xb), Ays = side_sum<SL>(P0yb), Aphs = side_sum<SL>(Aphb);
        const float obs = side_sum<SL>(ob), Dbs = side_sum<SL>(Db);
        if (c.per_phase) {
            // S_k is the previous phase's output: its adjoint stops here, and
            // the previous phase starts from its own term's seed on P_k
            Ls.x = Ls.y = Ls.ph = Ls.vx = Ls.vy = Ls.om = 0.0f;
        }
        if (b == 0) {
            const float Pxb = seeds[kk * kSeedFloats + lw], Pyb = seeds[kk * kSeedFloats + 64 + lw];
            if (c.per_phase) {
                Ls.x = Pxb;
                Ls.y = Pyb;
            } else {
                Ls.x += Axs + Pxb;
                Ls.y += Ays + Pyb;
                Ls.ph += Aphs;
            }
            // bound loss on o_k, D_k
            const float wb2 = 2.0f * cb * c.wb;
            const float obt = obs + wb2 * relu(fabsf(o) - c.omax) * copysignf(1.0f, o);
            const float Dbt = Dbs + wb2 * (relu(D - c.dmax) - relu(-D));
            if (a.live) {
                grad[(int64_t)(6 * kk + s) * N + i] = ab;
                if (s == 0) grad[(int64_t)(6 * kk + 4) * N + i] = obt;
                if (s == 1) grad[(int64_t)(6 * kk + 5) * N + i] = Dbt;
                bad = bad || !isfinite(ab) || !isfinite(obt) || !isfinite(Dbt);
            }
        }
    }
    if (status && bad) atomicOr(status, STAMP_STATUS_NONFINITE_GRAD);
}

// The reverse sweep with each wave doing its own steps: the batched kernel's,
// and the per-call one's where the split below does not pay.
template <int B>
__device__ __forceinline__ void rollout_adj_lane(const SimConst& c, int N, const float* __restrict__ theta,
                                                 const float* __restrict__ tape, const TapeGeom& g,
                                                 const float* __restrict__ cost_bar, float cb_scalar,
                                                 float* __restrict__ grad, float* __restrict__ seg,
                                                 uint32_t* status, int64_t lane, float* tab) {
    const AdjLane<B> a(N, lane, g);
    const BlkConst<B> k = blk_const<B>(c, a.b);
    const int H = c.H, T = c.T, b = a.b;
    const int64_t stride = a.stride;
    const uint32_t off = a.off;
    phase_table(theta, N, a.i, a.s, H, tab, a.lw);
    auto rev = [&](int kk, int entry, const Push& p, Blk& L, float& P0xb, float& P0yb, float& Vxb, float& Vyb) {
        const int nst = phase_start(kk + 1, T, H) - phase_start(kk, T, H);
        Profile prof;
        prof.reset(1.0f / (float)nst);
        if (g.ckpt == 0) {
            // reverse sweep over the full tape; the states of the next two
            // (earlier) steps are in flight while a step is reversed.  The
            // loads are unconditional (indices clamped at entry 0, whose
            // extra copies go unused): with a load on some paths only, the
            // compiler waits for every load in flight at the loop head.
            const float* base = tape + (int64_t)entry * stride;  // step j's entry: base + j stride
            int j = nst - 1;
            Blk XA, XB;
            load_blk_at(XA, base + (int64_t)j * stride, off);
            load_blk_at(XB, base + (int64_t)max(j - 1, 0) * stride, off);
            for (; j >= 1; j -= 2) {
                Blk X = XA;
                load_blk_at(XA, base + (int64_t)max(j - 2, 0) * stride, off);
                step_reverse<B>(c, k, b, X, L, p, prof.at(j), P0xb, P0yb, Vxb, Vyb);
                X = XB;
                load_blk_at(XB, base + (int64_t)max(j - 3, 0) * stride, off);
                step_reverse<B>(c, k, b, X, L, p, prof.at(j - 1), P0xb, P0yb, Vxb, Vyb);
            }
            if (j == 0) step_reverse<B>(c, k, b, XA, L, p, prof.at(0), P0xb, P0yb, Vxb, Vyb);
        } else {
            for (int q = (nst + g.ckpt - 1) / g.ckpt - 1; q >= 0; --q) {
                const int js = q * g.ckpt;
                const int je = min(js + g.ckpt, nst);
                Blk X;
                load_blk_at(X, tape + (int64_t)(entry + q) * stride, off);
                for (int j = js; j < je; ++j) {  // replay the segment
                    store_blk_at(X, seg + (int64_t)(j - js) * stride, off);
                    step_forward<B>(c, k, b, X, p, prof.at(j));
                }
                for (int j = je - 1; j >= js; --j) {
                    load_blk_at(X, seg + (int64_t)(j - js) * stride, off);  // a lane reads its own writes
                    step_reverse<B>(c, k, b, X, L, p, prof.at(j), P0xb, P0yb, Vxb, Vyb);
                }
            }
        }
    };
    reverse_sweep<B>(c, N, a, tape, g, cost_bar, cb_scalar, grad, status, tab, rev);
}

// ---------------------------------------------------------------------------
// The reverse sweep of a small particle set, split over the waves of a
// workgroup.  Such a set has fewer waves than the chip has SIMDs, and the
// sweep is one serial chain of T steps per lane: its time is the chain's
// length times the latency of a step.  Half of a step's instructions do not
// depend on the adjoint (linearise), so other waves of the workgroup, on SIMDs
// that would idle, compute them a chunk of steps ahead and pass them through
// LDS; wave 0 runs the recursion alone (step_adjoint).  The same instructions
// on the same operands as step_reverse: the same bits.
// Full tape, T = 200, N = 1024: B = 1 58 -> 33 us, B = 3 90 -> 47, B = 4 104 ->
// 54 (chunks of 2, 6 or 8 steps and 1, 3 or 4 helpers were no faster; one
// helper is the bottleneck itself, 83 us at B = 3).  Checkpoints every 32
// steps, T = 1000, N = 4096, B = 1: 490 -> 198 us (292 with a replay wave alone).

// A workgroup barrier that orders LDS only: __syncthreads would also wait for
// the loads of tape states in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kPipeHelpers = 2;  // waves that linearise: each takes every kPipeHelpers-th step of a chunk
// one of the two buffers of chunks of C steps
template <int B, int C>
__host__ __device__ constexpr int pipe_buffer_floats() { return C * Lin<B>::N4 * 4 * 64; }

// Step o of a chunk in its LDS buffer (q: this lane's column).
template <int B>
__device__ __forceinline__ void put_lin(float4* q, int o, Lin<B>& t) {
    constexpr int N4 = Lin<B>::N4;
#pragma unroll
    for (int v = Lin<B>::N; v < 4 * N4; ++v) t.v[v] = 0.0f;
#pragma unroll
    for (int v = 0; v < N4; ++v)
        q[(o * N4 + v) * 64] = make_float4(t.v[4 * v], t.v[4 * v + 1], t.v[4 * v + 2], t.v[4 * v + 3]);
}

// Push profile of the steps j0 .. j0 + 63, one per lane (profile_block's
// expression from any first step; profile_lane(v, j - j0) reads step j).
__device__ __forceinline__ float profile_from(int j0, float invL) {
    return push_profile((float)(j0 + 1 + (int)__lane_id()) * invL);
}

// The recursion over a chunk's steps jh, jh - 1, ... (those >= jl).
template <int B, int C>
__device__ __forceinline__ void chunk_adjoint(const SimConst& c, const BlkConst<B>& k, int b, const float4* q, int jh,
                                              int jl, float invL, Blk& L, const Push& p, float& P0xb, float& P0yb,
                                              float& Vxb, float& Vyb) {
    constexpr int N4 = Lin<B>::N4;
    const float v = profile_from(jh - C + 1, invL);
    Lin<B> t[C];
#pragma unroll
    for (int o = 0; o < C; ++o)
#pragma unroll
        for (int v = 0; v < N4; ++v) {
            const float4 x = q[(o * N4 + v) * 64];
            t[o].v[4 * v + 0] = x.x;
            t[o].v[4 * v + 1] = x.y;
            t[o].v[4 * v + 2] = x.z;
            t[o].v[4 * v + 3] = x.w;
        }
#pragma unroll
    for (int o = 0; o < C; ++o)
        if (jh - o >= jl) step_adjoint<B>(c, k, b, t[o], L, p, profile_lane(v, C - 1 - o), P0xb, P0yb, Vxb, Vyb);
}

// Full tape: two chunk buffers, filled and read in turn.
template <int B, int C>
__global__ __launch_bounds__(64 * (1 + kPipeHelpers)) void k_rollout_adj_split(SimConst c, int N, const float* __restrict__ theta,
                                                               const float* __restrict__ tape, TapeGeom g,
                                                               const float* __restrict__ cost_bar, float cb_scalar,
                                                               float* __restrict__ grad, uint32_t* status) {
    constexpr int W = kPipeHelpers, PER = C / W;
    static_assert(C % W == 0, "whole steps per helper");
    extern __shared__ __align__(16) float lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const AdjLane<B> a(N, (int64_t)blockIdx.x * 64 + (threadIdx.x & 63), g);
    const BlkConst<B> k = blk_const<B>(c, a.b);
    const int H = c.H, T = c.T;
    float4* buf = reinterpret_cast<float4*>(lds + adj_table_floats(H)) + a.lw;
    constexpr int kBuf = pipe_buffer_floats<B, C>() / 4;  // float4 of one buffer
    if (wave == 0) phase_table(theta, N, a.i, a.s, H, lds, a.lw);
    lds_barrier();
    int it = 0;  // chunk counter, the same in every wave
    if (wave == 0) {
        auto rev = [&](int kk, int, const Push& p, Blk& L, float& P0xb, float& P0yb, float& Vxb, float& Vyb) {
            const int nst = phase_start(kk + 1, T, H) - phase_start(kk, T, H);
            const float invL = 1.0f / (float)nst;
            for (int jh = nst - 1; jh >= 0; jh -= C, ++it) {
                lds_barrier();  // the chunk is filled
                chunk_adjoint<B, C>(c, k, a.b, buf + (it & 1) * kBuf, jh, 0, invL, L, p, P0xb, P0yb, Vxb, Vyb);
            }
        };
        reverse_sweep<B>(c, N, a, tape, g, cost_bar, cb_scalar, grad, status, lds, rev);
        lds_barrier();
        return;
    }
    // helpers: steps jh - o of each chunk, o = wave - 1, wave - 1 + W, ...
    const int o0 = wave - 1;
    Push p;
    side_frame(a.s, p);
    Blk A, X[PER];
    load_blk_at(A, tape + (int64_t)phase_start(H - 1, T, H) * a.stride, a.off);
#pragma unroll
    for (int m = 0; m < PER; ++m)
        load_blk_at(X[m], tape + (int64_t)max(T - 1 - (o0 + W * m), 0) * a.stride, a.off);
    for (int kk = H - 1; kk >= 0; --kk) {
        const int tk = phase_start(kk, T, H), nst = phase_start(kk + 1, T, H) - tk;
        const float* pt = lds + kk * kPhaseFloats + a.lw;
        Anchor an;
        phase_push(c, A.x, A.y, A.ph, pt[64], pt[128], p, an);
        if (kk > 0) load_blk_at(A, tape + (int64_t)phase_start(kk - 1, T, H) * a.stride, a.off);
        const float invL = 1.0f / (float)nst;
        for (int jh = nst - 1; jh >= 0; jh -= C, ++it) {
            // the next chunk's states load while this one's are linearised (the
            // next phase's first chunk starts at its last step)
            const int tn = jh - C >= 0 ? tk + jh - C : tk - 1;
            Blk Xn[PER];
#pragma unroll
            for (int m = 0; m < PER; ++m)
                load_blk_at(Xn[m], tape + (int64_t)max(tn - (o0 + W * m), 0) * a.stride, a.off);
            float4* q = buf + (it & 1) * kBuf;
            const float v = profile_from(jh - C + 1, invL);
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                const int o = o0 + W * m, j = jh - o;
                if (j >= 0) {
                    Lin<B> t;
                    linearise<B>(c, k, X[m], p, profile_lane(v, C - 1 - o), t);
                    put_lin<B>(q, o, t);
                }
                X[m] = Xn[m];
            }
            lds_barrier();  // the chunk is filled; wave 0 is past the other buffer
        }
    }
    lds_barrier();
}

// The segments of a checkpointed tape in reverse order, as every wave of the
// kernels below walks them: segment q of phase k, steps js .. js + n - 1.
struct SegWalk {
    int H, T, K, k, q, nst, n;
    __device__ __forceinline__ void phase(int kk) {
        k = kk;
        nst = phase_start(kk + 1, T, H) - phase_start(kk, T, H);
        q = (nst + K - 1) / K - 1;
        n = nst - q * K;
    }
    __device__ __forceinline__ SegWalk(int H_, int T_, int K_) : H(H_), T(T_), K(K_) { phase(H - 1); }
    // false past the first segment (n = 0 then)
    __device__ __forceinline__ bool next() {
        if (q > 0) {
            --q;
            n = K;
            return true;
        }
        if (k > 0) {
            phase(k - 1);
            return true;
        }
        n = 0;
        return false;
    }
};

// Checkpoints: while wave 0 runs the recursion over one segment, waves 1 and 2
// linearise its steps a chunk ahead, from states in LDS, and wave 3 replays
// the segment before it from its checkpoint into the other state buffer
// [K][3][64] float2 (a segment's replay needs no other's).  Everything moves in
// intervals of C steps, one barrier each; a segment's stage has as many
// intervals as its own chunks or the next replay's need.
template <int B, int C>
__global__ __launch_bounds__(64 * (2 + kPipeHelpers)) void k_rollout_adj_ckpt(SimConst c, int N, const float* __restrict__ theta,
                                                              const float* __restrict__ tape, TapeGeom g,
                                                              const float* __restrict__ cost_bar, float cb_scalar,
                                                              float* __restrict__ grad, uint32_t* status) {
    constexpr int W = kPipeHelpers, PER = C / W;
    extern __shared__ __align__(16) float lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const AdjLane<B> a(N, (int64_t)blockIdx.x * 64 + (threadIdx.x & 63), g);
    const BlkConst<B> k = blk_const<B>(c, a.b);
    const int H = c.H, T = c.T, K = g.ckpt;
    constexpr int kBuf = pipe_buffer_floats<B, C>() / 4;
    float4* buf = reinterpret_cast<float4*>(lds + adj_table_floats(H)) + a.lw;
    float2* states = reinterpret_cast<float2*>(lds + adj_table_floats(H) + 8 * kBuf) + a.lw;
    const int kStates = K * 3 * 64;  // float2 of one state buffer
    auto intervals = [&](int n) { return (n + C - 1) / C; };
    if (wave == 0) phase_table(theta, N, a.i, a.s, H, lds, a.lw);
    lds_barrier();
    SegWalk w(H, T, K);
    int it = 0;  // interval counter, the same in every wave
    if (wave == 0) {
        auto rev = [&](int kk, int, const Push& p, Blk& L, float& P0xb, float& P0yb, float& Vxb, float& Vyb) {
            if (kk == H - 1)  // the first segment's replay
                for (int m = intervals(w.n); m > 0; --m, ++it) lds_barrier();
            const float invL = 1.0f / (float)w.nst;
            for (bool more = true; more && w.k == kk;) {
                const int js = w.q * K, n = w.n, nc = intervals(n);
                more = w.next();
                for (int m = 0; m < max(nc, intervals(w.n)); ++m, ++it) {
                    lds_barrier();  // the chunk is filled
                    if (m < nc)
                        chunk_adjoint<B, C>(c, k, a.b, buf + (it & 1) * kBuf, js + n - 1 - m * C, js, invL, L, p, P0xb,
                                            P0yb, Vxb, Vyb);
                }
            }
        };
        reverse_sweep<B>(c, N, a, tape, g, cost_bar, cb_scalar, grad, status, lds, rev);
        lds_barrier();
        return;
    }
    Push p;
    side_frame(a.s, p);
    int kp = -1;  // the phase p is for
    float invL = 0.0f;
    Blk A;  // the next phase's anchor
    load_blk_at(A, tape + (int64_t)phase_entry(g, H - 1, T, H) * a.stride, a.off);
    auto enter = [&](int kk, int nst) {  // at a phase's first segment
        if (kk == kp) return;
        kp = kk;
        const float* pt = lds + kk * kPhaseFloats + a.lw;
        Anchor an;
        phase_push(c, A.x, A.y, A.ph, pt[64], pt[128], p, an);
        if (kk > 0) load_blk_at(A, tape + (int64_t)phase_entry(g, kk - 1, T, H) * a.stride, a.off);
        invL = 1.0f / (float)nst;
    };
    if (wave <= W) {
        const int o0 = wave - 1;
        for (int m = intervals(w.n); m > 0; --m, ++it) lds_barrier();
        int par = 0;
        for (bool more = true; more; par ^= 1) {
            enter(w.k, w.nst);
            const int js = w.q * K, n = w.n, nc = intervals(n);
            more = w.next();
            for (int m = 0; m < max(nc, intervals(w.n)); ++m, ++it) {
                float4* q = buf + (it & 1) * kBuf;
                const float v = profile_from(js + n - (m + 1) * C, invL);
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const int o = o0 + W * u, r = n - 1 - m * C - o;  // step js + r
                    if (r >= 0) {
                        const float2* e = states + par * kStates + 3 * r * 64;
                        const float2 x = e[0], y = e[64], z = e[128];
                        const Blk X{x.x, x.y, y.x, y.y, z.x, z.y};
                        Lin<B> t;
                        linearise<B>(c, k, X, p, profile_lane(v, C - 1 - o), t);
                        put_lin<B>(q, o, t);
                    }
                }
                lds_barrier();
            }
        }
        lds_barrier();
        return;
    }
    // replay: the first segment in a stage of its own, each other one during
    // the stage of the segment after it
    int64_t entry = g.n_entries - 1;  // the segment's checkpoint
    Blk X, Xn;
    load_blk_at(Xn, tape + entry * a.stride, a.off);
    int par = 0, before = 0;  // before: chunks of the segment whose stage this is
    for (;; par ^= 1) {
        const int n = w.n;
        X = Xn;
        if (n > 0) enter(w.k, w.nst);
        entry = max(entry - 1, (int64_t)0);
        load_blk_at(Xn, tape + entry * a.stride, a.off);
        const int js = w.q * K;
        float2* e = states + par * kStates;
        for (int m = 0; m < max(before, intervals(n)); ++m, ++it) {
            const float v = profile_from(js + m * C, invL);
            auto step = [&](int o) {
                e[0] = make_float2(X.x, X.y);
                e[64] = make_float2(X.ph, X.vx);
                e[128] = make_float2(X.vy, X.om);
                e += 3 * 64;
                step_forward<B>(c, k, a.b, X, p, profile_lane(v, o));
            };
            if (n >= (m + 1) * C) {
#pragma unroll
                for (int o = 0; o < C; ++o) step(o);
            } else {
                for (int o = 0; m * C + o < n; ++o) step(o);
            }
            lds_barrier();
        }
        if (n == 0) break;
        before = intervals(n);
        w.next();
    }
    lds_barrier();
}

// The same for segments too long for that kernel's LDS: wave 1 replays, wave
// 0 reverses the segment after it, each step whole.
template <int B>
__global__ __launch_bounds__(128) void k_rollout_adj_replay(SimConst c, int N, const float* __restrict__ theta,
                                                            const float* __restrict__ tape, TapeGeom g,
                                                            const float* __restrict__ cost_bar, float cb_scalar,
                                                            float* __restrict__ grad, uint32_t* status) {
    extern __shared__ __align__(16) float lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const AdjLane<B> a(N, (int64_t)blockIdx.x * 64 + (threadIdx.x & 63), g);
    const BlkConst<B> k = blk_const<B>(c, a.b);
    const int H = c.H, T = c.T, K = g.ckpt;
    float2* buf = reinterpret_cast<float2*>(lds + adj_table_floats(H)) + a.lw;
    const int kBuf = K * 3 * 64;  // float2 of one buffer
    if (wave == 0) phase_table(theta, N, a.i, a.s, H, lds, a.lw);
    lds_barrier();
    int it = 0;  // segment counter, the same in both waves
    if (wave == 0) {
        auto rev = [&](int kk, int, const Push& p, Blk& L, float& P0xb, float& P0yb, float& Vxb, float& Vyb) {
            const int nst = phase_start(kk + 1, T, H) - phase_start(kk, T, H);
            Profile prof;
            prof.reset(1.0f / (float)nst);
            for (int q = (nst + K - 1) / K - 1; q >= 0; --q, ++it) {
                lds_barrier();  // the segment is replayed
                const int js = q * K, je = min(js + K, nst);
                const float2* e = buf + (it & 1) * kBuf;
                auto read = [&](int j) {
                    const float2 x = e[3 * (j - js) * 64], y = e[(3 * (j - js) + 1) * 64], w = e[(3 * (j - js) + 2) * 64];
                    return Blk{x.x, x.y, y.x, y.y, w.x, w.y};
                };
                Blk X = read(je - 1);
                for (int j = je - 1; j >= js; --j) {
                    const Blk Xn = read(max(j - 1, js));  // the next step's state loads during this one
                    step_reverse<B>(c, k, a.b, X, L, p, prof.at(j), P0xb, P0yb, Vxb, Vyb);
                    X = Xn;
                }
            }
        };
        reverse_sweep<B>(c, N, a, tape, g, cost_bar, cb_scalar, grad, status, lds, rev);
        lds_barrier();
        return;
    }
    Push p;
    side_frame(a.s, p);
    int entry = phase_entry(g, H - 1, T, H);
    Blk A, X;
    load_blk_at(A, tape + (int64_t)entry * a.stride, a.off);
    load_blk_at(X, tape + (g.n_entries - 1) * a.stride, a.off);
    for (int kk = H - 1; kk >= 0; --kk) {
        const int nst = phase_start(kk + 1, T, H) - phase_start(kk, T, H);
        const float* pt = lds + kk * kPhaseFloats + a.lw;
        Anchor an;
        phase_push(c, A.x, A.y, A.ph, pt[64], pt[128], p, an);
        const int here = entry;
        if (kk > 0) {
            entry -= phase_segments(kk - 1, T, H, K);
            load_blk_at(A, tape + (int64_t)entry * a.stride, a.off);
        }
        for (int q = (nst + K - 1) / K - 1; q >= 0; --q, ++it) {
            const int js = q * K, je = min(js + K, nst);
            Blk Xn;  // the checkpoint of the segment before
            load_blk_at(Xn, tape + (int64_t)max(here + q - 1, 0) * a.stride, a.off);
            float2* e = buf + (it & 1) * kBuf;
            auto put = [&]() {
                e[0] = make_float2(X.x, X.y);
                e[64] = make_float2(X.ph, X.vx);
                e[128] = make_float2(X.vy, X.om);
                e += 3 * 64;
            };
            for_steps(js, je - 1, 1.0f / (float)nst, [&](int, float sig) {
                put();
                step_forward<B>(c, k, a.b, X, p, sig);
            });
            put();  // the last step's result is the next segment's checkpoint
            X = Xn;
            lds_barrier();  // the segment is replayed; wave 0 is past the other buffer
        }
    }
    lds_barrier();
}

// ---------------------------------------------------------------------------
// Packed lanes: one lane per (particle i, side s) sub-rollout, holding all B
// blocks (lane = 4i + s).  A step then costs B frictions, B(B-1)/2 pair terms
// (each once) and one pusher per lane, with no cross-lane moves, instead of
// 4 SL lanes per particle that repeat every pair term twice and the pusher on
// every block slot (at B = 3 one slot in four idles).  It rounds exactly as
// the block-per-lane form: each block's forces add in the same order
// (friction, partners by increasing index, pusher), the higher block of a
// pair takes the lower block's term with Delta negated (negation is exact),
// and the sides and blocks meet in the same sums.  Same tape layout.

// One semi-implicit Euler step of all B blocks of a sub-rollout.
template <int B>
__device__ __forceinline__ void step_forward_packed(const SimConst& c, Blk (&X)[B], const Push& p, float sig) {
    float Fx[B], Fy[B], Tq[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const float inv = hw_rsq(fmaf(X[b].vx, X[b].vx, fmaf(X[b].vy, X[b].vy, c.ev2[b])));
        const float kf = c.cf[b] * inv;
        Fx[b] = -kf * X[b].vx;
        Fy[b] = -kf * X[b].vy;
        const float invw = hw_rsq(fmaf(X[b].om, X[b].om, c.ew2[b]));
        Tq[b] = -(c.cr[b] * invw) * X[b].om;
    }
    // pair terms, once per pair b < q: Delta = x_b - x_q, force fr Delta on b
    float pdx[B][B], pdy[B][B], pfr[B][B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
        for (int q = b + 1; q < B; ++q) {
            const float dx = X[b].x - X[q].x, dy = X[b].y - X[q].y;
            const float d2 = fmaf(dx, dx, fmaf(dy, dy, c.er2));
            const float rinv = hw_rsq(d2);
            const float pen = fmaf(-d2, rinv, c.hsum[b][q]);
            pdx[b][q] = dx;
            pdy[b][q] = dy;
            pfr[b][q] = c.kb * softplus(pen, c.beta_log2e, c.ln2_over_beta) * rinv;
        }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
        for (int q = 0; q < B; ++q) {
            if (q == b) continue;
            const float fr = q > b ? pfr[b][q] : pfr[q][b];
            const float dx = q > b ? pdx[b][q] : -pdx[q][b];
            const float dy = q > b ? pdy[b][q] : -pdy[q][b];
            Fx[b] = fmaf(fr, dx, Fx[b]);
            Fy[b] = fmaf(fr, dy, Fy[b]);
        }
    }
    // the virtual pusher of this side, on block 0: contact normal e = R(phi0) n
    {
        const float relx = fmaf(sig, p.Vx, p.P0x) - X[0].x;
        const float rely = fmaf(sig, p.Vy, p.P0y) - X[0].y;
        float s0, c0;
        sincos_rd(X[0].ph, s0, c0);
        const float ex = fmaf(c0, p.nx, -(s0 * p.ny)), ey = fmaf(s0, p.nx, c0 * p.ny);
        const float pen = c.h0 - fmaf(ex, relx, ey * rely);
        const float f = c.kp * softplus(pen, c.beta_log2e, c.ln2_over_beta);
        Fx[0] = fmaf(-f, ex, Fx[0]);
        Fy[0] = fmaf(-f, ey, Fy[0]);
        Tq[0] = fmaf(-f, fmaf(relx, ey, -(rely * ex)), Tq[0]);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        X[b].vx = fmaf(c.dtm[b], Fx[b], X[b].vx);
        X[b].vy = fmaf(c.dtm[b], Fy[b], X[b].vy);
        X[b].om = fmaf(c.dtI[b], Tq[b], X[b].om);
        X[b].x = fmaf(c.dt, X[b].vx, X[b].x);
        X[b].y = fmaf(c.dt, X[b].vy, X[b].y);
        X[b].ph = fmaf(c.dt, X[b].om, X[b].ph);
    }
}

// Reverse of step_forward_packed at pre-step states X; L: post-step adjoints
// on entry, pre-step adjoints on exit; pusher adjoints accumulate as in
// step_reverse (block 0).
template <int B>
__device__ __forceinline__ void step_reverse_packed(const SimConst& c, const Blk (&X)[B], Blk (&L)[B], const Push& p,
                                                    float sig, float& P0xb, float& P0yb, float& Vxb, float& Vyb) {
    float Fxb[B], Fyb[B], Tqb[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        L[b].vx = fmaf(c.dt, L[b].x, L[b].vx);
        L[b].vy = fmaf(c.dt, L[b].y, L[b].vy);
        L[b].om = fmaf(c.dt, L[b].ph, L[b].om);
        Fxb[b] = c.dtm[b] * L[b].vx;
        Fyb[b] = c.dtm[b] * L[b].vy;
        Tqb[b] = c.dtI[b] * L[b].om;
    }
    // pusher (block 0)
    {
        const float relx = fmaf(sig, p.Vx, p.P0x) - X[0].x;
        const float rely = fmaf(sig, p.Vy, p.P0y) - X[0].y;
        float s0, c0;
        sincos_rd(X[0].ph, s0, c0);
        const float ex = fmaf(c0, p.nx, -(s0 * p.ny)), ey = fmaf(s0, p.nx, c0 * p.ny);
        const float cross = fmaf(relx, ey, -(rely * ex));
        const float pen = c.h0 - fmaf(ex, relx, ey * rely);
        const float u = softplus_u(pen, c.beta_log2e);
        const float f = c.kp * fmaf(hw_log2(1.0f + u), c.ln2_over_beta, fmaxf(pen, 0.0f));
        const float rr = hw_rcp(1.0f + u);
        const float spg = pen >= 0.0f ? rr : u * rr;
        const float fb = -fmaf(cross, Tqb[0], fmaf(ex, Fxb[0], ey * Fyb[0]));
        const float crossb = -f * Tqb[0];
        const float penb = fb * c.kp * spg;
        const float exb = fmaf(-f, Fxb[0], -fmaf(crossb, rely, penb * relx));
        const float eyb = fmaf(-f, Fyb[0], fmaf(crossb, relx, -(penb * rely)));
        const float relxb = fmaf(crossb, ey, -(penb * ex));
        const float relyb = -fmaf(crossb, ex, penb * ey);
        const float c0b = fmaf(exb, p.nx, eyb * p.ny);
        const float s0b = fmaf(eyb, p.nx, -(exb * p.ny));
        L[0].ph += fmaf(c0, s0b, -(s0 * c0b));
        L[0].x -= relxb;
        L[0].y -= relyb;
        P0xb += relxb;
        P0yb += relyb;
        Vxb = fmaf(sig, relxb, Vxb);
        Vyb = fmaf(sig, relyb, Vyb);
    }
    // block-block contacts, once per pair b < q; each block adds its partners
    // in increasing order
    float pdx[B][B], pdy[B][B], pfr[B][B], pk2[B][B], pgx[B][B], pgy[B][B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
        for (int q = b + 1; q < B; ++q) {
            const float dx = X[b].x - X[q].x, dy = X[b].y - X[q].y;
            const float d2 = fmaf(dx, dx, fmaf(dy, dy, c.er2));
            const float rinv = hw_rsq(d2);
            const float pen = fmaf(-d2, rinv, c.hsum[b][q]);
            const float u = softplus_u(pen, c.beta_log2e);
            const float fr = c.kb * fmaf(hw_log2(1.0f + u), c.ln2_over_beta, fmaxf(pen, 0.0f)) * rinv;
            const float rr = hw_rcp(1.0f + u);
            const float fp = c.kb * (pen >= 0.0f ? rr : u * rr);
            const float gx = Fxb[b] - Fxb[q], gy = Fyb[b] - Fyb[q];
            const float gu = fmaf(gx, dx, gy * dy) * rinv;
            pdx[b][q] = dx;
            pdy[b][q] = dy;
            pfr[b][q] = fr;
            pk2[b][q] = (fr + fp) * gu * rinv;
            pgx[b][q] = gx;
            pgy[b][q] = gy;
        }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
        for (int q = 0; q < B; ++q) {
            if (q == b) continue;
            const int lo = q > b ? b : q, hi = q > b ? q : b;
            const float sg = q > b ? 1.0f : -1.0f;  // the higher block sees Delta and g negated
            const float fr = pfr[lo][hi], k2 = pk2[lo][hi];
            const float dx = sg * pdx[lo][hi], dy = sg * pdy[lo][hi];
            const float gx = sg * pgx[lo][hi], gy = sg * pgy[lo][hi];
            L[b].x += fmaf(fr, gx, -(k2 * dx));
            L[b].y += fmaf(fr, gy, -(k2 * dy));
        }
    }
    // friction
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const float inv = hw_rsq(fmaf(X[b].vx, X[b].vx, fmaf(X[b].vy, X[b].vy, c.ev2[b])));
        const float kf = c.cf[b] * inv;
        const float kd = kf * inv * inv * fmaf(Fxb[b], X[b].vx, Fyb[b] * X[b].vy);
        L[b].vx = fmaf(kd, X[b].vx, fmaf(-kf, Fxb[b], L[b].vx));
        L[b].vy = fmaf(kd, X[b].vy, fmaf(-kf, Fyb[b], L[b].vy));
        const float invw = hw_rsq(fmaf(X[b].om, X[b].om, c.ew2[b]));
        L[b].om = fmaf(-(c.crw2[b] * (invw * invw * invw)), Tqb[b], L[b].om);
    }
}

template <int B>
__device__ __forceinline__ void load_blks(Blk (&X)[B], const float* __restrict__ entry, uint32_t off) {
#pragma unroll
    for (int b = 0; b < B; ++b) load_blk_at(X[b], entry, off + 6 * b);
}

template <int B>
__device__ __forceinline__ void store_blks(const Blk (&X)[B], float* __restrict__ entry, uint32_t off) {
#pragma unroll
    for (int b = 0; b < B; ++b) store_blk_at(X[b], entry, off + 6 * b);
}

// Sum over the block slots in the block-per-lane form's order: (v0+v1)+(v2+v3),
// an absent fourth slot adding zero.
template <int B>
__device__ __forceinline__ float blocks_sum(const float (&v)[B]) {
    if constexpr (B == 1) return v[0];
    else if constexpr (B == 2) return v[0] + v[1];
    else if constexpr (B == 3) return (v[0] + v[1]) + (v[2] + 0.0f);
    else return (v[0] + v[1]) + (v[2] + v[3]);
}

// Orders a wave's LDS writes before its later LDS reads by other lanes of the
// same wave (and those reads before later writes): LDS instructions of one
// wave execute in issue order; the fences keep the compiler from moving them
// and wait for the writes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int B>
__device__ __forceinline__ void stage_blks(const Blk (&X)[B], float* stage, int lw) {
    float2* q = reinterpret_cast<float2*>(stage + lw * 6 * B);
#pragma unroll
    for (int b = 0; b < B; ++b) {
        q[3 * b + 0] = make_float2(X[b].x, X[b].y);
        q[3 * b + 1] = make_float2(X[b].ph, X[b].vx);
        q[3 * b + 2] = make_float2(X[b].vy, X[b].om);
    }
}

// Forward rollout of one packed lane (particle i, side s); as rollout_fwd_lane.
// lds: this wave's LDS, the phase table [H][3][64] and then the staging of its
// tape stores (64 lanes x 6B floats).
template <int B>
__device__ __forceinline__ void rollout_fwd_packed(const SimConst& c, int N, const float* __restrict__ theta,
                                                   float* __restrict__ cost, float* __restrict__ tape,
                                                   const TapeGeom& g, uint32_t* status, int64_t lane, float* lds) {
    const int64_t iw = lane / 4;
    const bool live = iw < N;
    const int i = live ? (int)iw : N - 1;
    const int s = (int)(lane % 4);
    const uint32_t off = (uint32_t)(((int64_t)4 * i + s) * B * 6);
    const int64_t stride = 6 * B * g.lanes;
    const int H = c.H, T = c.T;
    // the wave's span of a tape entry: its live lanes' 6B floats each, from
    // the first lane's slot on (a multiple of 4 floats: lanes come in
    // particles of 4)
    const int lw = (int)(lane & 63);
    float* stage = lds + H * kPhaseFloats;
    phase_table(theta, N, i, s, H, lds, lw);
    const int64_t lane0 = lane - lw;
    const int64_t wave_off = lane0 * 6 * B;
    const int span4 = (int)(min((int64_t)64, (int64_t)4 * N - lane0) * 6 * B / 4);
    Blk S[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        S[b].x = c.pose0[b][0];
        S[b].y = c.pose0[b][1];
        S[b].ph = c.pose0[b][2];
        S[b].vx = S[b].vy = S[b].om = 0.0f;
    }
    float Px[kMaxPushes + 1], Py[kMaxPushes + 1];
    float Lbound = 0.0f;
    Push p;
    side_frame(s, p);
    int64_t entry = 0;
    for (int kk = 0; kk < H; ++kk) {
        const int tk = phase_start(kk, T, H), tk1 = phase_start(kk + 1, T, H);
        const float invL = 1.0f / (float)(tk1 - tk);
        Px[kk] = S[0].x;
        Py[kk] = S[0].y;
        const float* ph = lds + kk * kPhaseFloats + lw;
        const float z = ph[0], o = ph[64], D = ph[128];
        Anchor an;
        phase_push(c, S[0].x, S[0].y, S[0].ph, o, D, p, an);
        Lbound += relu(fabsf(o) - c.omax) * relu(fabsf(o) - c.omax) + relu(-D) * relu(-D) +
                  relu(D - c.dmax) * relu(D - c.dmax);
        Blk X[B];
#pragma unroll
        for (int b = 0; b < B; ++b) X[b] = S[b];
        const int nst = tk1 - tk;
        if (tape && g.ckpt == 0) {
            // Each step's states go through LDS so that the wave writes its
            // contiguous span of the entry with 16-byte stores of consecutive
            // lanes (a lane's own 6B floats would make every store
            // instruction touch B times the cache lines).
            float* e = tape + (int64_t)tk * stride + wave_off;
            for_steps(0, nst, invL, [&](int, float sig) {
                stage_blks<B>(X, stage, lw);
                wave_lds_sync();
                for (int k = lw; k < span4; k += 64)
                    *reinterpret_cast<float4*>(e + 4 * k) = *reinterpret_cast<const float4*>(stage + 4 * k);
                wave_lds_sync();
                e += stride;
                step_forward_packed<B>(c, X, p, sig);
            });
        } else if (tape) {
            for (int js = 0; js < nst; js += g.ckpt, ++entry) {
                if (live) store_blks<B>(X, tape + entry * stride, off);
                for_steps(js, min(js + g.ckpt, nst), invL, [&](int, float sig) { step_forward_packed<B>(c, X, p, sig); });
            }
        } else {
            for_steps(0, nst, invL, [&](int, float sig) { step_forward_packed<B>(c, X, p, sig); });
        }
        if (tape && live) store_blks<B>(X, tape + g.ends_off + (int64_t)kk * stride, off);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            S[b].x = side_sum<1>(z * X[b].x);
            S[b].y = side_sum<1>(z * X[b].y);
            S[b].ph = side_sum<1>(z * X[b].ph);
            S[b].vx = side_sum<1>(z * X[b].vx);
            S[b].vy = side_sum<1>(z * X[b].vy);
            S[b].om = side_sum<1>(z * X[b].om);
        }
    }
    Px[H] = S[0].x;
    Py[H] = S[0].y;
    if (s != 0 || !live) return;
    const float dxg = fabsf(Px[H] - c.goal[0]) - c.tol, dyg = fabsf(Py[H] - c.goal[1]) - c.tol;
    const float Ltarget = relu(dxg) * relu(dxg) + relu(dyg) * relu(dyg);
    const float Lrot = 1.0f - cosf(S[0].ph - c.goal[2]);
    float Ltraj = 0.0f;
    for (int kk = 1; kk <= H; ++kk) {
        Ltraj += smooth_abs(Px[kk - 1] - Px[kk], c.ea2) + smooth_abs(Py[kk - 1] - Py[kk], c.ea2);
        Ltraj += smooth_abs(Px[kk] - Px[H], c.ea2) + smooth_abs(Py[kk] - Py[H], c.ea2);
        Ltraj -= smooth_abs(Px[kk - 1] - Px[H], c.ea2) + smooth_abs(Py[kk - 1] - Py[H], c.ea2);
    }
    const float C = c.wt * Ltarget + c.wr * Lrot + c.wtr * Ltraj + c.wb * Lbound;
    cost[i] = C;
    if (status && !isfinite(C)) atomicOr(status, STAMP_STATUS_NONFINITE_COST);
}

// Reverse sweep of one packed lane; as rollout_adj_lane.
template <int B>
__device__ __forceinline__ void rollout_adj_packed(const SimConst& c, int N, const float* __restrict__ theta,
                                                   const float* __restrict__ tape, const TapeGeom& g,
                                                   const float* __restrict__ cost_bar, float cb_scalar,
                                                   float* __restrict__ grad, float* __restrict__ seg,
                                                   uint32_t* status, int64_t lane, float* tab) {
    const int64_t iw = lane / 4;
    const bool live = iw < N;
    const int i = live ? (int)iw : N - 1;
    const int s = (int)(lane % 4);
    const int64_t slot0 = ((int64_t)4 * i + s) * B;
    const uint32_t off = (uint32_t)(slot0 * 6);
    const int H = c.H, T = c.T;
    const int64_t stride = 6 * B * g.lanes;
    const int lw = (int)(lane & 63);
    phase_table(theta, N, i, s, H, tab, lw);

    float* seeds = tab + H * kPhaseFloats;
    float PHx, PHy, phT;
    {
        const float z = tab[(H - 1) * kPhaseFloats + lw];
        const float* e = tape + g.ends_off + (int64_t)(H - 1) * stride + slot0 * 6;
        PHx = side_sum<1>(z * e[0]);
        PHy = side_sum<1>(z * e[1]);
        phT = side_sum<1>(z * e[2]);
    }
    const float cb = cost_bar ? cost_bar[i] : cb_scalar;
    float xb, yb, phb;
    cost_seeds(
        c, H, cb,
        [&](int k, float& x, float& y) {
            const float* e = tape + (int64_t)phase_entry(g, k, T, H) * stride + slot0 * 6;
            x = e[0];
            y = e[1];
        },
        PHx, PHy, phT, seeds, lw, xb, yb, phb);
    Blk Ls[B];
#pragma unroll
    for (int b = 0; b < B; ++b) Ls[b].x = Ls[b].y = Ls[b].ph = Ls[b].vx = Ls[b].vy = Ls[b].om = 0.0f;
    Ls[0].x = xb;
    Ls[0].y = yb;
    Ls[0].ph = phb;

    Push p;
    side_frame(s, p);
    bool bad = false;
    int entry = phase_entry(g, H, T, H);  // of the phase's first step
    for (int kk = H - 1; kk >= 0; --kk) {
        entry -= g.ckpt == 0 ? phase_start(kk + 1, T, H) - phase_start(kk, T, H) : phase_segments(kk, T, H, g.ckpt);
        const int tk = phase_start(kk, T, H), tk1 = phase_start(kk + 1, T, H);
        const float invL = 1.0f / (float)(tk1 - tk);
        const float* pt = tab + kk * kPhaseFloats + lw;
        const float z = pt[0], o = pt[64], D = pt[128];
        Blk Xe[B], L[B];
        load_blks<B>(Xe, tape + g.ends_off + (int64_t)kk * stride, off);
        float zpb[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            zpb[b] = Ls[b].x * Xe[b].x + Ls[b].y * Xe[b].y + Ls[b].ph * Xe[b].ph + Ls[b].vx * Xe[b].vx +
                     Ls[b].vy * Xe[b].vy + Ls[b].om * Xe[b].om;
            L[b].x = z * Ls[b].x;
            L[b].y = z * Ls[b].y;
            L[b].ph = z * Ls[b].ph;
            L[b].vx = z * Ls[b].vx;
            L[b].vy = z * Ls[b].vy;
            L[b].om = z * Ls[b].om;
        }
        const float zb = blocks_sum<B>(zpb);
        const float ab = z * (zb - side_sum<1>(z * zb));  // softmax VJP
        Blk A;
        load_blk_at(A, tape + (int64_t)entry * stride, off);  // block 0's pose: the anchor
        Anchor an;
        phase_push(c, A.x, A.y, A.ph, o, D, p, an);
        float P0xb = 0.0f, P0yb = 0.0f, Vxb = 0.0f, Vyb = 0.0f;
        Profile prof;
        prof.reset(invL);
        if (g.ckpt == 0) {
            const float* base = tape + (int64_t)tk * stride;
            int j = tk1 - tk - 1;
            Blk XA[B], XB[B];
            load_blks<B>(XA, base + (int64_t)j * stride, off);
            load_blks<B>(XB, base + (int64_t)max(j - 1, 0) * stride, off);
            for (; j >= 1; j -= 2) {
                Blk X[B];
#pragma unroll
                for (int b = 0; b < B; ++b) X[b] = XA[b];
                load_blks<B>(XA, base + (int64_t)max(j - 2, 0) * stride, off);
                step_reverse_packed<B>(c, X, L, p, prof.at(j), P0xb, P0yb, Vxb, Vyb);
#pragma unroll
                for (int b = 0; b < B; ++b) X[b] = XB[b];
                load_blks<B>(XB, base + (int64_t)max(j - 3, 0) * stride, off);
                step_reverse_packed<B>(c, X, L, p, prof.at(j - 1), P0xb, P0yb, Vxb, Vyb);
            }
            if (j == 0) step_reverse_packed<B>(c, XA, L, p, prof.at(0), P0xb, P0yb, Vxb, Vyb);
        } else {
            const int nseg = (tk1 - tk + g.ckpt - 1) / g.ckpt;
            for (int q = nseg - 1; q >= 0; --q) {
                const int js = q * g.ckpt;
                const int je = min(js + g.ckpt, tk1 - tk);
                Blk X[B];
                load_blks<B>(X, tape + (int64_t)(entry + q) * stride, off);
                for (int j = js; j < je; ++j) {
                    if (live) store_blks<B>(X, seg + (int64_t)(j - js) * stride, off);
                    step_forward_packed<B>(c, X, p, prof.at(j));
                }
                for (int j = je - 1; j >= js; --j) {
                    if (live) load_blks<B>(X, seg + (int64_t)(j - js) * stride, off);
                    step_reverse_packed<B>(c, X, L, p, prof.at(j), P0xb, P0yb, Vxb, Vyb);
                }
            }
        }
        const float eAx = fmaf(an.cA, p.nx, -(an.sA * p.ny)), eAy = fmaf(an.sA, p.nx, an.cA * p.ny);
        const float Db = -fmaf(Vxb, eAx, Vyb * eAy);
        const float eAxb = -D * Vxb, eAyb = -D * Vyb;
        const float cAb = fmaf(eAxb, p.nx, eAyb * p.ny) + fmaf(P0xb, an.q0x, P0yb * an.q0y);
        const float sAb = fmaf(eAyb, p.nx, -(eAxb * p.ny)) + fmaf(P0yb, an.q0x, -(P0xb * an.q0y));
        const float q0xb = fmaf(an.cA, P0xb, an.sA * P0yb), q0yb = fmaf(an.cA, P0yb, -(an.sA * P0xb));
        const float ob = fmaf(q0xb, p.tx, q0yb * p.ty);
        const float Aphb = fmaf(an.cA, sAb, -(an.sA * cAb));
#pragma unroll
        for (int b = 0; b < B; ++b) {
            Ls[b].x = side_sum<1>(L[b].x);
            Ls[b].y = side_sum<1>(L[b].y);
            Ls[b].ph = side_sum<1>(L[b].ph);
            Ls[b].vx = side_sum<1>(L[b].vx);
            Ls[b].vy = side_sum<1>(L[b].vy);
            Ls[b].om = side_sum<1>(L[b].om);
        }
        const float Axs = side_sum<1>(P0xb), Ays = side_sum<1>(P0yb), Aphs = side_sum<1>(Aphb);
        const float obs = side_sum<1>(ob), Dbs = side_sum<1>(Db);
        const float Pxb = seeds[kk * kSeedFloats + lw], Pyb = seeds[kk * kSeedFloats + 64 + lw];
        if (c.per_phase) {
#pragma unroll
            for (int b = 0; b < B; ++b) Ls[b].x = Ls[b].y = Ls[b].ph = Ls[b].vx = Ls[b].vy = Ls[b].om = 0.0f;
            Ls[0].x = Pxb;
            Ls[0].y = Pyb;
        } else {
            Ls[0].x += Axs + Pxb;
            Ls[0].y += Ays + Pyb;
            Ls[0].ph += Aphs;
        }
        const float wb2 = 2.0f * cb * c.wb;
        const float obt = obs + wb2 * relu(fabsf(o) - c.omax) * copysignf(1.0f, o);
        const float Dbt = Dbs + wb2 * (relu(D - c.dmax) - relu(-D));
        if (live) {
            grad[(int64_t)(6 * kk + s) * N + i] = ab;
            if (s == 0) grad[(int64_t)(6 * kk + 4) * N + i] = obt;
            if (s == 1) grad[(int64_t)(6 * kk + 5) * N + i] = Dbt;
            bad = bad || !isfinite(ab) || !isfinite(obt) || !isfinite(Dbt);
        }
    }
    if (status && bad) atomicOr(status, STAMP_STATUS_NONFINITE_GRAD);
}

// The lanes a forward workgroup takes.  Workgroups go to the eight XCDs in turn,
// and each XCD has its own L2: where the tape's rows do not start at a cache
// line (96 B N bytes a row, B N no multiple of 4), two neighbours share a line
// between them, which then leaves two L2s in parts.  There each XCD takes a run of
// neighbours instead: N = 14 001, B = 3, packed 212 -> 149 us, N = 8 001, B = 3, block
// per lane 148 -> 112, N = 16 383, B = 2 143 -> 108.  The same above 57 344 blocks,
// where the rows come as fast as memory takes them (N = 16 384, B = 4 240 -> 229
// us); below that, aligned rows go as fast or faster in turn (N = 16 384, B = 3 173 us
// against 178, N = 12 288, B = 4 178 against 183).
constexpr int kXcdRunBlocks = 57344;
template <int B, int LANES>
__device__ __forceinline__ int64_t fwd_lane(int N) {
    uint32_t b = blockIdx.x;
    if ((B * N & 3) != 0 || B * N >= kXcdRunBlocks) {
        const uint32_t n = (uint32_t)(((int64_t)LANES * N + kRolloutBlock - 1) / kRolloutBlock), xcd = b & 7;
        b = xcd * (n >> 3) + min(xcd, n & 7) + (b >> 3);
    }
    return (int64_t)b * kRolloutBlock + threadIdx.x;
}

template <int B>
__global__ __launch_bounds__(kRolloutBlock) void k_rollout_fwd_packed(SimConst c, int N,
                                                                      const float* __restrict__ theta,
                                                                      float* __restrict__ cost,
                                                                      float* __restrict__ tape, TapeGeom g,
                                                                      uint32_t* status) {
    const int64_t lane = fwd_lane<B, 4>(N);
    extern __shared__ __align__(16) float lds[];
    rollout_fwd_packed<B>(c, N, theta, cost, tape, g, status, lane, lds);
}

template <int B>
__global__ __launch_bounds__(kRolloutBlock) void k_rollout_adj_packed(SimConst c, int N,
                                                                      const float* __restrict__ theta,
                                                                      const float* __restrict__ tape, TapeGeom g,
                                                                      const float* __restrict__ cost_bar,
                                                                      float cb_scalar, float* __restrict__ grad,
                                                                      float* __restrict__ seg, uint32_t* status) {
    const int64_t lane = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    extern __shared__ __align__(16) float lds[];
    rollout_adj_packed<B>(c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg, status, lane, lds);
}

// ---------------------------------------------------------------------------
template <int B>
__global__ __launch_bounds__(kRolloutBlock) void k_rollout_fwd(SimConst c, int N, const float* __restrict__ theta,
                                                               float* __restrict__ cost, float* __restrict__ tape,
                                                               TapeGeom g, uint32_t* status) {
    const int64_t lane = fwd_lane<B, Slots<B>::LANES>(N);
    extern __shared__ __align__(16) float lds[];
    rollout_fwd_lane<B>(c, N, theta, cost, tape, g, status, lane, lds);
}

template <int B>
__global__ __launch_bounds__(kRolloutBlock) void k_rollout_adj(SimConst c, int N, const float* __restrict__ theta,
                                                               const float* __restrict__ tape, TapeGeom g,
                                                               const float* __restrict__ cost_bar, float cb_scalar,
                                                               float* __restrict__ grad, float* __restrict__ seg,
                                                               uint32_t* status) {
    const int64_t lane = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    extern __shared__ __align__(16) float lds[];
    rollout_adj_lane<B>(c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg, status, lane, lds);
}

// ---------------------------------------------------------------------------
// Batched rollouts: one launch over the wave tiles of many problems.  Tile t is
// (problem p, first particle i0) and covers 64 lanes: 64 / (4 SL) particles
// (rollout_tile_particles); each wave takes tiles in a grid-stride loop.  The
// block count B of the problem selects the compiled body at run time.
template <int B, bool PK>
__device__ __forceinline__ void fwd_tile(const ProblemDesc& D, int i0, int l, const float* theta, float* cost,
                                         float* tape, uint32_t* status, float* lds) {
    const int64_t lane = (int64_t)(PK ? 4 : Slots<B>::LANES) * i0 + l;
    if constexpr (PK)
        rollout_fwd_packed<B>(D.c, D.N, theta + D.theta_off, cost + D.cost_off, tape ? tape + D.tape_off : nullptr,
                              D.g, status, lane, lds);
    else
        rollout_fwd_lane<B>(D.c, D.N, theta + D.theta_off, cost + D.cost_off, tape ? tape + D.tape_off : nullptr,
                            D.g, status, lane, lds);
}

template <int B, bool PK>
__device__ __forceinline__ void adj_tile(const ProblemDesc& D, int i0, int l, const float* theta, const float* tape,
                                         float cb_scalar, float* grad, float* seg, uint32_t* status, float* lds) {
    const int64_t lane = (int64_t)(PK ? 4 : Slots<B>::LANES) * i0 + l;
    if constexpr (PK)
        rollout_adj_packed<B>(D.c, D.N, theta + D.theta_off, tape + D.tape_off, D.g, nullptr, cb_scalar,
                              grad + D.theta_off, seg + D.seg_off, status, lane, lds);
    else
        rollout_adj_lane<B>(D.c, D.N, theta + D.theta_off, tape + D.tape_off, D.g, nullptr, cb_scalar,
                            grad + D.theta_off, seg + D.seg_off, status, lane, lds);
}

template <bool PK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PK ? 2 : 4))) void k_rollout_fwd_batched(const ProblemDesc* __restrict__ descs,
                                                             const int2* __restrict__ tiles, int ntiles,
                                                             const float* __restrict__ theta, float* __restrict__ cost,
                                                             float* __restrict__ tape, uint32_t* status,
                                                             int wave_floats) {
    const int waves = blockDim.x >> 6;
    // the wave index is uniform across the wave: readfirstlane lets the tile,
    // its problem descriptor and the scene constants live in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    extern __shared__ __align__(16) float lds_all[];
    float* lds = lds_all + wave * wave_floats;
    for (int t = blockIdx.x * waves + wave; t < ntiles; t += gridDim.x * waves) {
        const int2 tl = tiles[t];
        const ProblemDesc& D = descs[tl.x];
        switch (D.c.B) {
            case 1: fwd_tile<1, PK>(D, tl.y, l, theta, cost, tape, status, lds); break;
            case 2: fwd_tile<2, PK>(D, tl.y, l, theta, cost, tape, status, lds); break;
            case 3: fwd_tile<3, PK>(D, tl.y, l, theta, cost, tape, status, lds); break;
            default: fwd_tile<4, PK>(D, tl.y, l, theta, cost, tape, status, lds); break;
        }
    }
}

template <bool PK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PK ? 2 : 4))) void k_rollout_adj_batched(const ProblemDesc* __restrict__ descs,
                                                             const int2* __restrict__ tiles, int ntiles,
                                                             const float* __restrict__ theta,
                                                             const float* __restrict__ tape, float cb_scalar,
                                                             float* __restrict__ grad, float* __restrict__ seg,
                                                             uint32_t* status, int wave_floats) {
    const int waves = blockDim.x >> 6;
    // the wave index is uniform across the wave: readfirstlane lets the tile,
    // its problem descriptor and the scene constants live in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    extern __shared__ __align__(16) float lds_all[];
    float* lds = lds_all + wave * wave_floats;
    for (int t = blockIdx.x * waves + wave; t < ntiles; t += gridDim.x * waves) {
        const int2 tl = tiles[t];
        const ProblemDesc& D = descs[tl.x];
        switch (D.c.B) {
            case 1: adj_tile<1, PK>(D, tl.y, l, theta, tape, cb_scalar, grad, seg, status, lds); break;
            case 2: adj_tile<2, PK>(D, tl.y, l, theta, tape, cb_scalar, grad, seg, status, lds); break;
            case 3: adj_tile<3, PK>(D, tl.y, l, theta, tape, cb_scalar, grad, seg, status, lds); break;
            default: adj_tile<4, PK>(D, tl.y, l, theta, tape, cb_scalar, grad, seg, status, lds); break;
        }
    }
}

int rollout_tile_particles(int B, bool packed) { return packed ? 16 : 64 / (4 * (B == 1 ? 1 : (B == 2 ? 2 : 4))); }

// LDS of one rollout wave (floats): the phase table, and the packed forward's
// staging for B blocks (B = 0: none).  Sized at launch for the batch's largest
// H and B, so that the waves a CU holds are bound by registers.
static int rollout_lds_floats(int H, int B) { return H * kPhaseFloats + 64 * 6 * B; }

hipError_t launch_rollout_fwd_batched(const ProblemDesc* descs, const int2* tiles, int ntiles, int block,
                                      int grid, const float* theta, float* cost, float* tape, uint32_t* status,
                                      hipStream_t st, bool packed, int max_H, int max_B) {
    const int wf = rollout_lds_floats(max_H, packed ? max_B : 0);
    if (packed)
        hipLaunchKernelGGL(k_rollout_fwd_batched<true>, dim3(grid), dim3(block), (size_t)(block / 64) * wf * 4, st,
                           descs, tiles, ntiles, theta,
                           cost, tape, status, wf);
    else
        hipLaunchKernelGGL(k_rollout_fwd_batched<false>, dim3(grid), dim3(block), (size_t)(block / 64) * wf * 4, st,
                           descs, tiles, ntiles, theta,
                           cost, tape, status, wf);
    return hipGetLastError();
}

hipError_t launch_rollout_adj_batched(const ProblemDesc* descs, const int2* tiles, int ntiles, int block,
                                      int grid, const float* theta, const float* tape, float cb_scalar,
                                      float* grad, float* seg, uint32_t* status, hipStream_t st, bool packed,
                                      int max_H) {
    const int wf = adj_table_floats(max_H);
    if (packed)
        hipLaunchKernelGGL(k_rollout_adj_batched<true>, dim3(grid), dim3(block), (size_t)(block / 64) * wf * 4, st,
                           descs, tiles, ntiles, theta,
                           tape, cb_scalar, grad, seg, status, wf);
    else
        hipLaunchKernelGGL(k_rollout_adj_batched<false>, dim3(grid), dim3(block), (size_t)(block / 64) * wf * 4, st,
                           descs, tiles, ntiles, theta,
                           tape, cb_scalar, grad, seg, status, wf);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
static unsigned rollout_groups(int64_t lanes) { return (unsigned)((lanes + kRolloutBlock - 1) / kRolloutBlock); }

template <int B>
static hipError_t launch_fwd_b(const SimConst& c, int N, const float* theta, float* cost, float* tape,
                               const TapeGeom& g, uint32_t* status, hipStream_t st, bool packed) {
    // one block: both layouts are the same lanes; the block-per-lane kernel runs it
    if constexpr (B > 1)
        if (packed) {
            hipLaunchKernelGGL(k_rollout_fwd_packed<B>, dim3(rollout_groups((int64_t)4 * N)), dim3(kRolloutBlock),
                               rollout_lds_floats(c.H, B) * 4, st, c, N, theta, cost, tape, g, status);
            return hipGetLastError();
        }
    hipLaunchKernelGGL(k_rollout_fwd<B>, dim3(rollout_groups((int64_t)Slots<B>::LANES * N)), dim3(kRolloutBlock),
                       rollout_lds_floats(c.H, 0) * 4, st, c, N, theta, cost, tape, g, status);
    return hipGetLastError();
}

// Whether the split reverse sweep's workgroups (64 lanes and lds bytes each)
// are on the chip at once.  A second round of them costs as long as the first,
// while the waves of the whole-step sweep all fit: N = 4096, B = 3, H = 5 (1024
// workgroups, 54 KB with chunks of four steps) took 131 us in two rounds, 99
// whole-step, 93 with chunks of two steps (31 KB, one round).  That is the full
// tape's line; the checkpointed kernels take it too, where two rounds have not been
// measured (T = 400, K = 32, B = 1: one round at N = 4096 92 us, whole-step at 4097
// 223).  Where the states leave no room for the four-wave kernel (B = 3, K = 36..50)
// the two-wave one takes 178..211 us up to N = 1024, whole steps (K = 64) 292.
constexpr int64_t kLdsBytes = 160 * 1024;
static bool split_adjoint_pays(unsigned grid, int64_t lds) {
    return lds <= kLdsBytes && grid <= 256 * (kLdsBytes / lds);
}

template <int B>
static hipError_t launch_adj_b(const SimConst& c, int N, const float* theta, const float* tape,
                               const TapeGeom& g, const float* cost_bar, float cb_scalar, float* grad,
                               float* seg, uint32_t* status, hipStream_t st, bool packed) {
    if constexpr (B > 1)
        if (packed) {
            hipLaunchKernelGGL(k_rollout_adj_packed<B>, dim3(rollout_groups((int64_t)4 * N)), dim3(kRolloutBlock),
                               adj_table_floats(c.H) * 4, st, c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg,
                               status);
            return hipGetLastError();
        }
    const unsigned grid = rollout_groups((int64_t)Slots<B>::LANES * N);
    // LDS of the split sweeps: the table, two chunk buffers of 4 or 2 steps,
    // two buffers of a replayed segment's states
    const int64_t table = adj_table_floats(c.H) * 4, states = (int64_t)2 * g.ckpt * 6 * 64 * 4;
    const int64_t lds4 = table + 2 * pipe_buffer_floats<B, 4>() * 4, lds2 = table + 2 * pipe_buffer_floats<B, 2>() * 4;
    if (g.ckpt == 0 && split_adjoint_pays(grid, lds4))
        hipLaunchKernelGGL((k_rollout_adj_split<B, 4>), dim3(grid), dim3(64 * (1 + kPipeHelpers)), lds4, st, c, N,
                           theta, tape, g, cost_bar, cb_scalar, grad, status);
    else if (g.ckpt == 0 && split_adjoint_pays(grid, lds2))
        hipLaunchKernelGGL((k_rollout_adj_split<B, 2>), dim3(grid), dim3(64 * (1 + kPipeHelpers)), lds2, st, c, N,
                           theta, tape, g, cost_bar, cb_scalar, grad, status);
    else if (g.ckpt > 0 && split_adjoint_pays(grid, lds4 + states))
        hipLaunchKernelGGL((k_rollout_adj_ckpt<B, 4>), dim3(grid), dim3(64 * (2 + kPipeHelpers)), lds4 + states, st, c,
                           N, theta, tape, g, cost_bar, cb_scalar, grad, status);
    else if (g.ckpt > 0 && split_adjoint_pays(grid, table + states))
        hipLaunchKernelGGL(k_rollout_adj_replay<B>, dim3(grid), dim3(128), table + states, st, c, N, theta, tape, g,
                           cost_bar, cb_scalar, grad, status);
    else
        hipLaunchKernelGGL(k_rollout_adj<B>, dim3(grid), dim3(kRolloutBlock), adj_table_floats(c.H) * 4, st, c, N, theta, tape, g, cost_bar,
                           cb_scalar, grad, seg, status);
    return hipGetLastError();
}

hipError_t launch_rollout_fwd(const SimConst& c, int N, const float* theta, float* cost, float* tape,
                              const TapeGeom& g, uint32_t* status, hipStream_t st, bool packed) {
    switch (c.B) {
        case 1: return launch_fwd_b<1>(c, N, theta, cost, tape, g, status, st, packed);
        case 2: return launch_fwd_b<2>(c, N, theta, cost, tape, g, status, st, packed);
        case 3: return launch_fwd_b<3>(c, N, theta, cost, tape, g, status, st, packed);
        case 4: return launch_fwd_b<4>(c, N, theta, cost, tape, g, status, st, packed);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_rollout_adj(const SimConst& c, int N, const float* theta, const float* tape,
                              const TapeGeom& g, const float* cost_bar, float cb_scalar, float* grad,
                              float* seg, uint32_t* status, hipStream_t st, bool packed) {
    switch (c.B) {
        case 1: return launch_adj_b<1>(c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg, status, st, packed);
        case 2: return launch_adj_b<2>(c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg, status, st, packed);
        case 3: return launch_adj_b<3>(c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg, status, st, packed);
        case 4: return launch_adj_b<4>(c, N, theta, tape, g, cost_bar, cb_scalar, grad, seg, status, st, packed);
    }
    return hipErrorInvalidValue;
}

}  // namespace stamp
