// HIP kernels for gfx950 (CDNA4): trajectory generation, collision
// recognition and risk assessment of the multi-hypothesis criticality method
// (Sanchez Morales et al., IEEE IV 2019, Fig. 1: the three modules after
// street data processing, run in that order, each data-parallel inside).
#include "mhc_internal.h"

#include <algorithm>
#include <climits>
#include <math.h>
#include <mutex>

// The overlap tests combine their comparisons with bitwise & and | on bools
// on purpose: every comparison is evaluated and the results are merged as
// lane masks, with no branch per comparison.
#pragma clang diagnostic ignored "-Wbitwise-instead-of-logical"

namespace mhc {

// ===========================================================================
// K1: trajectory generation (Sec. IV-B) and probability normalisation
// (Sec. IV-D.1).
//
// Vehicles follow the Euler pose update of Sec. IV-B.1 with side slip 0 and
// no yaw acceleration: in step n the speed v_n, heading psi_n = psi0 + n*w*tau
// and acceleration give the displacement
//   dx_n = c(psi_n) v_n tau + c(psi_n) a_x tau^2/2 - s(psi_n) a_y tau^2/2
//   dy_n = s(psi_n) v_n tau + s(psi_n) a_x tau^2/2 + c(psi_n) a_y tau^2/2
// with a_x the acceleration cut so that the speed stops at 0 and
// a_y = v_n w. The speed of a constant acceleration with a stop at 0 has the
// closed form max(0, v0 + n a tau), so every step's displacement is
// independent: one wave integrates one trajectory, lane q computing step
// n0 + q (FP64, including its own sine/cosine), and the positions are the
// running sums of the displacements, formed by a wave-wide scan and carried
// from one 64-step chunk to the next. Pedestrians (Sec. IV-B.3) move by the
// constant displacement of their speed and heading each step.
// Poses are stored as FP32: float4 (x, y, cos psi, sin psi) for vehicles,
// float2 (x, y) for pedestrians, layout [t][position], slot t = step t+1. An
// object's trajectories sit in the order of traj_at, which keeps neighbours
// of the control grid together; every LEAF of them (one workgroup) gets the
// box of its positions at every step, from which the collision kernel tells
// which steps of a block of trajectory pairs can hold an overlap at all.
// ===========================================================================

// The integer summand of one colliding combination of probability p: p itself
// in units of 2^-62 (EXCLUSIVE reading: an object's trajectories exclude one
// another, so the q of an object is a sum of p), or -log(1 - p), capped at
// 64, in units of 2^-56 (INDEPENDENT reading: q = 1 - prod(1 - p) =
// 1 - exp(-sum of -log(1 - p))).
__device__ __forceinline__ unsigned long long fixed_term(int risk, double p)
{
    if (risk == RISK_EXCLUSIVE) return __double2ull_rn(p * kQScale);
    return __double2ull_rn(fmin(-log1p(-p), kLCap) * kLScale);
}

// q from its integer sum, under the object's reading.
__device__ __forceinline__ double q_of(int risk, unsigned long long v)
{
    if (risk == RISK_EXCLUSIVE) return fmin((double)v * kQInvScale, 1.0);
    return -expm1(-(double)v * kLInvScale);
}

// A double moved across lanes by the DPP control CTRL in the rows of
// ROW_MASK; a lane without a source (or outside those rows) gets `old`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double x, double old)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(x), CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(x), CTRL, ROW_MASK, 0xF, false);
    return __hiloint2double(hi, lo);
}

// The steps of a wave-wide inclusive scan over 64 lanes without LDS: shifts
// by 1, 2, 4 and 8 lanes within each row of 16 (row_shr), then lane 15 of
// rows 0 and 2 into rows 1 and 3 (row_bcast:15), then lane 31 into rows 2 and
// 3 (row_bcast:31). After step k every lane holds the combination of the
// lanes below it up to the step's reach, so after the six it holds lanes
// 0..l. DPP controls of the GFX9 family.
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143, kDppWaveShr1 = 0x138;

// Inclusive prefix sum over the 64 lanes of a wave (lane l gets the sum of
// lanes 0..l).
__device__ __forceinline__ double scan_add(double v, int lane)
{
    (void)lane;
    v += dpp_move<kDppRowShr1, 0xF>(v, 0.0);
    v += dpp_move<kDppRowShr2, 0xF>(v, 0.0);
    v += dpp_move<kDppRowShr4, 0xF>(v, 0.0);
    v += dpp_move<kDppRowShr8, 0xF>(v, 0.0);
    v += dpp_move<kDppRowBcast15, 0xA>(v, 0.0);
    v += dpp_move<kDppRowBcast31, 0xC>(v, 0.0);
    return v;
}

// The same of an int.
__device__ __forceinline__ int scan_add_int(int v)
{
#define MHC_SCAN_STEP(CTRL, ROWS) v += __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false)
    MHC_SCAN_STEP(kDppRowShr1, 0xF);
    MHC_SCAN_STEP(kDppRowShr2, 0xF);
    MHC_SCAN_STEP(kDppRowShr4, 0xF);
    MHC_SCAN_STEP(kDppRowShr8, 0xF);
    MHC_SCAN_STEP(kDppRowBcast15, 0xA);
    MHC_SCAN_STEP(kDppRowBcast31, 0xC);
#undef MHC_SCAN_STEP
    return v;
}

// The value of the lane below (lane 0 gets `first`).
__device__ __forceinline__ double lane_below(double x, double first) { return dpp_move<kDppWaveShr1, 0xF>(x, first); }

// The sum of v over the first WG threads of a workgroup, in a fixed order: each
// wave's sum by the DPP scan (its lane 63), then the waves' sums in wave order.
// Every thread of the workgroup must call it; the result is valid in every
// thread.
__device__ __forceinline__ double block_sum(double v, double *ws)
{
    const int lane = (int)(threadIdx.x & (WAVE - 1)), w = (int)(threadIdx.x / WAVE);
    v = scan_add(v, lane);
    if (lane == WAVE - 1 && w < WG / WAVE) ws[w] = v;
    __syncthreads();
    double s = ws[0];
#pragma unroll
    for (int k = 1; k < WG / WAVE; ++k) s += ws[k];
    return s;
}

// Thread tid < 256 adds the scores tid, tid + 256, ... in ascending order, eight
// loads in flight at a time, then the workgroup adds the 256 partial sums in a
// fixed order (block_sum): the order depends on T only.
__device__ void normalise_probabilities(const DObj &o, int obj, const double *__restrict__ vals,
                                        double *__restrict__ p, unsigned long long *__restrict__ pfix,
                                        unsigned long long *__restrict__ done)
{
    __shared__ double red[WG / WAVE];
    const int tid = threadIdx.x;
    const double *__restrict__ sc = vals + o.score_off;
    double part = 0.0;
    if (o.score_off >= 0 && tid < WG) {
        for (int base = 0; base < o.T; base += 8 * WG) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int idx = base + k * WG + tid;
                v[k] = idx < o.T ? sc[idx] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (base + k * WG + tid < o.T) part += v[k];
        }
    }
    const double total = block_sum(part, red);
    if (tid >= WG) return;
    for (int base = 0; base < o.T; base += 8 * WG) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int idx = base + k * WG + tid;
            v[k] = (o.score_off >= 0 && idx < o.T) ? sc[idx] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int idx = base + k * WG + tid;
            if (idx < o.T) {
                const double pk = o.score_off >= 0 ? v[k] / total : 1.0 / (double)o.T;
                p[o.traj_off + idx] = pk;
                pfix[o.traj_off + idx] = fixed_term(o.risk, pk);
            }
        }
    }
    // the object's completion counter of the risk kernel starts from zero
    // (each trajectory's wave clears its row of the q accumulators)
    if (tid == 0) done[obj] = 0ull;
}

// The box that a leaf's shapes cover at one step, as (x_min, x_max, y_min,
// y_max): the bounds of each trajectory's shape at its pose, of half length hl
// along the heading and half width hw across it (circles: the radius in both).
// A pose that an overlap test could not be trusted to separate (not finite, or
// so far out that its products overflow) makes the box infinite, so that no
// test of the leaf is left out at that step.
__device__ __forceinline__ float4 box_none() { return make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY); }

__device__ __forceinline__ float4 box_join(const float4 a, const float4 b)
{
    return make_float4(fminf(a.x, b.x), fmaxf(a.y, b.y), fminf(a.z, b.z), fmaxf(a.w, b.w));
}

__device__ __forceinline__ float4 box_of(float x, float y, float c, float s, float hl, float hw)
{
    const bool ok = (fabsf(x) <= kBoxMax) & (fabsf(y) <= kBoxMax) & (fabsf(c) <= 2.0f) & (fabsf(s) <= 2.0f);
    const float hx = fmaf(hl, fabsf(c), hw * fabsf(s)), hy = fmaf(hl, fabsf(s), hw * fabsf(c));
    return ok ? make_float4(x - hx, x + hx, y - hy, y + hy) : make_float4(-INFINITY, INFINITY, -INFINITY, INFINITY);
}

// Writes the boxes of the workgroup's leaf for steps n0 .. n0 + 63: every wave
// brings the box of its trajectory's pose at step n0 + lane (box_none where it
// has none), the first wave joins them. Every thread of the workgroup calls it.
__device__ __forceinline__ void store_leaf_boxes(char *__restrict__ poses, const DObj &o, int leaf, int n0, float4 mine)
{
    __shared__ float4 box[2][LEAF][WAVE];
    const int lane = (int)(threadIdx.x & (WAVE - 1)), w = (int)(threadIdx.x / WAVE);
    const int buf = (n0 / WAVE) & 1;   // the next chunk's boxes may be written while these are read
    box[buf][w][lane] = mine;
    __syncthreads();
    if (w == 0 && n0 + lane < o.H) {
        float4 b = box[buf][0][lane];
#pragma unroll
        for (int k = 1; k < LEAF; ++k) b = box_join(b, box[buf][k][lane]);
        reinterpret_cast<float4 *>(poses + o.box_off)[(size_t)leaf * o.H + n0 + lane] = b;
    }
}

// Workgroup wg writes its share, `per` 16-byte words, of -1 (no collision) over
// the n first-hit entries: the collision kernel stores colliding pairs only. The
// words go past the caches: on the 40-object stress scene, whose 1.64 GB of
// first hits are what the trajectory kernel's time goes to, 380 us (4.3 TB/s)
// against 390, and 19 against 23 us for the risk kernel after it.
__device__ __forceinline__ void clear_hits(int16_t *__restrict__ hits, int64_t n, int64_t per, int64_t wg)
{
    typedef uint32_t words __attribute__((ext_vector_type(4)));
    // entries before the first 16-byte boundary, 16-byte stores, the rest
    const int64_t head = min(n, (int64_t)((16 - (reinterpret_cast<uintptr_t>(hits) & 15)) & 15) / 2);
    const int64_t wide = (n - head) / 8;
    const int64_t k1 = min(wide, (wg + 1) * per);
    words *h16 = reinterpret_cast<words *>(hits + head);
    for (int64_t k = wg * per + threadIdx.x; k < k1; k += blockDim.x)
        __builtin_nontemporal_store(words{~0u, ~0u, ~0u, ~0u}, &h16[k]);
    if (wg == 0) {
        const int t = (int)threadIdx.x;
        if (t < head) hits[t] = -1;
        if (head + wide * 8 + t < n && t < 8) hits[head + wide * 8 + t] = -1;
    }
}

// Vehicle trajectory i on the linear one-track model (Sec. IV-B.1): side slip
// beta and yaw rate r obey
//   beta' = -(cf+cr)/(m v) beta + ((cr lr - cf lf)/(m v^2) - 1) r + cf/(m v) delta
//   r'    = (cr lr - cf lf)/Iz beta - (cf lf^2 + cr lr^2)/(Iz v) r + cf lf/Iz delta
// for the constant steering angle delta = w[l], integrated with the paper's
// Euler pose update (accelerations a_x, a_y in the vehicle frame from step
// n, the speed stopping at 0). Where the explicit step is unstable (an
// eigenvalue of I + tau A(v_n) of modulus >= 1, tested by the Jury
// conditions) the lateral state takes the steady state at v_{n+1} instead:
//   r = v delta / (L (1 + K v^2)), beta = delta (lr/L - m lf v^2/(cr L^2)) / (1 + K v^2),
// L = lf + lr, K = m (lr cr - lf cf) / (L^2 cf cr). FP64; poses stored as
// FP32 (x, y, cos psi, sin psi), [t][position].
//
// Evaluation: one wave per trajectory, a lane per step, chunks of 64 steps
// with the state carried across chunks. The speed has a closed form,
// v_n = max(v_0 + n a tau, 0), and it alone decides each step's
// update of s = (beta, r): an explicit Euler step s_{n+1} = M_n s_n + c_n
// where that step is stable, else the steady state of the speed reached,
// s_{n+1} = s*(v_{n+1}) (M_n = 0). These affine maps compose, so an
// inclusive scan over the lanes gives every s_n of the chunk at once; the
// rates of step n follow from s_n and s_{n+1} as in the serial update, and
// the heading and the position are prefix sums of the per-step increments.
// Only the order of the additions differs from the serial recursion.


__device__ void one_track_wave(const DObj &o, const double *__restrict__ vals, char *__restrict__ poses, int k, int l,
                               int pos, int leaf, bool exists, int lane)
{
    const double cf = o.params[0], cr = o.params[1], lf = o.params[2], lr = o.params[3];
    const double m = o.params[4], Iz = o.params[5];
    const double L = lf + lr;
    const double K = m * (lr * cr - lf * cf) / (L * L * cf * cr);
    const double cd = cr * lr - cf * lf;
    const double cq = cf * lf * lf + cr * lr * lr;
    // the model's coefficients without their speed factors
    const double kb = (cf + cr) / m, kc = cd / m, kf = cf / m;       // beta'
    const double kcz = cd / Iz, kq = cq / Iz, kfz = cf * lf / Iz;   // r'
    const double lr_L = lr / L, mlf_crL2 = m * lf / (cr * L * L);    // steady state
    const double accel = vals[o.u_off + k];
    const double delta = vals[o.w_off + l];
    const double tau = o.tau, h2 = tau * tau / 2.0, at = accel * tau;
    // state at the chunk's first step
    double cx = o.x, cy = o.y, cpsi = o.heading, cbeta = 0.0, crate = 0.0, csp, ccp;
    sincos(cpsi, &csp, &ccp);
    for (int n0 = 0; n0 < o.H; n0 += 64) {
        const int n = n0 + lane;
        const bool active = n < o.H && exists;
        const double v = fmax(o.speed + (double)n * at, 0.0);
        double vdot = accel, v1 = v + at;
        if (v1 < 0.0) {
            vdot = -v / tau;
            v1 = 0.0;
        }
        bool stable = false;
        const double iv = v > 0.0 ? 1.0 / v : 0.0;
        double a11 = 1.0, a12 = 0.0, a21 = 0.0, a22 = 1.0, b1 = 0.0, b2 = 0.0;  // identity past the horizon
        if (active) {
            if (v > 0.0) {
                const double m11 = 1.0 - tau * kb * iv, m12 = tau * (kc * iv * iv - 1.0);
                const double m21 = tau * kcz, m22 = 1.0 - tau * kq * iv;
                const double tr = m11 + m22, det = m11 * m22 - m12 * m21;
                stable = det < 1.0 && tr < 1.0 + det && tr > -(1.0 + det);
                if (stable) {
                    a11 = m11;
                    a12 = m12;
                    a21 = m21;
                    a22 = m22;
                    b1 = tau * kf * iv * delta;
                    b2 = tau * kfz * delta;
                }
            }
            if (!stable) {
                const double g = 1.0 + K * v1 * v1;
                a11 = a12 = a21 = a22 = 0.0;
                b1 = delta * (lr_L - mlf_crL2 * v1 * v1) / g;
                b2 = v1 * delta / (L * g);
            }
        }
        // lane n: the composition f_n o ... o f_{n0}; (A, b) o (P, q) = (AP, Aq + b),
        // in the steps of scan_add (a lane without a source composes with the
        // identity, which leaves its map as it is)
        auto compose = [&](double p11, double p12, double p21, double p22, double q1, double q2) {
            const double n11 = a11 * p11 + a12 * p21, n12 = a11 * p12 + a12 * p22;
            const double n21 = a21 * p11 + a22 * p21, n22 = a21 * p12 + a22 * p22;
            const double nb1 = a11 * q1 + a12 * q2 + b1, nb2 = a21 * q1 + a22 * q2 + b2;
            a11 = n11;
            a12 = n12;
            a21 = n21;
            a22 = n22;
            b1 = nb1;
            b2 = nb2;
        };
#define MHC_COMPOSE_STEP(CTRL, ROWS)                                                                           \
    compose(dpp_move<CTRL, ROWS>(a11, 1.0), dpp_move<CTRL, ROWS>(a12, 0.0), dpp_move<CTRL, ROWS>(a21, 0.0), \
            dpp_move<CTRL, ROWS>(a22, 1.0), dpp_move<CTRL, ROWS>(b1, 0.0), dpp_move<CTRL, ROWS>(b2, 0.0))
        MHC_COMPOSE_STEP(kDppRowShr1, 0xF);
        MHC_COMPOSE_STEP(kDppRowShr2, 0xF);
        MHC_COMPOSE_STEP(kDppRowShr4, 0xF);
        MHC_COMPOSE_STEP(kDppRowShr8, 0xF);
        MHC_COMPOSE_STEP(kDppRowBcast15, 0xA);
        MHC_COMPOSE_STEP(kDppRowBcast31, 0xC);
#undef MHC_COMPOSE_STEP
        // (beta, r) after step n, and before it (the previous lane's, or the carry)
        const double beta1 = a11 * cbeta + a12 * crate + b1;
        const double r1 = a21 * cbeta + a22 * crate + b2;
        const double beta = lane_below(beta1, cbeta), r = lane_below(r1, crate);
        double beta_dot, r_dot;
        if (stable) {
            beta_dot = -kb * iv * beta + (kc * iv * iv - 1.0) * r + kf * iv * delta;
            r_dot = kcz * beta - kq * iv * r + kfz * delta;
        } else {
            beta_dot = (beta1 - beta) / tau;
            r_dot = (r1 - r) / tau;
        }
        // heading after step n; the step itself turns with the heading before it
        const double psi1 = cpsi + scan_add(active ? r * tau + r_dot * h2 : 0.0, lane);
        double sp1, cp1;
        sincos(psi1, &sp1, &cp1);
        const double sp = lane_below(sp1, csp), cp = lane_below(cp1, ccp);
        double sb, cb;
        sincos(beta, &sb, &cb);
        const double spb = sp * cb + cp * sb, cpb = cp * cb - sp * sb;   // psi + beta
        const double ax = cb * vdot - sb * v * (beta_dot + r);
        const double ay = sb * vdot + cb * v * (beta_dot + r);
        const double x1 = cx + scan_add(active ? cpb * v * tau + cp * ax * h2 - sp * ay * h2 : 0.0, lane);
        const double y1 = cy + scan_add(active ? spb * v * tau + sp * ax * h2 + cp * ay * h2 : 0.0, lane);
        const float4 P = make_float4((float)x1, (float)y1, (float)cp1, (float)sp1);
        if (active) reinterpret_cast<float4 *>(poses + o.pose_off)[(size_t)n * o.T + pos] = P;
        if (o.box_off >= 0) store_leaf_boxes(poses, o, leaf, n0, active ? box_of(P.x, P.y, P.z, P.w, o.hl, o.hw) : box_none());
        cx = __shfl(x1, 63, 64);
        cy = __shfl(y1, 63, 64);
        cpsi = __shfl(psi1, 63, 64);
        csp = __shfl(sp1, 63, 64);
        ccp = __shfl(cp1, 63, 64);
        cbeta = __shfl(beta1, 63, 64);
        crate = __shfl(r1, 63, 64);
    }
}

// Grid: y = object; x = 0 is the object's probability normalisation (the
// longest block for large T, so it is dispatched first), x >= 1 are
// trajectory blocks of K1_TPB trajectories, one wave each.
// ONE_TRACK: whether the instance carries the one-track model's scan, whose
// FP64 state needs far more registers (129 VGPRs against the kinematic
// instance's 79); launches without one-track vehicles use the lighter instance,
// which also fits beside a running collision kernel on a shared GPU.
// For time-resolved scenes, trajectory block c also zeroes the c-th stretch
// of K1_TPB * W * H entries of the object's per-slot q sums. Where the launch
// asks for first hits, every workgroup writes its share of -1 over them.
template <bool ONE_TRACK>
__global__ __launch_bounds__(K1_WG) void k1_trajgen(const DObj *__restrict__ objs, const double *__restrict__ vals,
                                                 char *__restrict__ poses, double *__restrict__ p,
                                                 unsigned long long *__restrict__ pfix,
                                                 unsigned long long *__restrict__ qacc, unsigned long long *__restrict__ done,
                                                 unsigned long long *__restrict__ hist, const int2 *__restrict__ rows,
                                                 int16_t *__restrict__ hits, int64_t n_hits, int64_t hits_per_wg)
{
    if (hits) clear_hits(hits, n_hits, hits_per_wg, (int64_t)blockIdx.y * gridDim.x + blockIdx.x);
    // the row's object and the block of that object this workgroup is
    int obj = (int)blockIdx.y, xb = (int)blockIdx.x;
    if (rows) {
        const int2 r = rows[blockIdx.y];
        obj = r.x;
        xb += r.y;
    }
    const DObj o = objs[obj];
    if (xb == 0) {
        normalise_probabilities(o, obj, vals, p, pfix, done);
        return;
    }
    if (o.timeline) {
        const int64_t per = (int64_t)K1_TPB * o.tl_w * o.H;
        const int64_t total = (int64_t)o.T * o.tl_w * o.H;
        const int64_t lo = ((int64_t)xb - 1) * per;
        const int64_t hi = min(total, lo + per);
        // 16-byte stores: hist_off, the stretch and the total are even
        ulonglong2 *h2 = reinterpret_cast<ulonglong2 *>(hist + o.hist_off);
        for (int64_t k = lo / 2 + (int64_t)threadIdx.x; k < hi / 2; k += K1_WG) h2[k] = make_ulonglong2(0ull, 0ull);
    }
    const int lane = threadIdx.x & 63;
    const int leaf = xb - 1;
    if (leaf * LEAF >= o.T) return;  // whole workgroup
    // the trajectory of this wave's position; a wave past the last one keeps
    // step with the workgroup and writes nothing
    const int pos = leaf * LEAF + (int)(threadIdx.x >> 6);
    const bool exists = pos < o.T;
    int k, l;
    controls_at(min(pos, o.T - 1), o.n_u, o.n_w, o.strip, &k, &l);
    const int i = k * o.n_w + l;
    // this trajectory's row of the integer q accumulators starts from zero
    if (exists)
        for (int b = lane; b < o.n_scene_obj; b += 64) qacc[o.q_row + (int64_t)i * o.n_scene_obj + b] = 0ull;
    if constexpr (ONE_TRACK) {
        if (o.model == MODEL_ONE_TRACK) {
            one_track_wave(o, vals, poses, k, l, pos, leaf, exists, lane);
            return;
        }
    }
    const double tau = o.tau;
    const double half_tau2 = tau * tau / 2.0;
    const int H = o.H;
    const bool vehicle = o.kind == KIND_VEHICLE;
    const double u = vals[o.u_off + k];
    const double w = vals[o.w_off + l];
    // pedestrians: kinematic model (speed u, heading offset w) or the
    // acceleration model (acceleration u, absolute heading w, speed clamped
    // to [0, v_max]: after the first step v_n = clamp(v_1 + (n-1) u tau))
    const bool ped_accel = o.model == MODEL_PED_ACCEL;
    double ped_c = 0.0, ped_s = 0.0;
    if (!vehicle) sincos(ped_accel ? w : o.heading + w, &ped_s, &ped_c);
    const double v_max = o.params[0];
    const double v_first = ped_accel ? fmin(fmax(o.speed + u * tau, 0.0), v_max) : 0.0;
    double cx = o.x, cy = o.y;
    for (int n0 = 0; n0 < H; n0 += 64) {
        const int n = n0 + lane;
        const bool active = n < H && exists;
        double dx = 0.0, dy = 0.0;
        float c_next = 1.f, s_next = 0.f;   // circles: bounds hl by hw
        if (active) {
            if (vehicle) {
                const double wt = w * tau;
                double sn, cn, s1, c1;
                sincos(o.heading + (double)n * wt, &sn, &cn);
                sincos(o.heading + (double)(n + 1) * wt, &s1, &c1);
                const double at = u * tau;
                double v = o.speed + (double)n * at;
                const double v_next = o.speed + (double)(n + 1) * at;
                double ax = u;
                if (v_next < 0.0) {
                    if (v <= 0.0) {
                        v = 0.0;
                        ax = 0.0;
                    } else {
                        ax = -v / tau;
                    }
                }
                const double ay = v * w;
                dx = cn * v * tau + cn * ax * half_tau2 - sn * ay * half_tau2;
                dy = sn * v * tau + sn * ax * half_tau2 + cn * ay * half_tau2;
                c_next = (float)c1;
                s_next = (float)s1;
            } else if (ped_accel) {
                // step n -> n+1 moves by the mean of the two speeds
                const double vn = n == 0 ? o.speed : fmin(fmax(v_first + (double)(n - 1) * u * tau, 0.0), v_max);
                const double vn1 = fmin(fmax(v_first + (double)n * u * tau, 0.0), v_max);
                const double dist = (vn + vn1) * (tau / 2.0);
                dx = ped_c * dist;
                dy = ped_s * dist;
            } else {
                dx = ped_c * u * tau;
                dy = ped_s * u * tau;
            }
        }
        dx = scan_add(dx, lane);
        dy = scan_add(dy, lane);
        const double x = cx + dx, y = cy + dy;
        if (active) {
            const size_t k = (size_t)n * o.T + pos;
            if (vehicle)
                reinterpret_cast<float4 *>(poses + o.pose_off)[k] = make_float4((float)x, (float)y, c_next, s_next);
            else
                reinterpret_cast<float2 *>(poses + o.pose_off)[k] = make_float2((float)x, (float)y);
        }
        if (o.box_off >= 0)
            store_leaf_boxes(poses, o, leaf, n0, active ? box_of((float)x, (float)y, c_next, s_next, o.hl, o.hw) : box_none());
        cx = __shfl(x, 63, 64);
        cy = __shfl(y, 63, 64);
    }
}

// ===========================================================================
// K2: collision recognition (Sec. IV-C).
//
// Every trajectory pair of every object pair is decided at every step, most of
// them together: at a step at which the boxes of two leaves of trajectories lie
// apart, no pair of theirs overlaps. What is left is tested in units, item rows
// by item columns of one object pair, an item being an RI x RJ micro-tile of
// trajectory pairs (of neighbouring positions); the steps of an item go from
// later to earlier, and the earliest overlap of a pair is kept in LDS. Tests are
// exact closed-shape
// tests in FP32:
//   rectangle-rectangle: separating axes u_P, v_P, u_Q, v_Q; the projected
//     half extents use |cos(psi_Q - psi_P)| and |sin(psi_Q - psi_P)|;
//   rectangle-circle: distance from the centre to the rectangle <= r;
//   circle-circle: centre distance <= r_P + r_Q.
// The point-in-polygon mode instead tests the four corners of each rectangle
// against the other rectangle (the paper's test, both ways).
// ===========================================================================


// A vehicle pose (x, y, cos, sin) in its own frame: K = (x cos + y sin,
// y cos - x sin) is its centre there, and (K_x, K_y, cos, sin) is what the
// rectangle tests take for the rectangle they measure in its frame.
__device__ __forceinline__ float4 rect_frame(const float4 P)
{
    return make_float4(fmaf(P.x, P.z, P.y * P.w), fmaf(P.y, P.z, -(P.x * P.w)), P.z, P.w);
}

// Which pose a test takes in its own frame: neither, a's or b's.
struct PrepNone {
    template <class P> __device__ static __forceinline__ P prep_a(const P p) { return p; }
    template <class P> __device__ static __forceinline__ P prep_b(const P p) { return p; }
};
struct PrepA : PrepNone {
    __device__ static __forceinline__ float4 prep_a(const float4 p) { return rect_frame(p); }
};
struct PrepB : PrepNone {
    __device__ static __forceinline__ float4 prep_b(const float4 p) { return rect_frame(p); }
};

// Rectangle-rectangle (separating axes). With C = u_P.u_Q and S = v_P.u_Q
// (so u_P = C u_Q - S v_Q, v_P = S u_Q + C v_Q) and d = c_Q - c_P, the
// rectangles overlap iff
//   |d.u_P| <= lP + lQ|C| + wQ|S|,   |d.v_P| <= wP + lQ|S| + wQ|C|,
//   |d.u_Q| <= lQ + lP|C| + wP|S|,   |d.v_Q| <= wQ + lP|S| + wP|C|.
// Q's pose comes in its own frame (rect_frame: K = c_Q there, formed once per
// pose and step), so d.u_Q = K.x - (x_P cos_Q + y_P sin_Q) and d.v_Q = K.y - (y_P cos_Q - x_P
// sin_Q) are two FMA chains each, and d.u_P, d.v_P follow from them by the
// rotation (C, S): 25 VALU per test.
struct CheckVV : PrepB {
    float lP, wP, lQ, wQ;
    __device__ __forceinline__ CheckVV(const DPair &p) : lP(p.la), wP(p.wa), lQ(p.lb), wQ(p.wb) {}
    __device__ __forceinline__ bool operator()(const float4 P, const float4 Qk) const
    {
        const float C = fmaf(P.z, Qk.z, P.w * Qk.w);    // u_P . u_Q = v_P . v_Q
        const float S = fmaf(P.z, Qk.w, -(P.w * Qk.z)); // v_P . u_Q = -u_P . v_Q
        const float aC = fabsf(C), aS = fabsf(S);
        const float p3 = fmaf(-P.x, Qk.z, fmaf(-P.y, Qk.w, Qk.x));  // d . u_Q
        const float p4 = fmaf(-P.y, Qk.z, fmaf(P.x, Qk.w, Qk.y));   // d . v_Q
        const float p1 = fmaf(C, p3, -(S * p4));                     // d . u_P
        const float p2 = fmaf(S, p3, C * p4);                        // d . v_P
        const float r1 = fmaf(lQ, aC, fmaf(wQ, aS, lP));
        const float r2 = fmaf(lQ, aS, fmaf(wQ, aC, wP));
        const float r3 = fmaf(lP, aC, fmaf(wP, aS, lQ));
        const float r4 = fmaf(lP, aS, fmaf(wP, aC, wQ));
        return (fabsf(p1) <= r1) & (fabsf(p2) <= r2) & (fabsf(p3) <= r3) & (fabsf(p4) <= r4);
    }
};

// Point-in-polygon both ways for two rectangles. A corner of Q is
// c_Q + al*lQ*u_Q + be*wQ*v_Q (al, be = +-1); in P's frame it sits at
//   x = d.u_P + al*lQ*C - be*wQ*S,   y = d.v_P + al*lQ*S + be*wQ*C
// (C = u_P.u_Q, S = v_P.u_Q, d = c_Q - c_P) and lies in the closed P iff
// |x| <= lP and |y| <= wP. The corners of P in Q's frame follow with the roles
// swapped; flipping both signs of a corner leaves |x| and |y| unchanged, so
// they are (d.u_Q + al*lP*C + be*wP*S, d.v_Q - al*lP*S + be*wP*C).
// Q's pose comes in its own frame and the projections are formed as in the
// separating-axes test.
struct CheckVVPip : PrepB {
    float lP, wP, lQ, wQ;
    __device__ __forceinline__ CheckVVPip(const DPair &p) : lP(p.la), wP(p.wa), lQ(p.lb), wQ(p.wb) {}
    __device__ __forceinline__ bool operator()(const float4 P, const float4 Qk) const
    {
        const float C = fmaf(P.z, Qk.z, P.w * Qk.w);
        const float S = fmaf(P.z, Qk.w, -(P.w * Qk.z));
        const float p3 = fmaf(-P.x, Qk.z, fmaf(-P.y, Qk.w, Qk.x));  // d . u_Q
        const float p4 = fmaf(-P.y, Qk.z, fmaf(P.x, Qk.w, Qk.y));   // d . v_Q
        const float p1 = fmaf(C, p3, -(S * p4));                     // d . u_P
        const float p2 = fmaf(S, p3, C * p4);                        // d . v_P
        // Q's corners in P: (p1 +- g, p2 +- k) and (p1 +- h, p2 +- m), signs paired
        const float wQS = wQ * S, wQC = wQ * C;
        const float g = fmaf(lQ, C, -wQS), h = fmaf(lQ, C, wQS);
        const float k = fmaf(lQ, S, wQC), m = fmaf(lQ, S, -wQC);
        const bool q_in_p = ((fabsf(p1 + g) <= lP) & (fabsf(p2 + k) <= wP)) |
                            ((fabsf(p1 - g) <= lP) & (fabsf(p2 - k) <= wP)) |
                            ((fabsf(p1 + h) <= lP) & (fabsf(p2 + m) <= wP)) |
                            ((fabsf(p1 - h) <= lP) & (fabsf(p2 - m) <= wP));
        // P's corners in Q: (p3 +- g2, p4 -+ k2) and (p3 +- h2, p4 -+ m2)
        const float wPS = wP * S, wPC = wP * C;
        const float g2 = fmaf(lP, C, wPS), h2 = fmaf(lP, C, -wPS);
        const float k2 = fmaf(lP, S, -wPC), m2 = fmaf(lP, S, wPC);
        const bool p_in_q = ((fabsf(p3 + g2) <= lQ) & (fabsf(p4 - k2) <= wQ)) |
                            ((fabsf(p3 - g2) <= lQ) & (fabsf(p4 + k2) <= wQ)) |
                            ((fabsf(p3 + h2) <= lQ) & (fabsf(p4 - m2) <= wQ)) |
                            ((fabsf(p3 - h2) <= lQ) & (fabsf(p4 + m2) <= wQ));
        return q_in_p | p_in_q;
    }
};

// Rectangle-circle: the circle centre Q in P's frame is (lam, mu) =
// ((Q - c_P) . u_P, (Q - c_P) . v_P), and the two overlap iff the distance
// from Q to the rectangle, sqrt(max(|lam| - l, 0)^2 + max(|mu| - w, 0)^2), is
// at most r. The rectangle's pose comes in its own frame (rect_frame): K = (x_P cos + y_P sin, y_P cos - x_P sin) is c_P there, so
//   (lam, mu) = (x_Q cos + y_Q sin - K.x, y_Q cos - x_Q sin - K.y)
// (two FMA chains each) without the difference Q - c_P: 12 VALU per test.
// Every tile computes each test with the same operations, so results do not
// depend on the tile.
__device__ __forceinline__ bool rect_circle(const float4 Pk, const float2 Q, float lP, float wP, float rr)
{
    const float lam = fmaf(Q.x, Pk.z, fmaf(Q.y, Pk.w, -Pk.x));
    const float mu = fmaf(Q.y, Pk.z, fmaf(-Q.x, Pk.w, -Pk.y));
    const float ex = fmaxf(fabsf(lam) - lP, 0.0f);
    const float ey = fmaxf(fabsf(mu) - wP, 0.0f);
    return fmaf(ex, ex, ey * ey) <= rr;
}

struct CheckVP : PrepA {  // a: the rectangle, in its own frame
    float lP, wP, rr;
    __device__ __forceinline__ CheckVP(const DPair &p) : lP(p.la), wP(p.wa), rr(p.rr) {}
    __device__ __forceinline__ bool operator()(const float4 Pk, const float2 Q) const { return rect_circle(Pk, Q, lP, wP, rr); }
};

struct CheckPV : PrepB {  // b: the rectangle, in its own frame
    float lQ, wQ, rr;
    __device__ __forceinline__ CheckPV(const DPair &p) : lQ(p.lb), wQ(p.wb), rr(p.rr) {}
    __device__ __forceinline__ bool operator()(const float2 P, const float4 Qk) const { return rect_circle(Qk, P, lQ, wQ, rr); }
};

struct CheckPP : PrepNone {
    float rr;
    __device__ __forceinline__ CheckPP(const DPair &p) : rr(p.rr) {}
    __device__ __forceinline__ bool operator()(const float2 P, const float2 Q) const
    {
        const float dx = Q.x - P.x;
        const float dy = Q.y - P.y;
        return fmaf(dx, dx, dy * dy) <= rr;
    }
};

// General convex polygons (vehicle outlines; Sec. IV-C.1 allows polygons of
// any complexity). Q's vertices in P's frame are c + v_x (C, S) + v_y (-S, C) with
// c = (d.u_P, d.v_P); P's in Q's frame are c' + v_x (C, -S) + v_y (S, C)
// with c' = (-d.u_Q, -d.v_Q). With the unit outward edge normals n_e and
// offsets h_e of a polygon, a point x is inside iff n_e.x <= h_e for all e.
//   separating axes: disjoint iff for some edge of either polygon every
//     vertex of the other has n_e.x > h_e;
//   point-in-polygon (the paper's test, both ways): a hit iff some vertex of
//     one has n_e.x <= h_e for every edge of the other.
// Both read the same vertex-edge values. Polygons come padded to KP, KQ = 4
// or 8 vertices (repeated vertices and edges change none of the tests), so
// loop lengths are known; their constants are read from the wave's copy of the
// two polygons in LDS, an edge's in two 16-byte words. The separating-axis
// tests are bound by instruction issue and, with one edge at a time, by the LDS
// latency of each. Collision kernel on the octagon scene, mean of four scenes: a
// comparison per vertex and edge 80 us, the least of an edge's values against
// its offset instead 65, the words of two edges read together 51 (four: the
// same; all eight: spills), giving up between the two polygons' edges 49.

// Whether every one of K points lies beyond an edge, n.x > h: the least of them
// does (a minimum that keeps NaNs, which lie beyond nothing).
template <int K>
__device__ __forceinline__ bool beyond(const DEdge &E, const float (&x)[K], const float (&y)[K])
{
    const float nx = E.nx, ny = E.ny;
    float least = fmaf(nx, x[0], ny * y[0]);
#pragma unroll
    for (int v = 1; v < K; ++v) least = __builtin_elementwise_minimum(least, fmaf(nx, x[v], ny * y[v]));
    return least > E.h;
}

template <int KP, int KQ, bool PIPMODE>
struct CheckGG : PrepNone {
    const DPoly *P, *Q;   // LDS
    __device__ __forceinline__ CheckGG(const DPoly *p, const DPoly *q) : P(p), Q(q) {}
    __device__ __forceinline__ bool operator()(const float4 a, const float4 b) const
    {
        const float dx = b.x - a.x;
        const float dy = b.y - a.y;
        const float C = fmaf(a.z, b.z, a.w * b.w);       // u_P . u_Q
        const float S = fmaf(a.z, b.w, -(a.w * b.z));    // v_P . u_Q
        const float lam = fmaf(dx, a.z, dy * a.w);       // d . u_P
        const float mu = fmaf(dy, a.z, -(dx * a.w));     // d . v_P
        const float lam2 = -fmaf(dx, b.z, dy * b.w);     // -d . u_Q
        const float mu2 = -fmaf(dy, b.z, -(dx * b.w));   // -d . v_Q
        float qx[KQ], qy[KQ], px[KP], py[KP];
#pragma unroll
        for (int v = 0; v < KQ; ++v) {
            qx[v] = fmaf(Q->edge[v].vx, C, fmaf(-Q->edge[v].vy, S, lam));
            qy[v] = fmaf(Q->edge[v].vx, S, fmaf(Q->edge[v].vy, C, mu));
        }
#pragma unroll
        for (int v = 0; v < KP; ++v) {
            px[v] = fmaf(P->edge[v].vx, C, fmaf(P->edge[v].vy, S, lam2));
            py[v] = fmaf(-P->edge[v].vx, S, fmaf(P->edge[v].vy, C, mu2));
        }
        if constexpr (!PIPMODE) {
            bool sep = false;
#pragma unroll 2
            for (int e = 0; e < KP; ++e) sep |= beyond<KQ>(P->edge[e], qx, qy);
            if (__all(sep)) return false;
#pragma unroll 2
            for (int e = 0; e < KQ; ++e) sep |= beyond<KP>(Q->edge[e], px, py);
            return !sep;
        } else {
            // octagons within 3 m, with boxes and without, edges one by one 113
            // and 627 us, four together 82 and 366 (all: 84 and 266, but then
            // the separating axes of the same instance 117 us for 102)
            bool in_q[KQ], in_p[KP];
#pragma unroll
            for (int v = 0; v < KQ; ++v) in_q[v] = true;
#pragma unroll
            for (int v = 0; v < KP; ++v) in_p[v] = true;
#pragma unroll 4
            for (int e = 0; e < KP; ++e) {
                const float nx = P->edge[e].nx, ny = P->edge[e].ny, h = P->edge[e].h;
#pragma unroll
                for (int v = 0; v < KQ; ++v) in_q[v] &= fmaf(nx, qx[v], ny * qy[v]) <= h;
            }
#pragma unroll 4
            for (int e = 0; e < KQ; ++e) {
                const float nx = Q->edge[e].nx, ny = Q->edge[e].ny, h = Q->edge[e].h;
#pragma unroll
                for (int v = 0; v < KP; ++v) in_p[v] &= fmaf(nx, px[v], ny * py[v]) <= h;
            }
            bool hit = false;
#pragma unroll
            for (int v = 0; v < KQ; ++v) hit |= in_q[v];
#pragma unroll
            for (int v = 0; v < KP; ++v) hit |= in_p[v];
            return hit;
        }
    }
};

// Convex polygon G (K vertices, padded) at N poses and M circles (squared
// radius rr): a centre in G's frame; a hit iff it is inside or its squared
// distance to some edge segment is at most rr. All N x M pairs go along one
// walk over the edges, whose constants are read once for them.
// (Scene 2 of those, where these pairs take the most time: 46 us with a walk for
// each pair, 24 so.)
template <int K, int N, int M>
__device__ __forceinline__ void poly_circle(const float4 (&P)[N], const float2 (&c)[M], const DPoly *G, float rr,
                                            bool (&hit)[N][M])
{
    float lam[N][M], mu[N][M], best[N][M];
    bool inside[N][M];
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const float dx = c[m].x - P[n].x;
            const float dy = c[m].y - P[n].y;
            lam[n][m] = fmaf(dx, P[n].z, dy * P[n].w);
            mu[n][m] = fmaf(dy, P[n].z, -(dx * P[n].w));
            inside[n][m] = true;
            best[n][m] = 3.0e38f;
        }
#pragma unroll 2
    for (int e = 0; e < K; ++e) {
        const DEdge E = G->edge[e];
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int m = 0; m < M; ++m) {
                inside[n][m] &= fmaf(E.nx, lam[n][m], E.ny * mu[n][m]) <= E.h;
                const float ax = lam[n][m] - E.vx, ay = mu[n][m] - E.vy;
                const float t = fminf(fmaxf(fmaf(ax, E.ex, ay * E.ey) * E.il, 0.0f), 1.0f);
                const float cx = fmaf(-t, E.ex, ax), cy = fmaf(-t, E.ey, ay);
                best[n][m] = fminf(best[n][m], fmaf(cx, cx, cy * cy));
            }
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int m = 0; m < M; ++m) hit[n][m] = inside[n][m] | (best[n][m] <= rr);
}

template <int K>
struct CheckGC : PrepNone {
    const DPoly *G;   // LDS
    float rr;
    __device__ __forceinline__ CheckGC(const DPoly *g, float r2) : G(g), rr(r2) {}
};

template <int K>
struct CheckCG : PrepNone {
    const DPoly *G;   // LDS
    float rr;
    __device__ __forceinline__ CheckCG(const DPoly *g, float r2) : G(g), rr(r2) {}
};

// The tests of an item at step t: found[r][s] = t where a[r] and b[s] overlap.
template <int RI, int RJ, class PA, class PB, class Check>
__device__ __forceinline__ void test_tile(const Check &chk, const PA (&a)[RI], const PB (&b)[RJ], int (&found)[RI][RJ],
                                          int t)
{
#pragma unroll
    for (int r = 0; r < RI; ++r)
#pragma unroll
        for (int s = 0; s < RJ; ++s)
            if (chk(a[r], b[s])) found[r][s] = t;
}

template <int RI, int RJ, int K>
__device__ __forceinline__ void test_tile(const CheckGC<K> &chk, const float4 (&a)[RI], const float2 (&b)[RJ],
                                          int (&found)[RI][RJ], int t)
{
    bool hit[RI][RJ];
    poly_circle<K>(a, b, chk.G, chk.rr, hit);
#pragma unroll
    for (int r = 0; r < RI; ++r)
#pragma unroll
        for (int s = 0; s < RJ; ++s)
            if (hit[r][s]) found[r][s] = t;
}

template <int RI, int RJ, int K>
__device__ __forceinline__ void test_tile(const CheckCG<K> &chk, const float2 (&a)[RI], const float4 (&b)[RJ],
                                          int (&found)[RI][RJ], int t)
{
    bool hit[RJ][RI];
    poly_circle<K>(b, a, chk.G, chk.rr, hit);
#pragma unroll
    for (int r = 0; r < RI; ++r)
#pragma unroll
        for (int s = 0; s < RJ; ++s)
            if (hit[s][r]) found[r][s] = t;
}

// Raw buffer descriptor (CDNA: dword3 = 0x00020000) over `bytes` bytes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pose_rsrc(const char *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), (short)0, (int)bytes, 0x00020000);
}

template <class P>
__device__ __forceinline__ P load_pose(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff);

template <>
__device__ __forceinline__ float4 load_pose<float4>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

template <>
__device__ __forceinline__ float2 load_pose<float2>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
}

// When a step needs no tests: the boxes of two groups of trajectories lie apart
// at that step, along x or along y, by more than the rounding of the tests.
//
// That no test of such a step finds an overlap holds for the FP32 tests as
// they are computed, not only for the shapes. With u = 2^-24 and M the largest
// coordinate of the two boxes, positions are at most M, half extents 1.42 M and
// vertices 2 M, so that the roundings add up to at most about
//   rectangles  45 u M: projections onto the other's axes 25, radii 15, axes 5;
//   outlines    60 u M: a vertex in the other's frame 25 a coordinate, an edge's
//                       normal, product and offset 20, axes 5;
//   circles     55 u M: centre in the frame 8 a coordinate, nearest point of an
//                       edge 25 a coordinate, square and radius 7, axes 5;
//   boxes        8 u M: extents, sides and the gap itself.
// Shapes whose boxes lie m apart are separated by at least 0.7 m along one of
// the axes of a rectangle test, by 0.38 m along one of the edge normals of an
// outline test (neighbouring normals turn by at most 135 degrees, interior
// angles being 45 degrees or more; the cosine of half of it), and a circle by m
// itself. A step is left out at m > 256 u M (kBoxSlack): 98 u M against 68.
// A gap of at least kBoxLeast (M counts as 2^16 times that or more) keeps that
// from underflow: the tests' squares are 0 in FP32 below 1e-22 m and the circle
// tests then find overlaps that are none, but a gap of 2^-50 m leaves at least
// 2^-100 between the squares that they compare.
// Boxes with an infinite side separate nothing, and the comparison is made so
// that a NaN keeps the step.
__device__ __forceinline__ float box_size(const float4 a)
{
    return fmaxf(fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))), kBoxLeast / kBoxSlack);
}

// size: the larger box_size of the two.
__device__ __forceinline__ bool boxes_meet(const float4 a, const float4 b, float size)
{
    const float gx = fmaxf(b.x - a.y, a.x - b.y), gy = fmaxf(b.z - a.w, a.z - b.w);
    return !(fmaxf(gx, gy) > size * kBoxSlack);
}

// The boxes at this lane's step t of `side` leaves from leaf0 on (past those and
// past the object's last leaf: the last again).
__device__ __forceinline__ void load_boxes(float4 (&box)[BLOCK_LEAVES], const char *__restrict__ poses, int64_t off,
                                           int T, int H, int t, int leaf0, int side)
{
    const int leaves = (T + LEAF - 1) / LEAF, last = min(leaf0 + side, leaves) - 1;
    const __amdgpu_buffer_rsrc_t R = pose_rsrc(poses + off, (uint32_t)(leaves * H) * 16u);
#pragma unroll
    for (int i = 0; i < BLOCK_LEAVES; ++i)
        box[i] = load_pose<float4>(R, (uint32_t)min(t, H - 1) * 16u, (uint32_t)(min(leaf0 + i, last) * H) * 16u);
}

__device__ __forceinline__ float4 join_boxes(const float4 (&b)[BLOCK_LEAVES])
{
    static_assert(BLOCK_LEAVES == 4);
    return box_join(box_join(b[0], b[1]), box_join(b[2], b[3]));
}

// Which of the blocks (bi, bj0 .. bj0 + n - 1) of a pair have a step to test.
__device__ __forceinline__ uint32_t blocks_to_test(const DPair &pr, const char *__restrict__ poses, int side, int bi,
                                                   int bj0, int n)
{
    if (pr.box_a < 0) return (1u << n) - 1u;
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    uint32_t alive = 0;
    for (int w0 = 0; w0 < pr.H; w0 += WAVE) {
        const int t = w0 + lane;
        float4 box[BLOCK_LEAVES];
        load_boxes(box, poses, pr.box_a, pr.Ta, pr.H, t, bi * side, side);
        const float4 a = join_boxes(box);
        const float ma = box_size(a);
        for (int j = 0; j < n; ++j) {
            load_boxes(box, poses, pr.box_b, pr.Tb, pr.H, t, (bj0 + j) * side, side);
            const float4 b = join_boxes(box);
            if (__any((t < pr.H) & boxes_meet(a, b, fmaxf(ma, box_size(b))))) alive |= 1u << j;
        }
    }
    return alive;
}

// A wave's LDS operations complete in order; keeps the compiler from moving
// its reads above its other lanes' writes, and the other way round.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// __syncthreads() of the collision kernel. The wait for this wave's own LDS
// operations is written out: after the loop over the units the compiler (ROCm
// 7.2) left it out, and the last overlaps of a workgroup were then missed by
// the waves that were past the barrier before they had landed.
__device__ __forceinline__ void workgroup_sync()
{
    constexpr int kLgkmcnt0 = 0xC07F;   // lgkmcnt(0), the other counters not waited for
    __builtin_amdgcn_s_waitcnt(kLgkmcnt0);
    __syncthreads();
}

constexpr uint32_t kNoHit = ~0u;

// Tests the item (ig, jg) of this lane at `rounds` rounds of S steps, one of
// each round by this lane's part: of the n steps that lanes 0 .. n-1 hold in
// `step`, those at k, k - S, ... below the end, from later to earlier. Records
// each pair's earliest overlap in first[r * stride + s]; returns whether this
// lane found one. Poses are read with buffer loads, whose range check makes
// reads past the pose block (positions past the last trajectory) return 0; a
// position past Ta inside the block is the next step's pose. What such
// positions find is dropped with the results.
template <int RI, int RJ, class PA, class PB, class Check>
__device__ __forceinline__ bool test_item(const DPair &pr, const char *__restrict__ poses, int ig, int jg, int step,
                                          int k, int rounds, uint32_t *first, int stride, const Check chk)
{
    const int S = 1 << pr.tshift;
    const uint32_t strideA = (uint32_t)pr.Ta * (uint32_t)sizeof(PA), strideB = (uint32_t)pr.Tb * (uint32_t)sizeof(PB);
    const __amdgpu_buffer_rsrc_t A = pose_rsrc(poses + pr.pose_a, (uint32_t)pr.H * strideA);
    const __amdgpu_buffer_rsrc_t B = pose_rsrc(poses + pr.pose_b, (uint32_t)pr.H * strideB);
    const uint32_t oa = (uint32_t)(ig * RI) * (uint32_t)sizeof(PA), ob = (uint32_t)(jg * RJ) * (uint32_t)sizeof(PB);
    int found[RI][RJ];
#pragma unroll
    for (int r = 0; r < RI; ++r)
#pragma unroll
        for (int s = 0; s < RJ; ++s) found[r][s] = -1;
    for (int m = 0; m < rounds; ++m, k -= S) {
        const int t = __builtin_amdgcn_ds_bpermute(max(k, 0) << 2, step);
        const uint32_t va = oa + (uint32_t)t * strideA, vb = ob + (uint32_t)t * strideB;
        PA a[RI];
        PB b[RJ];
#pragma unroll
        for (int r = 0; r < RI; ++r) a[r] = load_pose<PA>(A, va + r * (uint32_t)sizeof(PA), 0);
#pragma unroll
        for (int s = 0; s < RJ; ++s) b[s] = load_pose<PB>(B, vb + s * (uint32_t)sizeof(PB), 0);
#pragma unroll
        for (int r = 0; r < RI; ++r) a[r] = chk.prep_a(a[r]);
#pragma unroll
        for (int s = 0; s < RJ; ++s) b[s] = chk.prep_b(b[s]);
        test_tile(chk, a, b, found, t);
    }
    bool any = false;
#pragma unroll
    for (int r = 0; r < RI; ++r)
#pragma unroll
        for (int s = 0; s < RJ; ++s)
            if (found[r][s] >= 0) {
                atomicMin(&first[r * stride + s], (uint32_t)found[r][s]);
                any = true;
            }
    return any;
}

// Copies the two polygons of a polygon pair into this wave's LDS slot (each
// lane a few words), so that their constants reach the tests as vector
// registers instead of competing for scalar ones. Once for all items of a pair
// that the wave tests one after another: octagons within 3 m 102 us with a copy
// an item, 100 so.
__device__ __forceinline__ void stage_polygons(DPoly *slot, const DPoly *__restrict__ polys, const DPair &pr)
{
    constexpr int words = (int)(sizeof(DPoly) / sizeof(int32_t));
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    int32_t *dst = reinterpret_cast<int32_t *>(slot);
    const int32_t *pa = reinterpret_cast<const int32_t *>(polys + (pr.poly_a >= 0 ? pr.poly_a : pr.poly_b));
    const int32_t *pb = reinterpret_cast<const int32_t *>(polys + (pr.poly_b >= 0 ? pr.poly_b : pr.poly_a));
    for (int k = lane; k < words; k += WAVE) {
        dst[k] = pa[k];
        dst[words + k] = pb[k];
    }
    wave_lds_fence();
}

// FAM: the test classes this kernel instance carries. FAM_PLAIN: rectangles
// and circles; FAM_PIP: also the point-in-polygon rectangle test; FAM_POLY:
// also the polygon classes. The larger code and tiles of the later families
// need more registers, which would lower the occupancy of the earlier ones;
// a launch uses the smallest family that covers its pairs.
// TL: whether it can add to per-slot sums (time-resolved scenes); likewise
// kept out of the instances that launches without such scenes use.
template <int V, int FAM>
__device__ __forceinline__ bool test_items(const DPair &pr, const char *__restrict__ poses, int ig, int jg, int step,
                                           int k, int rounds, uint32_t *first, int er, int ec, int stride,
                                           const DPoly *lp)
{
#define MHC_TEST(CLS, PA, PB, CHK)                                                                                      \
    test_item<kTiles[V][CLS].ri, kTiles[V][CLS].rj, PA, PB>(                                                           \
        pr, poses, ig, jg, step, k, rounds, first + er * kTiles[V][CLS].ri * stride + ec * kTiles[V][CLS].rj, stride, \
        CHK)
    if constexpr (FAM >= FAM_PIP) {
        if (pr.cls == CLS_VV_PIP) return MHC_TEST(CLS_VV_PIP, float4, float4, CheckVVPip(pr));
    }
    if constexpr (FAM >= FAM_POLY) {
        const DPoly *P = lp, *Q = lp + 1;  // the pair's polygons
        switch (pr.cls) {
        case CLS_GG:
        case CLS_GG_PIP: {
            const int shape = (P->k == 8 ? 2 : 0) + (Q->k == 8 ? 1 : 0) + (pr.cls == CLS_GG_PIP ? 4 : 0);
            switch (shape) {
#define MHC_GG(S, KP, KQ, PIPM) \
    case S: return MHC_TEST(CLS_GG, float4, float4, (CheckGG<KP, KQ, PIPM>(P, Q)));
                MHC_GG(0, 4, 4, false)
                MHC_GG(1, 4, 8, false)
                MHC_GG(2, 8, 4, false)
                MHC_GG(3, 8, 8, false)
                MHC_GG(4, 4, 4, true)
                MHC_GG(5, 4, 8, true)
                MHC_GG(6, 8, 4, true)
                MHC_GG(7, 8, 8, true)
#undef MHC_GG
            }
            return false;
        }
        case CLS_GC:
            return P->k == 8 ? MHC_TEST(CLS_GC, float4, float2, CheckGC<8>(P, pr.rr))
                             : MHC_TEST(CLS_GC, float4, float2, CheckGC<4>(P, pr.rr));
        case CLS_CG:
            return P->k == 8 ? MHC_TEST(CLS_CG, float2, float4, CheckCG<8>(P, pr.rr))
                             : MHC_TEST(CLS_CG, float2, float4, CheckCG<4>(P, pr.rr));
        default:
            break;
        }
    }
    switch (pr.cls) {
    case CLS_VV: return MHC_TEST(CLS_VV, float4, float4, CheckVV(pr));
    case CLS_VP: return MHC_TEST(CLS_VP, float4, float2, CheckVP(pr));
    case CLS_PV: return MHC_TEST(CLS_PV, float2, float4, CheckPV(pr));
    default: return MHC_TEST(CLS_PP, float2, float2, CheckPP(pr));
    }
#undef MHC_TEST
}

// The pair that strip g of the launch belongs to: the last p with strip0[p] <= g,
// by the wave's 64 lanes together (two rounds for up to 4096 pairs).
__device__ __forceinline__ int pair_of_strip(const int64_t *__restrict__ strip0, int n_pairs, int64_t g)
{
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    int lo = 0, len = n_pairs;
    while (len > 1) {
        const int step = (len + WAVE - 1) / WAVE;
        const int k = lane * step;
        const bool le = k < len && strip0[lo + min(k, len - 1)] <= g;
        const int last = (__popcll(__ballot(le)) - 1) * step;
        lo += last;
        len = min(step, len - last);
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Waves per SIMD that an instance is held to: three workgroups a CU for the
// rectangle and circle classes (80 vector registers; two, with 94, measured
// 412 against 357 us on the 40-object stress scene and 28 against 23 us on the
// 3-object road with the point-in-polygon test), two for the polygon classes.
template <int FAM>
constexpr int kCollideMinWaves = FAM == FAM_POLY ? 4 : 6;

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// What the results of a block need of its pair.
struct BlockLds {
    int Ta, Tb, wa, wb, na;  // trajectory counts, lanes of the per-slot sums (0: none), objects
    int pad;
    int64_t hit, qa, qb;     // first-hit entry and q sums of (i = 0, j = 0)
    int64_t ha, hb;          // per-slot sums of slot 0, i = 0 and j = 0
};

// The LDS of a collision workgroup: the blocks of the round that have steps to
// test, and of the K2_SLOTS of them that are taken together
struct K2Lds {
    int4 alive[K2_SLOTS * MAX_STRIP];               // pair, block row, block column, horizon
    BlockLds block[K2_SLOTS];
    uint32_t first[K2_SLOTS * BLOCK_PAIRS];         // earliest overlap of every trajectory pair, [slot][row][column]
    unsigned long long mask[K2_UNITS];              // steps to test of the units that have any
    uint32_t unit[K2_UNITS];                        // slot, window, time split and unit of the block (unit_word)
    unsigned long long leaf_mask[K2_SLOTS][BLOCK_LEAVES * BLOCK_LEAVES];
    // trajectories at the blocks' rows and columns, their integer
    // probabilities, and the sums over the colliding pairs of a row or column
    int ti[K2_SLOTS][BLOCK_SIDE], tj[K2_SLOTS][BLOCK_SIDE];
    unsigned long long pa[K2_SLOTS][BLOCK_SIDE], pb[K2_SLOTS][BLOCK_SIDE];
    unsigned long long sum_a[K2_SLOTS][BLOCK_SIDE], sum_b[K2_SLOTS][BLOCK_SIDE];
    int n_alive[3], n_units[3], any_hit;
};

__device__ __forceinline__ uint32_t unit_word(int slot, int window, int tshift, int u)
{
    return (uint32_t)(slot << 16 | window << 15 | tshift << 12 | u);
}

// Lists the units of the block in a slot that have steps to test among w0 ..
// w0 + 127, by one wave: lane l looks at step l of a window of 64, for all the
// block's pairs of leaves; a unit's steps are those of its leaves.
__device__ __forceinline__ void list_units(K2Lds &w, int *n_units, int slot, const DPair &pr, int side, int bi, int bj,
                                           int w0, const char *__restrict__ poses)
{
    const int lane = (int)(threadIdx.x & (WAVE - 1)), H = pr.H;
    const int na = (pr.Ta + LEAF - 1) / LEAF - bi * side, nb = (pr.Tb + LEAF - 1) / LEAF - bj * side;
    // lane u: unit u of the block
    const int ur = lane >> pr.block_ucs, uc = lane & ((1 << pr.block_ucs) - 1);
    const bool unit = ur < pr.block_ur && bi * pr.block_ur + ur < pr.nui && (bj << pr.block_ucs) + uc < pr.nuj;
    for (int window = 0; window < 2 && w0 + window * WAVE < H; ++window) {
        const int t = w0 + window * WAVE + lane;
        unsigned long long mine = 0;   // lane i * 4 + j: of leaf i of a and j of b
        if (pr.box_a < 0) {
            mine = __ballot(t < H);
        } else {
            float4 a[BLOCK_LEAVES], b[BLOCK_LEAVES];
            load_boxes(a, poses, pr.box_a, pr.Ta, H, t, bi * side, side);
            load_boxes(b, poses, pr.box_b, pr.Tb, H, t, bj * side, side);
            float mb[BLOCK_LEAVES];
#pragma unroll
            for (int j = 0; j < BLOCK_LEAVES; ++j) mb[j] = box_size(b[j]);
#pragma unroll
            for (int i = 0; i < BLOCK_LEAVES; ++i) {
                if (i >= side) break;
                const float ma = box_size(a[i]);
#pragma unroll
                for (int j = 0; j < BLOCK_LEAVES; ++j) {
                    if (j >= side) break;
                    const unsigned long long m = __ballot((t < H) & boxes_meet(a[i], b[j], fmaxf(ma, mb[j])));
                    if (lane == i * BLOCK_LEAVES + j) mine = m;
                }
            }
        }
        if (lane < BLOCK_LEAVES * BLOCK_LEAVES)
            w.leaf_mask[slot][lane] = lane / BLOCK_LEAVES < min(na, side) && lane % BLOCK_LEAVES < min(nb, side) ? mine : 0ull;
        wave_lds_fence();
        if (unit) {
            const int i0 = ur << pr.unit_rs, j0 = uc << pr.unit_cs;
            const int i1 = (i0 + (1 << pr.unit_rs) - 1) / LEAF, j1 = (j0 + (1 << pr.unit_cs) - 1) / LEAF;
            unsigned long long m = 0;
            for (int i = i0 / LEAF; i <= i1; ++i)
                for (int j = j0 / LEAF; j <= j1; ++j) m |= w.leaf_mask[slot][i * BLOCK_LEAVES + j];
            if (m) {
                const int at = atomicAdd(n_units, 1);
                w.mask[at] = m;
                w.unit[at] = unit_word(slot, window, pr.tshift, lane);
            }
        }
        wave_lds_fence();   // before the next window's leaf masks
    }
}

// Fills in the results part of a slot, by one wave.
__device__ __forceinline__ void block_tables(K2Lds &w, int slot, const DPair &pr, int side_leaves, int bi, int bj,
                                             const DObj *__restrict__ objs, const unsigned long long *__restrict__ pfix)
{
    const int lane = (int)(threadIdx.x & (WAVE - 1)), x = lane & (BLOCK_SIDE - 1);
    const int side = side_leaves * LEAF;
    const DObj &oa = objs[pr.a], &ob = objs[pr.b];
    // the first half of the wave a's rows, the second b's columns
    const bool is_row = lane < BLOCK_SIDE;
    const int pos = (is_row ? bi : bj) * side + x, T = is_row ? oa.T : ob.T;
    const int i = x < side && pos < T ? (is_row ? traj_at(pos, oa.n_u, oa.n_w, oa.strip)
                                                : traj_at(pos, ob.n_u, ob.n_w, ob.strip)) : -1;
    const unsigned long long p = i >= 0 ? pfix[(is_row ? oa.traj_off : ob.traj_off) + i] : 0ull;
    (is_row ? w.ti : w.tj)[slot][x] = i;
    (is_row ? w.pa : w.pb)[slot][x] = p;
    (is_row ? w.sum_a : w.sum_b)[slot][x] = 0ull;
    if (lane == 0) {
        BlockLds &b = w.block[slot];
        b.Ta = oa.T;
        b.Tb = ob.T;
        b.na = oa.n_scene_obj;
        b.wa = oa.timeline ? oa.tl_w : 0;
        b.wb = ob.tl_w;
        b.hit = pr.hit_off;
        b.qa = oa.q_row + ob.local;
        b.qb = ob.q_row + oa.local;
        b.ha = oa.hist_off + ob.local;
        b.hb = ob.hist_off + oa.local;
    }
}

// Collision kernel. The launch's blocks (up to 32 x 32 trajectory pairs) are
// looked at in strips of a block row, pair after pair, in rounds: in round r
// wave w of workgroup b takes a strip of row r * 8 + w (grid strips a row,
// strip_in_row) and finds out from the two groups' boxes in which of its
// blocks any step can hold an overlap. The few such blocks are then taken by
// the workgroup together, eight at a time, for every 128 steps of the horizon:
//   - a wave per block finds the steps to test of the block's units from the
//     boxes of their leaves, and lists the units that have any, while another
//     looks up what the results will need;
//   - the listed units' rounds of S steps are dealt evenly to the waves, which
//     test them and keep the earliest overlap of every pair in LDS;
// and last the pairs that overlap are stored and summed up. Which blocks meet
// is known to nobody beforehand, so work is spread in three ways: a workgroup's
// strips of a round come from far apart in the sequence, the strips of a pair
// are in an order that keeps neighbours apart (strip_at), and inside a
// workgroup no wave owns a unit. With most blocks gone after one look, a
// launch is bound by the latency of its dependent reads (pair, boxes, poses,
// tables: 1 to 2 us each when first touched on a CU), so each of them is made
// once per block, by waves side by side.
// A launch may run a part of the plan (strips_before_part): its strips, from
// strip_lo on, fill full_rows rows and last_row strips of the next. A wave
// tests 2^item_shift rounds of S steps of a unit at a time. The small numbers
// come in one argument (k2_sizes): as one each they left two of the 80 vector
// registers of some instances in scratch memory (11-object scene 14.7 us, 14.3
// so).
template <int V, int FAM, bool TL>
__global__ __launch_bounds__(K2_WG) __attribute__((amdgpu_waves_per_eu(kCollideMinWaves<FAM>))) void k2_collide(
    const DPair *__restrict__ pairs, const DObj *__restrict__ objs, const int64_t *__restrict__ strip0, int n_pairs,
    int64_t strip_lo, int full_rows, int last_row, uint32_t sizes, const char *__restrict__ poses,
    int16_t *__restrict__ hits, const unsigned long long *__restrict__ pfix, unsigned long long *__restrict__ qacc,
    unsigned long long *__restrict__ hist, const DPoly *__restrict__ polys)
{
    constexpr int NW = K2_WG / WAVE;
    const int strip_len = (int)(sizes & 0xFF), side_shift = (int)(sizes >> 8 & 0xFF);
    const int item_shift = (int)(sizes >> 16), item_rounds = 1 << item_shift;
    const int side = (1 << side_shift) / LEAF;   // leaves to a side of a block
    static_assert(NW == K2_SLOTS);
    const int tid = (int)threadIdx.x, lane = tid & (WAVE - 1), wave = uniform(tid / WAVE);
    // per wave: the two polygons of its current polygon pair
    constexpr bool poly = FAM >= FAM_POLY;
    __shared__ DPoly lds_polys[poly ? 2 * NW : 1];
    __shared__ K2Lds w;
    DPoly *lp = lds_polys + (poly ? 2 * wave : 0);
    int staged = -1;   // the pair whose polygons are there
    // The counters n_alive and n_units go round three places: one is used now,
    // the next one is emptied before a barrier. That one was last read before
    // the barrier of the use before this one, which every wave has passed.
    if (tid < 3) w.n_alive[tid] = w.n_units[tid] = 0;
    if (tid == 0) w.any_hit = 0;
    workgroup_sync();
    auto next = [](int at) { return at == 2 ? 0 : at + 1; };
    int alive_at = 0, units_at = 0;
    for (int row0 = 0; row0 < full_rows + (last_row > 0); row0 += NW) {
        const int row = row0 + wave, x = strip_in_row(row, (int)blockIdx.x, (int)gridDim.x);
        if (row < full_rows || (row == full_rows && x < last_row)) {
            const int64_t g = strip_lo + (int64_t)row * gridDim.x + x;
            const int p = pair_of_strip(strip0, n_pairs, g);
            const DPair &pr = pairs[p];
            int bi, bj;
            strip_at(pr, (uint32_t)(g - strip0[p]), &bi, &bj);
            bj *= strip_len;
            const uint32_t alive = blocks_to_test(pr, poses, side, bi, bj, min(strip_len, pr.nbj - bj));
            if (lane < strip_len && alive >> lane & 1u)
                w.alive[atomicAdd(&w.n_alive[alive_at], 1)] = make_int4(p, bi, bj + lane, pr.H);
        }
        if (tid == 0) w.n_alive[next(alive_at)] = 0;
        workgroup_sync();
        const int n = uniform(w.n_alive[alive_at]);
        alive_at = next(alive_at);
        for (int k0 = 0; k0 < n; k0 += K2_SLOTS) {
            const int slots = min(n - k0, K2_SLOTS);
            int H = 0;
            for (int k = 0; k < slots; ++k) H = max(H, uniform(w.alive[k0 + k].w));
            // up to four blocks: the tables by the other waves
            const int tables = 2 * slots <= NW ? NW - 1 - wave : wave;
            for (int q = tid; q < slots << 2 * side_shift; q += K2_WG) w.first[q] = kNoHit;
            for (int w0 = 0; w0 < H; w0 += 2 * WAVE) {
                if (wave < slots) {
                    const int4 b = w.alive[k0 + wave];
                    list_units(w, &w.n_units[units_at], wave, pairs[uniform(b.x)], side, uniform(b.y), uniform(b.z), w0,
                               poses);
                }
                if (w0 == 0 && tables < slots) {
                    const int4 b = w.alive[k0 + tables];
                    block_tables(w, tables, pairs[uniform(b.x)], side, uniform(b.y), uniform(b.z), objs, pfix);
                }
                if (tid == 0) w.n_units[next(units_at)] = 0;
                workgroup_sync();
                // the tests
                const int n_units = uniform(w.n_units[units_at]);
                units_at = next(units_at);
                int turn = 0;   // items of the units before
                for (int x0 = 0; x0 < n_units; x0 += WAVE) {
                    // lane l: unit x0 + l, its items (item_rounds rounds of
                    // S steps) and those of the units before it
                    const int x = min(x0 + lane, n_units - 1);
                    const int ts = w.unit[x] >> 12 & 7;
                    const int rounds = (__popcll(w.mask[x]) + (1 << ts) - 1) >> ts;
                    const int upto = scan_add_int(x0 + lane < n_units ? (rounds + item_rounds - 1) >> item_shift : 0);
                    const int items = __builtin_amdgcn_readlane(upto, WAVE - 1);
                    for (int it = (wave - turn) & (NW - 1); it < items; it += NW) {
                        const int l = __popcll(__ballot(upto <= it));
                        const int m0 = (it - (l ? __builtin_amdgcn_readlane(upto, l - 1) : 0)) << item_shift;
                        const unsigned long long mask = w.mask[x0 + l];
                        const int word = uniform((int)w.unit[x0 + l]), slot = word >> 16, u = word & 0xFFF;
                        const int4 b = w.alive[k0 + slot];
                        const DPair &pr = pairs[uniform(b.x)];
                        if (poly && pr.cls >= CLS_GG && staged != uniform(b.x)) {
                            stage_polygons(lp, polys, pr);
                            staged = uniform(b.x);
                        }
                        const int ur = u >> pr.block_ucs, uc = u & ((1 << pr.block_ucs) - 1);
                        const int per = WAVE >> pr.tshift, e = lane & (per - 1), part = lane >> (6 - pr.tshift);
                        const int er = e >> pr.bshift, ec = e & ((1 << pr.bshift) - 1);
                        // lane i < n_steps gets the i-th step to test
                        const int n_steps = __popcll(mask);
                        const int rank = (int)__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                        const int dest = (mask >> lane) & 1ull ? rank : n_steps + lane - rank;
                        const int step = __builtin_amdgcn_ds_permute(dest << 2, w0 + (word >> 15 & 1) * WAVE + lane);
                        const bool any = test_items<V, FAM>(
                            pr, poses, (uniform(b.y) * pr.block_ur + ur) * (per >> pr.bshift) + er,
                            (((uniform(b.z) << pr.block_ucs) + uc) << pr.bshift) + ec, step,
                            n_steps - 1 - (m0 << pr.tshift) - part,
                            min(((n_steps + (1 << pr.tshift) - 1) >> pr.tshift) - m0, item_rounds),
                            &w.first[(((slot << side_shift) + (ur << pr.unit_rs)) << side_shift) + (uc << pr.unit_cs)], er,
                            ec, 1 << side_shift, lp);
                        if (any) w.any_hit = 1;
                    }
                    turn += items;
                }
                workgroup_sync();
            }
            // Results: the first hits of colliding trajectory pairs (the
            // entries start at -1), and the blocks' share of the q sums. A
            // colliding pair (i, j) adds p_{b,j} to q_{a,i;b} and p_{a,i} to
            // q_{b,j;a}; sums are exact integers (p * 2^62), so their value
            // does not depend on the order of the adds.
            if (!uniform(w.any_hit)) continue;
            for (int q = tid; q < slots << 2 * side_shift; q += K2_WG) {
                const uint32_t f = w.first[q];
                if (f == kNoHit) continue;
                const int k = q >> 2 * side_shift;
                const int rr = (q >> side_shift) & ((1 << side_shift) - 1), cc = q & ((1 << side_shift) - 1);
                const int i = w.ti[k][rr], j = w.tj[k][cc];
                if (i < 0 || j < 0) continue;
                const BlockLds &b = w.block[k];
                if (hits) hits[b.hit + (int64_t)i * b.Tb + j] = (int16_t)f;
                if (TL && b.wa) {
                    // time-resolved: each colliding pair adds to the sums of
                    // its first colliding slot
                    atomicAdd(&hist[b.ha + ((int64_t)f * b.Ta + i) * b.wa], w.pb[k][cc]);
                    atomicAdd(&hist[b.hb + ((int64_t)f * b.Tb + j) * b.wb], w.pa[k][rr]);
                } else {
                    atomicAdd(&w.sum_a[k][rr], w.pb[k][cc]);
                    atomicAdd(&w.sum_b[k][cc], w.pa[k][rr]);
                }
            }
            workgroup_sync();
            if (tid == 0) w.any_hit = 0;
            if (wave < slots) {
                const BlockLds &b = w.block[wave];
                const int x = lane & (BLOCK_SIDE - 1);
                const bool is_row = lane < BLOCK_SIDE;
                const unsigned long long sum = (is_row ? w.sum_a : w.sum_b)[wave][x];
                if (sum) atomicAdd(&qacc[is_row ? b.qa + (int64_t)w.ti[wave][x] * b.na : b.qb + (int64_t)w.tj[wave][x] * b.na], sum);
            }
            workgroup_sync();   // before the next blocks' tables
        }
        if (n > 0) workgroup_sync();   // before the next round's blocks
    }
}

// -1 over the first hits, for a collision stage that runs without the
// trajectory stage of the same call (which writes them otherwise).
__global__ __launch_bounds__(WG) void k2_clear(int16_t *__restrict__ hits, int64_t n_hits, int64_t per_wg)
{
    clear_hits(hits, n_hits, per_wg, (int64_t)blockIdx.x);
}

// ===========================================================================
// K3: risk assessment (Sec. IV-D, IV-D.2).
//
// The collision kernel has left the q_{a,i;b} as exact integer sums (p in
// units of 2^-62, or -log(1 - p) in units of 2^-56 for the INDEPENDENT
// reading; for time-resolved scenes the k3_timeline kernel has added up the
// per-slot sums into the same accumulators). Grid: y = object, x = chunk of 256
// trajectories; thread tid of chunk c takes trajectory i = 256 c + tid,
// converts its sums (rounding once), clamps to 1, writes q and forms
//   crit_{a,i} = 1 - prod_{b != a} (1 - q_{a,i;b})     (ascending b).
// The workgroup adds p_{a,i} crit_{a,i} over its chunk in a fixed order. An
// object of one chunk writes C_a directly; otherwise the chunks add their
// sums in fixed point into a per-object word (zeroed by the trajectory
// kernel) that also counts them, and the chunk that completes the count
// writes C_a. Nothing depends on how the collision work was tiled or
// batched, or on which chunk ends last, so every result is identical for any
// tiling and any batch.
// ===========================================================================

constexpr int K3_LOADS = 16;
constexpr unsigned long long kChunkOne = 1ull << 56;  // one finished chunk in the per-object word
constexpr double kCritScale = 0x1p55, kCritInvScale = 0x1p-55;

__global__ __launch_bounds__(WG) void k3_crit(const DObj *__restrict__ objs,
                                              const unsigned long long *__restrict__ qacc,
                                              const double *__restrict__ p, double *__restrict__ q,
                                              double *__restrict__ traj_crit, double *__restrict__ obj_crit,
                                              unsigned long long *__restrict__ done)
{
    __shared__ double red[WG / WAVE];
    const int obj = (int)blockIdx.y;
    const DObj o = objs[obj];
    const int chunks = (o.T + WG - 1) / WG;
    const int c = (int)blockIdx.x;
    if (c >= chunks) return;  // whole workgroup
    const int n = o.n_scene_obj;
    const int tid = threadIdx.x;
    double acc = 0.0;
    const int i = c * WG + tid;
    if (i < o.T) {
        // The trajectory kernel zeroed all n accumulators of this trajectory,
        // so b == a and objects outside the pair set read as q = 0. Loads are
        // issued sixteen at a time (scenes of up to 16 objects in one round),
        // ahead of the dependent product.
        const unsigned long long *__restrict__ qa = qacc + o.q_row + (int64_t)i * n;
        double *__restrict__ qi = q ? q + o.q_row + (int64_t)i * n : nullptr;
        const double pi = p[o.traj_off + i];
        double no_collision = 1.0;
        for (int b0 = 0; b0 < n; b0 += K3_LOADS) {
            unsigned long long v[K3_LOADS];
#pragma unroll
            for (int k = 0; k < K3_LOADS; ++k) v[k] = b0 + k < n ? qa[b0 + k] : 0ull;
#pragma unroll
            for (int k = 0; k < K3_LOADS; ++k) {
                if (b0 + k < n) {
                    const double qv = q_of(o.risk, v[k]);
                    if (qi) qi[b0 + k] = qv;
                    no_collision *= 1.0 - qv;
                }
            }
        }
        const double crit = 1.0 - no_collision;
        traj_crit[o.traj_off + i] = crit;
        acc = pi * crit;
    }
    const double chunk_sum = block_sum(acc, red);
    if (chunks == 1) {
        if (tid == 0) obj_crit[o.obj_out] = chunk_sum;
        return;
    }
    if (tid != 0) return;
    // One atomic per chunk adds the chunk's sum in fixed point (units of
    // 2^-55; an object's sum is at most 1, so it stays below 2^56) together
    // with a count of one at bit 56 (at most 128 chunks). The chunk whose add
    // completes the count has the whole sum in the value it gets back; the
    // sum is exact in integers, so it does not depend on which chunk ends
    // last, and nothing else is shared between the chunks.
    const unsigned long long mine = kChunkOne + __double2ull_rn(chunk_sum * kCritScale);
    const unsigned long long before = atomicAdd(&done[obj], mine);
    if ((before >> 56) != (unsigned long long)(chunks - 1)) return;
    obj_crit[o.obj_out] = (double)((before + mine) & (kChunkOne - 1)) * kCritInvScale;
    done[obj] = 0ull;  // the risk stage may run again on the same sums
}

// ===========================================================================
// Time-resolved risk (Sec. IV-D.2 over the horizon; the criticality curve the
// anticipation time of Sec. IV-D / VI-A is read from).
//
// For time-resolved scenes the collision kernel adds the summand of every
// colliding trajectory pair to the sums of its first colliding slot s:
// hist_a[s][i][b] (object a's block, b padded to W = the power of two >= n,
// so the W sums of one trajectory and slot are contiguous). For trajectory
// (a, i) with running sums Q_b(s) = sum_{s' <= s} hist_a[s'][i][b] and
// no-collision factors f_b(s) = 1 - q(Q_b(s)), the combinations are taken
// slot by slot, ascending b within a slot; the probability that the first
// collision happens with b at slot s is
//   (f_b(s-1) - f_b(s)) * prod_{b' < b} f_{b'}(s) * prod_{b' > b} f_{b'}(s-1)
// Adding these up over slots gives the attribution A_{a,i;b}, and
// crit_{a,i}(s) = 1 - prod_b f_b(s).
// ===========================================================================

constexpr int K3T_SLOTS = 8;  // slots processed together: loads one group ahead, scans interleaved

// A double from the lane d below (UP) or above (!UP) in the same row of 16
// lanes (DPP row shift; lanes whose source lies outside the row get 0).
template <int D, bool UP>
__device__ __forceinline__ double row_shift(double x)
{
    constexpr int ctrl = (UP ? 0x110 : 0x100) | D;  // row_shr:D / row_shl:D
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// One step of the segmented inclusive products: lo over lanes b' <= b,
// hi over lanes b' >= b, for every slot of the group.
template <int D>
__device__ __forceinline__ void scan_step_row(double (&lo)[K3T_SLOTS], double (&hi)[K3T_SLOTS], int b, int W)
{
#pragma unroll
    for (int k = 0; k < K3T_SLOTS; ++k) {
        const double tl = row_shift<D, true>(lo[k]);
        const double th = row_shift<D, false>(hi[k]);
        if (b >= D) lo[k] *= tl;
        if (b + D < W) hi[k] *= th;
    }
}

// The running product of one trajectory's factors over its slots, for one
// risk reading (a template parameter, so the slot loop has no branch on it).
template <int RISK>
__device__ __forceinline__ double keep_of(unsigned long long v)
{
    if constexpr (RISK == RISK_EXCLUSIVE) return 1.0 - fmin((double)v * kQInvScale, 1.0);
    else return 1.0 + expm1(-(double)v * kLInvScale);
}

// Inclusive product over the lanes b' <= b of each trajectory's segment of W
// lanes (DPP row shifts for W <= 16, lane permutes for W = 32, 64).
__device__ __forceinline__ double segment_product(double x, int b, int W)
{
    if (W <= 16) {
        double t;
        if (W > 1) { t = row_shift<1, true>(x); if (b >= 1) x *= t; }
        if (W > 2) { t = row_shift<2, true>(x); if (b >= 2) x *= t; }
        if (W > 4) { t = row_shift<4, true>(x); if (b >= 4) x *= t; }
        if (W > 8) { t = row_shift<8, true>(x); if (b >= 8) x *= t; }
        return x;
    }
    for (int d = 1; d < W; d <<= 1) {
        const double t = __shfl_up(x, d, W);
        if (b >= d) x *= t;
    }
    return x;
}

// Slots [s_begin, s_end) of trajectory (a, i), lane b, from the running sum
// Q of all slots before s_begin (the last lane of the segment also gets
// all_carry = prod_b f_b(s_begin - 1)). Writes the criticality of these
// slots and returns this lane's attribution terms over them; the sums of
// each group of slots are loaded one group ahead of their use.
template <int RISK>
__device__ __forceinline__ double timeline_chunk(const DObj &o, const unsigned long long *__restrict__ hist,
                                                 double *__restrict__ ct_w, double *__restrict__ traj_crit_t, int i,
                                                 int b, int W, int s_begin, int s_end, unsigned long long Q,
                                                 double all_carry)
{
    const int H = o.H;
    const int64_t T = o.T;
    const bool valid = i < o.T && b < o.n_scene_obj;
    const bool writer = b == W - 1 && i < o.T;
    const int64_t slot_stride = T * W;
    if (s_begin >= s_end) return 0.0;
    // every lane loads (padding lanes b >= n hold zeros; lanes past the last
    // trajectory read trajectory 0 and slots past the chunk read its last
    // slot), and the values that do not belong to the lane are masked: no
    // branch per load
    const unsigned long long *__restrict__ h = hist + o.hist_off + (int64_t)(i < o.T ? i : 0) * W + b;
    double f_carry = valid ? keep_of<RISK>(Q) : 1.0, A = 0.0;
    const int last = s_end - 1;
    unsigned long long v[K3T_SLOTS];
#pragma unroll
    for (int k = 0; k < K3T_SLOTS; ++k) v[k] = h[(int64_t)min(s_begin + k, last) * slot_stride];
    for (int s0 = s_begin; s0 < s_end; s0 += K3T_SLOTS) {
        unsigned long long vn[K3T_SLOTS];
#pragma unroll
        for (int k = 0; k < K3T_SLOTS; ++k) vn[k] = h[(int64_t)min(s0 + K3T_SLOTS + k, last) * slot_stride];
        bool change = false;
#pragma unroll
        for (int k = 0; k < K3T_SLOTS; ++k) change |= valid && s0 + k < s_end && v[k] != 0ull;
        if (!__any(change)) {
            // no first hit in these slots for any trajectory of the wave: the
            // factors, the attribution and the criticality stay as they are
            if (writer) {
#pragma unroll
                for (int k = 0; k < K3T_SLOTS; ++k) {
                    const int s = s0 + k;
                    if (s < s_end) {
                        ct_w[o.tl_traj + (int64_t)s * T + i] = 1.0 - all_carry;
                        if (traj_crit_t) traj_crit_t[o.tl_traj + (int64_t)i * H + s] = 1.0 - all_carry;
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < K3T_SLOTS; ++k) v[k] = vn[k];
            continue;
        }
        // factors after (g) and before (f) each slot; slots past the chunk repeat the last
        double g[K3T_SLOTS], f[K3T_SLOTS];
#pragma unroll
        for (int k = 0; k < K3T_SLOTS; ++k) {
            f[k] = k == 0 ? f_carry : g[k - 1];
            Q += (valid && s0 + k < s_end) ? v[k] : 0ull;
            g[k] = valid ? keep_of<RISK>(Q) : 1.0;
        }
        f_carry = g[K3T_SLOTS - 1];
        double lo[K3T_SLOTS], hi[K3T_SLOTS];
#pragma unroll
        for (int k = 0; k < K3T_SLOTS; ++k) {
            lo[k] = g[k];
            hi[k] = f[k];
        }
        double below[K3T_SLOTS], above[K3T_SLOTS];
        if (W <= 16) {
            if (W > 1) scan_step_row<1>(lo, hi, b, W);
            if (W > 2) scan_step_row<2>(lo, hi, b, W);
            if (W > 4) scan_step_row<4>(lo, hi, b, W);
            if (W > 8) scan_step_row<8>(lo, hi, b, W);
#pragma unroll
            for (int k = 0; k < K3T_SLOTS; ++k) {
                below[k] = row_shift<1, true>(lo[k]);
                above[k] = row_shift<1, false>(hi[k]);
            }
        } else {
            for (int d = 1; d < W; d <<= 1) {
#pragma unroll
                for (int k = 0; k < K3T_SLOTS; ++k) {
                    const double tl = __shfl_up(lo[k], d, W);
                    const double th = __shfl_down(hi[k], d, W);
                    if (b >= d) lo[k] *= tl;
                    if (b + d < W) hi[k] *= th;
                }
            }
#pragma unroll
            for (int k = 0; k < K3T_SLOTS; ++k) {
                below[k] = __shfl_up(lo[k], 1, W);
                above[k] = __shfl_down(hi[k], 1, W);
            }
        }
#pragma unroll
        for (int k = 0; k < K3T_SLOTS; ++k) {
            const double bl = b > 0 ? below[k] : 1.0;      // inclusive -> exclusive
            const double ab = b + 1 < W ? above[k] : 1.0;
            A += (f[k] - g[k]) * bl * ab;                   // 0 past the chunk: f == g there
        }
        if (writer) {  // lo at the last lane = prod_b f_b(s)
#pragma unroll
            for (int k = 0; k < K3T_SLOTS; ++k) {
                const int s = s0 + k;
                if (s < s_end) {
                    ct_w[o.tl_traj + (int64_t)s * T + i] = 1.0 - lo[k];
                    if (traj_crit_t) traj_crit_t[o.tl_traj + (int64_t)i * H + s] = 1.0 - lo[k];
                }
            }
        }
        all_carry = lo[K3T_SLOTS - 1];
#pragma unroll
        for (int k = 0; k < K3T_SLOTS; ++k) v[k] = vn[k];
    }
    return A;
}

// K3t: grid y = object, x = group of 64 / W trajectories, lane = (trajectory,
// b); the four waves of a workgroup take the same lanes and split the slots
// into four consecutive chunks, so that every trajectory's slots are walked
// by four waves side by side. Wave c first adds up the per-slot sums of its
// chunk (one load per slot and lane); after a barrier it starts from the sums
// of the chunks before it (added in chunk order), their factors and, in the
// segment's last lane, their product, and walks its chunk: slots go in
// groups of K3T_SLOTS, the lanes load the group's sums (one group ahead),
// form the running sums and factors, and the segment of W lanes of every
// trajectory forms, for all slots of the group at once (independent chains,
// so their latencies overlap), the products of the factors below b (new) and
// above b (old): DPP row shifts for W <= 16, lane permutes for W = 32, 64.
// Lane b then adds its attribution terms; the last lane of the segment holds
// prod_b f_b(s). After a second barrier wave 0 adds the four chunks'
// attribution terms in chunk order. Writes the criticality over time as
// [s][i] scratch (and traj_crit_t (i, s) if asked for), the attribution as
// [b][i] scratch (and (i, b) if asked for), and the total sums of every b
// into the integer accumulators k3_crit reads. Timeline scenes have at most
// 64 objects.
__global__ __launch_bounds__(WG) void k3_timeline(const DObj *__restrict__ objs,
                                                  const unsigned long long *__restrict__ hist,
                                                  unsigned long long *__restrict__ qacc, double *__restrict__ att_w,
                                                  double *__restrict__ ct_w, double *__restrict__ traj_crit_t,
                                                  double *__restrict__ traj_attrib)
{
    constexpr int CHUNKS = WG / WAVE;
    __shared__ unsigned long long chunk_sum[CHUNKS][WAVE];
    __shared__ double chunk_att[CHUNKS][WAVE];
    const DObj o = objs[blockIdx.y];
    if (!o.timeline) return;  // whole workgroup
    const int W = o.tl_w;
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    const int c = (int)(threadIdx.x / WAVE);
    const int per_wave = WAVE / W;
    const int first_i = (int)blockIdx.x * per_wave;
    if (first_i >= o.T) return;  // whole workgroup: every lane below takes part in the exchanges
    const int i = first_i + lane / W;
    const int b = lane & (W - 1);
    const bool valid = i < o.T && b < o.n_scene_obj;
    const int H = o.H;
    const int len = (H + CHUNKS - 1) / CHUNKS;
    const int s_begin = min(c * len, H), s_end = min(s_begin + len, H);
    // this chunk's sums, eight loads in flight at a time
    const unsigned long long *__restrict__ h = hist + o.hist_off + (int64_t)(i < o.T ? i : 0) * W + b;
    const int64_t slot_stride = (int64_t)o.T * W;
    unsigned long long sum = 0ull;
    for (int s0 = s_begin; s0 < s_end; s0 += 8) {
        unsigned long long v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = h[(int64_t)min(s0 + k, s_end - 1) * slot_stride];
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += s0 + k < s_end ? v[k] : 0ull;
    }
    chunk_sum[c][lane] = valid ? sum : 0ull;
    __syncthreads();
    unsigned long long Q = 0ull;
    for (int k = 0; k < c; ++k) Q += chunk_sum[k][lane];
    const double f0 =
        valid ? (o.risk == RISK_EXCLUSIVE ? keep_of<RISK_EXCLUSIVE>(Q) : keep_of<RISK_INDEPENDENT>(Q)) : 1.0;
    const double all_carry = segment_product(f0, b, W);
    const double A = o.risk == RISK_EXCLUSIVE
                         ? timeline_chunk<RISK_EXCLUSIVE>(o, hist, ct_w, traj_crit_t, i, b, W, s_begin, s_end, Q,
                                                          all_carry)
                         : timeline_chunk<RISK_INDEPENDENT>(o, hist, ct_w, traj_crit_t, i, b, W, s_begin, s_end, Q,
                                                            all_carry);
    chunk_att[c][lane] = A;
    __syncthreads();
    if (c != 0 || !valid) return;
    double At = 0.0;
    unsigned long long Qt = 0ull;
    for (int k = 0; k < CHUNKS; ++k) {
        At += chunk_att[k][lane];
        Qt += chunk_sum[k][lane];
    }
    const int n = o.n_scene_obj;
    qacc[o.q_row + (int64_t)i * n + b] = Qt;
    att_w[o.q_row + (int64_t)b * o.T + i] = At;
    if (traj_attrib) traj_attrib[o.q_row + (int64_t)i * n + b] = At;
}

// Sum of a double over the 64 lanes of a wave in a fixed butterfly order.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = WAVE / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}

// K4t: grid x = object, y = row: rows 0..H-1 are the slots (C_a(s)), rows
// H..H+n-1 the collision objects (A_{a,b}). Thread t adds p_{a,i} times the
// trajectory value over i = t, t + 256, ... in ascending order (loads four
// ahead), and the workgroup adds the 256 partial sums in a fixed order
// (block_sum): every sum has a fixed order.
__global__ __launch_bounds__(WG) void k4_timeline(const DObj *__restrict__ objs, const double *__restrict__ p,
                                                  const double *__restrict__ ct_w, const double *__restrict__ att_w,
                                                  double *__restrict__ crit_t, double *__restrict__ attrib)
{
    __shared__ double red[WG / WAVE];
    const DObj o = objs[blockIdx.x];
    if (!o.timeline) return;
    const int row = (int)blockIdx.y;
    const int n = o.n_scene_obj, H = o.H, T = o.T;
    if (row >= H + n) return;  // whole workgroup
    const int tid = (int)threadIdx.x;
    const double *__restrict__ pp = p + o.traj_off;
    const double *__restrict__ r =
        row < H ? ct_w + o.tl_traj + (int64_t)row * T : att_w + o.q_row + (int64_t)(row - H) * T;
    double acc = 0.0;
    for (int base = 0; base < T; base += 4 * WG) {
        double x[4], w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int idx = base + k * WG + tid;
            x[k] = idx < T ? r[idx] : 0.0;
            w[k] = idx < T ? pp[idx] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (base + k * WG + tid < T) acc += w[k] * x[k];
    }
    const double total = block_sum(acc, red);
    if (tid != 0) return;
    if (row < H)
        crit_t[o.tl_obj + row] = total;
    else
        attrib[o.tl_att + (row - H)] = total;
}

// ===========================================================================
// Launchers
// ===========================================================================

// 16-byte words of the first hits that each of n workgroups writes
static int64_t hits_per_workgroup(const Launch &L, int64_t n) { return (L.n_hits / 8 + n - 1) / n; }

hipError_t launch_trajgen(const Launch &L, hipStream_t s)
{
    if (L.n_obj <= 0) return hipSuccess;
    const int64_t per_wg = hits_per_workgroup(L, (int64_t)L.k1_x * L.k1_nrows);
    if (L.one_track)
        hipLaunchKernelGGL(k1_trajgen<true>, dim3(L.k1_x, L.k1_nrows), dim3(K1_WG), 0, s, L.objs, L.vals, L.poses, L.p,
                           L.pfix, L.qacc, L.done, L.hist, L.k1_rows, L.hits, L.n_hits, per_wg);
    else
        hipLaunchKernelGGL(k1_trajgen<false>, dim3(L.k1_x, L.k1_nrows), dim3(K1_WG), 0, s, L.objs, L.vals, L.poses, L.p,
                           L.pfix, L.qacc, L.done, L.hist, L.k1_rows, L.hits, L.n_hits, per_wg);
    return hipGetLastError();
}

static hipError_t launch_clear_hits(const Launch &L, hipStream_t s)
{
    if (!L.hits || L.n_hits <= 0) return hipSuccess;
    // 16 KB a workgroup, at most 8 workgroups a CU
    const int64_t blocks = std::min<int64_t>((L.n_hits * 2 + (16 << 10) - 1) / (16 << 10), 2048);
    hipLaunchKernelGGL(k2_clear, dim3((unsigned)blocks), dim3(WG), 0, s, L.hits, L.n_hits, hits_per_workgroup(L, blocks));
    return hipGetLastError();
}

static uint32_t k2_sizes(const Launch &L)
{
    return (uint32_t)L.strip_len | (uint32_t)L.side_shift << 8 | (uint32_t)L.item_shift << 16;
}

template <int V, int FAM, bool TL>
static hipError_t launch_k2(const Launch &L, hipStream_t s)
{
    int64_t lo = 0, hi = L.n_strips;
    if (L.collide_parts > 0) {
        if (L.part_lo < 0 || L.part_hi > L.collide_parts || L.part_lo > L.part_hi) return hipErrorInvalidValue;
        lo = strips_before_part(L.n_strips, L.part_lo, L.collide_parts);
        hi = strips_before_part(L.n_strips, L.part_hi, L.collide_parts);
    }
    if (lo == hi) return hipSuccess;
    if (L.n_strips / L.k2_grid >= INT_MAX - K2_WG) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k2_collide<V, FAM, TL>), dim3(L.k2_grid), dim3(K2_WG), 0, s, L.pairs, L.objs, L.strip0, L.n_pairs,
                       lo, (int)((hi - lo) / L.k2_grid), (int)((hi - lo) % L.k2_grid), k2_sizes(L), L.poses, L.hits,
                       L.pfix, L.qacc, L.hist, L.polys);
    return hipGetLastError();
}

template <int V, int FAM, bool TL>
static int k2_resident_blocks()
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k2_collide<V, FAM, TL>, K2_WG, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    return per_cu;
}

// The kernel instance of (variant, class family, per-slot sums):
// F::run<V, FAM, TL>() is called for the instance.
template <int FAM, bool TL, class F>
static auto with_variant(int variant, const F &f)
{
    switch (variant) {
    case 0: return f.template run<0, FAM, TL>();
    case 1: return f.template run<1, FAM, TL>();
    case 2: return f.template run<2, FAM, TL>();
    default: return f.template run<3, FAM, TL>();
    }
}

template <int FAM, class F>
static auto with_timeline(int variant, bool tl, const F &f)
{
    return tl ? with_variant<FAM, true>(variant, f) : with_variant<FAM, false>(variant, f);
}

template <class F>
static auto with_instance(int variant, int family, bool tl, const F &f)
{
    switch (family) {
    case FAM_PLAIN: return with_timeline<FAM_PLAIN>(variant, tl, f);
    case FAM_PIP: return with_timeline<FAM_PIP>(variant, tl, f);
    default: return with_timeline<FAM_POLY>(variant, tl, f);
    }
}

struct LaunchK2 {
    const Launch &L;
    hipStream_t s;
    template <int V, int FAM, bool TL>
    hipError_t run() const { return launch_k2<V, FAM, TL>(L, s); }
};

struct ResidentK2 {
    template <int V, int FAM, bool TL>
    int run() const { return k2_resident_blocks<V, FAM, TL>(); }
};

hipError_t launch_collide(const Launch &L, hipStream_t s)
{
    if (L.n_strips <= 0) return hipSuccess;
    if (L.variant < 0 || L.variant >= N_VARIANTS || L.family < FAM_PLAIN || L.family > FAM_POLY || L.k2_grid < 1 ||
        L.strip_len < 1 || L.strip_len > MAX_STRIP || L.side_shift < 0 || 1 << L.side_shift > BLOCK_SIDE ||
        L.item_shift < 0 || 1 << L.item_shift > WAVE)
        return hipErrorInvalidValue;
    if (L.clear_hits) {
        const hipError_t e = launch_clear_hits(L, s);
        if (e != hipSuccess) return e;
    }
    return with_instance(L.variant, L.family, L.timeline != 0, LaunchK2{L, s});
}

int collide_blocks_per_cu(int variant, int family, bool timeline, bool waves)
{
    return with_instance(variant, family, timeline, ResidentK2{}) * (waves ? K2_WG / WAVE : 1);
}

// ===========================================================================
// Workspace of the allocation-free entry point (mhc_evaluate_noalloc): a
// file-scope device array, one copy on every GPU, held until the process
// ends. Host code must not pass its name to a kernel (on the host it is a
// stand-in, not a device address); noalloc_scratch_address looks up this
// GPU's address once, with the device current, and every later use goes
// through that address.
// ===========================================================================

static __device__ __align__(256) char noalloc_scratch[kNoallocBytes];

hipError_t noalloc_scratch_address(int device, char **out)
{
    static std::mutex mu;
    static char *addr[kMaxDevices] = {};
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;  // the caller makes `device` current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch));
        if (e != hipSuccess) return e;
        if (!p || reinterpret_cast<uintptr_t>(p) % 256 != 0) return hipErrorInvalidSymbol;
        addr[device] = static_cast<char *>(p);
    }
    *out = addr[device];
    return hipSuccess;
}

hipError_t launch_risk(const Launch &L, hipStream_t s)
{
    if (L.n_obj <= 0) return hipSuccess;
    if (L.timeline) {
        hipLaunchKernelGGL(k3_timeline, dim3(L.k3t_x, L.n_obj), dim3(WG), 0, s, L.objs, L.hist, L.qacc, L.att_w,
                           L.ct_w, L.traj_crit_t, L.traj_attrib);
        hipLaunchKernelGGL(k4_timeline, dim3(L.n_obj, L.k4t_y), dim3(WG), 0, s, L.objs, L.p, L.ct_w, L.att_w,
                           L.crit_t, L.attrib);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k3_crit, dim3(L.k3_x, L.n_obj), dim3(WG), 0, s, L.objs, L.qacc, L.p, L.q, L.traj_crit,
                       L.obj_crit, L.done);
    return hipGetLastError();
}

}  // namespace mhc
