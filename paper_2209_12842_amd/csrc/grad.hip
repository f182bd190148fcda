// Gradient of the free energy with respect to the mean sequence, on the
// device.  J(V) = -lambda log((1/K) sum_k exp(-S~_k/lambda)) with the noise
// fixed, and dJ/dV = sum_k w_hat_k dS~_k/dV, where (Eq. 14-19)
//   dS~_k = dS_k + A 1[CVaR_k > C_u] (1/n_tail) sum_tail (B dL_m + (1 - B) dLbar).
// After the forward rollout (which records each draw's rank in its sample)
// and the update in gradient mode (which writes J, w_hat and the list of
// samples of non-zero weight), k_grad_rollouts takes every (weighted sample,
// rollout that reaches its gradient): the nominal rollout and the tail draws
// (every draw when B != 1).  Each is recomputed from the same Philox
// counters, keeping its states, the adjoint (backward) recursion of the Euler
// steps runs over them, and the coefficient times dCost/dV is written as one
// row: by one lane per rollout, or where the rollouts are few, with their
// steps shared out over lanes (grad_rows_by_time).  k_grad_reduce adds the
// rows in a fixed order.  Indicators (collisions, the C_u test, tail membership) have
// zero gradient almost everywhere; du/dv is 1 strictly inside the box for
// warm samples and 0 otherwise.
#include <algorithm>

#include "launch.h"
#include "step_device.h"

namespace ramppi {

// du/dv of sample k at step t, per component (1 strictly inside the box for
// warm samples, else 0), from the same control draw as sample_control; v is
// (v_t0, v_t1).
// Computed in every lane and selected (no branch).
__device__ __forceinline__ float2 control_jacobian(const StepConst& c, float2 v, int k, int t) {
    const uint4 r = philox4x32_10((uint32_t)t, kCtrlWord, (uint32_t)k, c.step_idx, c.key0, c.key1);
    float z0, z1;
    box_muller(uniform01(r.x), uniform01(r.y), z0, z1);
    const float a = __fmaf_rn(c.se0, z0, v.x);
    const float d = __fmaf_rn(c.se1, z1, v.y);
    const bool warm = k < c.n_warm;
    return make_float2((warm && a > c.u_lo0 && a < c.u_hi0) ? 1.0f : 0.0f,
                       (warm && d > c.u_lo1 && d < c.u_hi1) ? 1.0f : 0.0f);
}

// What a row (weighted sample, rollout) is: its sample, its draw (-1: the
// nominal rollout) and its coefficient.
struct GradRow {
    int k, m;
    float coef;
};

__device__ __forceinline__ GradRow grad_row(const StepConst& c, const GradArgs& a, int l) {
    const int slot = l / a.R;
    const int j = l - slot * a.R;
    GradRow r;
    r.k = a.act_list[slot];
    const float wk = a.w_hat[r.k];
    r.m = -1;
    if (j == 0) {
        r.coef = wk;
    } else {
        const bool risk = (a.cvar[r.k] > c.C_u) && (c.A != 0.0f);
        if (!c.scale_risk) {
            r.m = a.tail_idx[(size_t)r.k * c.n_tail + (j - 1)];
            r.coef = risk ? wk * c.A / (float)c.n_tail : 0.0f;
        } else {
            r.m = j - 1;
            const bool in_tail = a.ranks[(size_t)r.k * c.M + r.m] < c.n_tail;
            r.coef =
                risk ? wk * c.A * ((in_tail ? c.B / (float)c.n_tail : 0.0f) + (1.0f - c.B) / (float)c.M) : 0.0f;
        }
    }
    return r;
}

// ---- few rows: the steps of a rollout side by side ----
//
// A rollout is a chain of T steps forward and T back, but little of a step
// belongs to the chain: the draws, controls and steering tangents do not
// depend on the state at all; heading and speed form a chain of their own (a
// few fused multiply-adds per step); sines and cosines of the headings are
// then independent; the positions are a second chain; cost gradients and the
// coefficients of the adjoint are independent again; the adjoint is a third
// chain; the control Jacobians and outputs are independent.  A workgroup
// takes kTimeRows rows and kTimeTile steps at a time: what is independent
// runs over (row, step) pairs in all lanes, the chains in one lane per row,
// values in LDS.  Every value is formed by the operations of the one-lane
// form in the same order.  With one lane per row and a few hundred rows the
// launch waits on the latency of 2 T whole steps (T = 50: 33.4 us for 8 rows
// as for 10 thousand; here 12.2 us for 8 rows, about 13 for 4 thousand).
constexpr int kTimeRows = 8;
constexpr int kTimeTile = 64;
constexpr int kTimeStride = kTimeTile + 1;  // LDS row stride: rows on different banks
// LDS fields per (row, step); a field's later contents follow its first
// ones: forward (kFpsi, kFv: the state's heading and speed; P_i, Q_i: the
// disturbance of component i is P_i Q_i), then the coefficients of the
// adjoint, then its heading and speed components.
enum {
    kFda, kFkap, kFp2, kFq2, kFp3, kFq3, kFp0, kFq0, kFp1, kFq1, kFpsi, kFv, kTimeFields,
    kFsn = kFda, kFcs = kFkap, kFx = kFp2, kFy = kFp3,
    kFc4 = kFda, kFc3 = kFkap, kFgx = kFp2, kFgy = kFp3, kFc5 = kFp0, kFgw = kFq0, kFgd = kFp1, kFc1 = kFpsi,
    kFc2 = kFv, kFlw = kFq1, kFlz = kFq2
};
// Largest grid of the row-by-time form for horizons of T steps; more rows than
// that fill the device with one lane each.  What a workgroup does besides its
// chains costs as much as a chain of some eight steps per row (whole gradient
// by time and by lanes: T = 5 26.2 and 24.3 us at 500 rows; T = 10 27.1 and
// 28.0, 35.5 and 36.4 at 8 thousand, 47.6 and 42.5 at 16; T = 20 30.1 and
// 35.8, 40.7 and 46.6, 54.6 and 53.0; T = 50 40.5 and 61.9, 55.1 and 74.2,
// 75.5 and 82.2, at 24 thousand 88.7 and 84.5).
__host__ __device__ constexpr int time_grid(int T) { return T < 8 ? 0 : T < 25 ? 1024 : 2048; }

template <int kNoise>
__device__ __forceinline__ void grad_rows_by_time(const StepConst& c, const GradArgs& a, int n_rows) {
    __shared__ float f[kTimeFields][kTimeRows * kTimeStride];
    __shared__ int rk[kTimeRows], rm[kTimeRows];
    __shared__ float rcoef[kTimeRows], endx[2 * kTimeRows];
    const int tid = threadIdx.x;
    const int l0 = blockIdx.x * kTimeRows;
    if (l0 >= n_rows) return;  // uniform
    if (tid < kTimeRows) {
        const GradRow r = grad_row(c, a, min(l0 + tid, n_rows - 1));  // rows past the last repeat it, unwritten
        rk[tid] = r.k;
        rm[tid] = r.m;
        rcoef[tid] = r.coef;
    }
    __syncthreads();
    const int T = c.T, K = c.K;
    const int n_tiles = (T + kTimeTile - 1) / kTimeTile;
    const float dt = c.dt;
    // the chains' lanes: row crow; axis 0 and 1 for the positions
    const int crow = tid & (kTimeRows - 1), axis = tid >> 3;
    const int cb = crow * kTimeStride;
    float psi = c.psi0, v = c.v0, pos = 0.0f;
    for (int tile = 0; tile < n_tiles; ++tile) {
        const int t0 = tile * kTimeTile, nt = min(kTimeTile, T - t0);
        // controls and disturbances (a wave per row)
        for (int i = tid; i < kTimeRows * kTimeTile; i += 256) {
            const int row = i >> 6, tt = i & 63, t = t0 + tt;
            if (tt >= nt) continue;
            const int q = row * kTimeStride + tt;
            const int k = rk[row], m = rm[row];
            const float2 uu = a.u[(size_t)t * K + k];
            f[kFda][q] = dt * uu.x;
            f[kFkap][q] = tan_steer(uu.y) * c.inv_wheelbase;
            float4 P = make_float4(0.0f, 0.0f, 0.0f, 0.0f), Q = P;
            if (m >= 0 && t + 1 < T) {
                const uint4 r = philox4x32_10((uint32_t)t, (uint32_t)m, (uint32_t)k, c.step_idx, c.key0, c.key1);
                const float4 d = disturbance_draw<kNoise>(c, r, 0x7Fu);
                if (kNoise == 0) {
                    P = make_float4(c.sw0 * d.x, c.sw1 * d.x, c.sw2 * d.y, c.sw3 * d.y);
                    Q = make_float4(__builtin_amdgcn_cosf(d.z), __builtin_amdgcn_sinf(d.z), __builtin_amdgcn_cosf(d.w),
                                    __builtin_amdgcn_sinf(d.w));
                } else if (kNoise == 1) {
                    P = make_float4(c.sw0, c.sw1, c.sw2, c.sw3);
                    Q = d;
                } else {
                    P = make_float4(d.x, d.x, 0.0f, 0.0f);
                    Q = make_float4(__builtin_amdgcn_cosf(d.y), __builtin_amdgcn_sinf(d.y), 0.0f, 0.0f);
                }
            }
            f[kFp0][q] = P.x;
            f[kFq0][q] = Q.x;
            f[kFp1][q] = P.y;
            f[kFq1][q] = Q.y;
            f[kFp2][q] = P.z;
            f[kFq2][q] = Q.z;
            f[kFp3][q] = P.w;
            f[kFq3][q] = Q.w;
        }
        __syncthreads();
        if (tid < kTimeRows) {  // heading and speed
#pragma unroll 4
            for (int tt = 0; tt < nt; ++tt) {
                const int q = cb + tt;
                f[kFpsi][q] = psi;
                f[kFv][q] = v;
                psi = __fmaf_rn(dt * v, f[kFkap][q], psi);
                {
#pragma clang fp contract(off)
                    v = v + f[kFda][q];
                }
                psi = __fmaf_rn(f[kFp2][q], f[kFq2][q], psi);
                v = __fmaf_rn(f[kFp3][q], f[kFq3][q], v);
            }
        }
        __syncthreads();
        for (int i = tid; i < kTimeRows * kTimeTile; i += 256) {
            const int q = (i >> 6) * kTimeStride + (i & 63);
            if ((i & 63) >= nt) continue;
            const float r = f[kFpsi][q] * 0.159154943091895335769f;  // as in bicycle_step
            f[kFsn][q] = __builtin_amdgcn_sinf(r);
            f[kFcs][q] = __builtin_amdgcn_cosf(r);
        }
        __syncthreads();
        if (tid < 2 * kTimeRows) {  // positions: lanes 0..7 x, 8..15 y
            const float* dir = f[axis ? kFsn : kFcs];
            const float* P = f[axis ? kFp1 : kFp0];
            const float* Q = f[axis ? kFq1 : kFq0];
            float* out = f[axis ? kFy : kFx];
#pragma unroll 4
            for (int tt = 0; tt < nt; ++tt) {
                const int q = cb + tt;
                const float d = dir[q], pp = P[q], qq = Q[q], dv = dt * f[kFv][q];
                out[q] = pos;
                pos = __fmaf_rn(dv, d, pos);
                pos = __fmaf_rn(pp, qq, pos);
            }
            if (tile + 1 == n_tiles) endx[axis * kTimeRows + crow] = pos;
        }
        __syncthreads();
        if (n_tiles > 1) {  // the states of every tile, for the way back
            for (int i = tid; i < kTimeRows * nt; i += 256) {
                const int row = i & (kTimeRows - 1), tt = i >> 3, q = row * kTimeStride + tt;
                if (l0 + row < n_rows)
                    a.states[(size_t)(t0 + tt) * a.stride + l0 + row] =
                        make_float4(f[kFx][q], f[kFy][q], f[kFpsi][q], f[kFv][q]);
            }
            __syncthreads();
        }
    }
    // backward: lam = dCost/dx_t, seeded with the terminal cost (nominal only)
    float4 lam = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (tid < kTimeRows && rm[tid] < 0 && c.use_term)
        lam = terminal_cost_grad(c, State{endx[tid], endx[kTimeRows + tid], 0.0f, 0.0f});
    for (int tile = n_tiles - 1; tile >= 0; --tile) {
        const int t0 = tile * kTimeTile, nt = min(kTimeTile, T - t0);
        for (int i = tid; i < kTimeRows * kTimeTile; i += 256) {
            const int row = i >> 6, tt = i & 63, t = t0 + tt;
            if (tt >= nt) continue;
            const int q = row * kTimeStride + tt;
            State x;
            float sn, cs;
            if (n_tiles > 1) {
                const float4 xv = a.states[(size_t)t * a.stride + min(l0 + row, n_rows - 1)];
                x = State{xv.x, xv.y, xv.z, xv.w};
                const float r = x.psi * 0.159154943091895335769f;
                sn = __builtin_amdgcn_sinf(r);
                cs = __builtin_amdgcn_cosf(r);
            } else {
                x = State{f[kFx][q], f[kFy][q], f[kFpsi][q], f[kFv][q]};
                sn = f[kFsn][q];
                cs = f[kFcs][q];
            }
            const float tnd = tan_steer(a.u[(size_t)t * K + rk[row]].y);
            const float dv = dt * x.v;
            const float4 gq = smooth_cost_grad(c, x);
            f[kFc1][q] = -dv * sn;
            f[kFc2][q] = dv * cs;
            f[kFc3][q] = dt * cs;
            f[kFc4][q] = dt * sn;
            f[kFc5][q] = dt * tnd * c.inv_wheelbase;
            f[kFgx][q] = gq.x;
            f[kFgy][q] = gq.y;
            f[kFgw][q] = gq.w;
            f[kFgd][q] = dv * __fmaf_rn(tnd, tnd, 1.0f) * c.inv_wheelbase;
        }
        __syncthreads();
        if (tid < kTimeRows) {  // the adjoint
#pragma unroll 4
            for (int tt = nt - 1; tt >= 0; --tt) {
                const int q = cb + tt;
                f[kFlw][q] = lam.w;
                f[kFlz][q] = lam.z;
                float4 nl;
                nl.x = f[kFgx][q] + lam.x;
                nl.y = f[kFgy][q] + lam.y;
                nl.z = __fmaf_rn(f[kFc1][q], lam.x, __fmaf_rn(f[kFc2][q], lam.y, lam.z));
                nl.w = f[kFgw][q] + __fmaf_rn(f[kFc3][q], lam.x,
                                              __fmaf_rn(f[kFc4][q], lam.y, __fmaf_rn(f[kFc5][q], lam.z, lam.w)));
                lam = nl;
            }
        }
        __syncthreads();
        for (int i = tid; i < kTimeRows * nt; i += 256) {
            const int row = i & (kTimeRows - 1), tt = i >> 3, t = t0 + tt, q = row * kTimeStride + tt;
            if (l0 + row >= n_rows) continue;
            const int k = rk[row];
            const float coef = rcoef[row];
            const float2 vt = make_float2(a.V[2 * t], a.V[2 * t + 1]);
            const float2 dudv = control_jacobian(c, vt, k, t);
            float g0 = dt * f[kFlw][q] * dudv.x, g1 = f[kFgd][q] * f[kFlz][q] * dudv.y;
            if (rm[row] < 0 && c.use_ctrl) {  // d/dv of gamma v^T Sigma^-1 u(v), nominal rollout only
                const float2 uu = a.u[(size_t)t * K + k];
                g0 = __fmaf_rn(c.gamma * c.inv_var0, __fmaf_rn(vt.x, dudv.x, uu.x), g0);
                g1 = __fmaf_rn(c.gamma * c.inv_var1, __fmaf_rn(vt.y, dudv.y, uu.y), g1);
            }
            a.rows[(size_t)(2 * t) * a.stride + l0 + row] = coef == 0.0f ? 0.0f : coef * g0;
            a.rows[(size_t)(2 * t + 1) * a.stride + l0 + row] = coef == 0.0f ? 0.0f : coef * g1;
        }
        __syncthreads();  // the fields are refilled
    }
}

// Steps by which the gradient rollouts load ahead of their use.
constexpr int kGradAhead = 4;

template <int kNoise>
__device__ __forceinline__ void grad_rows_by_lane(const StepConst& c, const GradArgs& a, int n_rows) {
    const int l = blockIdx.x * 256 + threadIdx.x;
    if (l >= n_rows) return;  // no barrier below
    const int T = c.T, K = c.K;
    const GradRow row = grad_row(c, a, l);
    const int k = row.k, m = row.m;
    const float coef = row.coef;
    if (coef == 0.0f) {
        for (int q = 0; q < 2 * T; ++q) a.rows[(size_t)q * a.stride + l] = 0.0f;
        return;
    }
    // forward: the rollout again, keeping its states.  Each step's loads are
    // issued kGradAhead steps ahead (a lane's chain of steps would otherwise
    // wait a memory round trip per step; the index is clamped, the extra
    // loads at the end unused); the ring of loaded values is indexed by the
    // unrolled position, so it stays in registers.  The disturbance is drawn
    // in every lane and added where it belongs (a select, not a branch), so
    // a whole run of kGradAhead steps is one block the compiler can
    // interleave.
    State s{0.0f, 0.0f, c.psi0, c.v0};
    const bool disturbed = m >= 0;
    float2 ur[kGradAhead];
#pragma unroll
    for (int i = 0; i < kGradAhead; ++i) ur[i] = a.u[(size_t)min(i, T - 1) * K + k];
    auto fstep = [&](int t, float2& slot) {
        a.states[(size_t)t * a.stride + l] = make_float4(s.x, s.y, s.psi, s.v);
        const float2 uu = slot;
        slot = a.u[(size_t)min(t + kGradAhead, T - 1) * K + k];
        bicycle_step(s, c.dt * uu.x, tan_steer(uu.y) * c.inv_wheelbase, c.dt);
        const uint4 r = philox4x32_10((uint32_t)t, (uint32_t)m, (uint32_t)k, c.step_idx, c.key0, c.key1);
        const State n = disturbed_successor<kNoise>(c, r, s);
        const bool add = disturbed && t + 1 < T;
        s.x = add ? n.x : s.x;
        s.y = add ? n.y : s.y;
        s.psi = add ? n.psi : s.psi;
        s.v = add ? n.v : s.v;
    };
    for (int tb = 0; tb < T; tb += kGradAhead) {
        if (tb + kGradAhead <= T) {
#pragma unroll
            for (int i = 0; i < kGradAhead; ++i) fstep(tb + i, ur[i]);
        } else {
#pragma unroll
            for (int i = 0; i < kGradAhead; ++i)
                if (tb + i < T) fstep(tb + i, ur[i]);
        }
    }
    // backward: lam = dCost/dx_{t}, seeded with the terminal cost (nominal
    // only); states, controls and v_t loaded kGradAhead steps ahead likewise
    float4 lam = (m < 0 && c.use_term) ? terminal_cost_grad(c, s) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float4 xr[kGradAhead];
    float2 uq[kGradAhead], vr[kGradAhead];
#pragma unroll
    for (int i = 0; i < kGradAhead; ++i) {
        const int t = max(T - 1 - i, 0);
        xr[i] = a.states[(size_t)t * a.stride + l];
        uq[i] = a.u[(size_t)t * K + k];
        vr[i] = make_float2(a.V[2 * t], a.V[2 * t + 1]);
    }
    const bool ctrl_term = m < 0 && c.use_ctrl;  // d/dv of gamma v^T Sigma^-1 u(v), nominal rollout only
    auto bstep = [&](int t, float4& xs, float2& us, float2& vs) {
        const float4 xv = xs;
        const State x{xv.x, xv.y, xv.z, xv.w};
        const float2 uu = us;
        const float2 vt = vs;
        const int tn = max(t - kGradAhead, 0);
        xs = a.states[(size_t)tn * a.stride + l];
        us = a.u[(size_t)tn * K + k];
        vs = make_float2(a.V[2 * tn], a.V[2 * tn + 1]);
        const float tnd = tan_steer(uu.y);
        const float r = x.psi * 0.159154943091895335769f;  // as in bicycle_step
        const float sn = __builtin_amdgcn_sinf(r), cs = __builtin_amdgcn_cosf(r);
        const float dt = c.dt, dv = dt * x.v;
        const float gua = dt * lam.w;                                                 // d v' / d a
        const float gud = dv * __fmaf_rn(tnd, tnd, 1.0f) * c.inv_wheelbase * lam.z;   // d psi' / d delta
        const float4 gq = smooth_cost_grad(c, x);
        float4 nl;
        nl.x = gq.x + lam.x;
        nl.y = gq.y + lam.y;
        nl.z = gq.z + __fmaf_rn(-dv * sn, lam.x, __fmaf_rn(dv * cs, lam.y, lam.z));
        nl.w = gq.w + __fmaf_rn(dt * cs, lam.x, __fmaf_rn(dt * sn, lam.y, __fmaf_rn(dt * tnd * c.inv_wheelbase,
                                                                                   lam.z, lam.w)));
        lam = nl;
        const float2 dudv = control_jacobian(c, vt, k, t);
        float g0 = gua * dudv.x, g1 = gud * dudv.y;
        const float h0 = __fmaf_rn(c.gamma * c.inv_var0, __fmaf_rn(vt.x, dudv.x, uu.x), g0);
        const float h1 = __fmaf_rn(c.gamma * c.inv_var1, __fmaf_rn(vt.y, dudv.y, uu.y), g1);
        g0 = ctrl_term ? h0 : g0;
        g1 = ctrl_term ? h1 : g1;
        a.rows[(size_t)(2 * t) * a.stride + l] = coef * g0;
        a.rows[(size_t)(2 * t + 1) * a.stride + l] = coef * g1;
    };
    for (int tb = T - 1; tb >= 0; tb -= kGradAhead) {
        if (tb - (kGradAhead - 1) >= 0) {
#pragma unroll
            for (int i = 0; i < kGradAhead; ++i) bstep(tb - i, xr[i], uq[i], vr[i]);
        } else {
#pragma unroll
            for (int i = 0; i < kGradAhead; ++i)
                if (tb - i >= 0) bstep(tb - i, xr[i], uq[i], vr[i]);
        }
    }
}

// The form of the rows.  Where the horizon or the largest number of rows leaves
// one only, its kernel holds no code of the other (T = 5, 18 thousand rows by
// lanes: 8.5 us from a kernel of both, 7.6 alone).
enum { kRowsByTime, kRowsByLane, kRowsEither };

struct GradLaunch {
    StepConst c;
    GradArgs a;
};

__device__ __forceinline__ GradArgs global_view(const GradArgs& a) {
    GradArgs g = a;
    g.V = as_global(a.V);
    g.u = as_global(a.u);
    g.cvar = as_global(a.cvar);
    g.w_hat = as_global(a.w_hat);
    g.act_list = as_global(a.act_list);
    g.n_act = as_global(a.n_act);
    g.tail_idx = as_global(a.tail_idx);
    g.ranks = as_global(a.ranks);
    g.states = as_global(a.states);
    g.rows = as_global(a.rows);
    return g;
}

template <int kNoise, int kForm>
__global__ void __launch_bounds__(256) k_grad_rollouts(GradLaunch g) {
    const int n_rows = *g.a.n_act * g.a.R;
    if constexpr (kForm == kRowsByTime) {
        grad_rows_by_time<kNoise>(g.c, g.a, n_rows);
    } else if constexpr (kForm == kRowsByLane) {
        grad_rows_by_lane<kNoise>(g.c, g.a, n_rows);
    } else {
        // each form reads the arguments again, as in RolloutLate: read once
        // for both they filled the scalar registers and spilled
        const GradLaunch* e = late_ptr<GradLaunch>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
        if (n_rows <= kTimeRows * time_grid(e->c.T))
            grad_rows_by_time<kNoise>(e->c, global_view(e->a), n_rows);
        else
            grad_rows_by_lane<kNoise>(e->c, global_view(e->a), n_rows);
    }
}

// Sum of the gradient rows: output q in workgroups (q, 0), (q, 1), ...  The
// rows are added in blocks of 256 (lane i of a wave adds rows i, i + 64,
// i + 128, i + 192 of a block, then the wave adds its lanes), each wave taking
// every n-th block of its workgroup's n waves, and one wave adds the block sums
// in block order.  Up to kReduceBlocks blocks one workgroup does it all, its
// block sums in LDS; more blocks are split over the workgroups of the output,
// which hand their sums over in memory to the last of them.  Bound by the trips
// to memory, for rows that other XCDs wrote: with as many waves as a workgroup
// can have its loads are one trip, and so are the sums of up to 1024 blocks (134
// thousand rows at T = 5 8.0 us, 16 thousand at T = 9 4.4; with four waves, 64
// sums a trip, each added from the lane that held it, 34 and 13).
constexpr int kReduceAhead = 4;   // blocks whose loads a wave has in flight
constexpr int kReduceBlocks = 64;  // block sums of one workgroup

__global__ void __launch_bounds__(1024) k_grad_reduce(GradArgs a) {
    __shared__ float sums[1024];
    __shared__ int flag_sh;
    const int n_rows = *a.n_act * a.R;
    const int nb = max(1, (n_rows + 255) / 256);
    const int q = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6, n_waves = (int)blockDim.x >> 6;
    const float* rq = a.rows + (size_t)q * a.stride;
    if (nb == 1) {
        if (wv != 0 || blockIdx.y != 0) return;
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += lane + 64 * j < n_rows ? rq[lane + 64 * j] : 0.0f;
        acc = wave_sum(acc);
        if (lane == 0) a.grad_out[q] = acc;
        return;
    }
    const bool alone = nb <= kReduceBlocks;
    const int per = alone ? nb : (nb + (int)gridDim.y - 1) / (int)gridDim.y;
    const int b0 = (int)blockIdx.y * per, b1 = min(nb, b0 + per);
    if (b0 >= b1) return;  // uniform
    float* part = a.rpart + (size_t)q * a.n_blocks;
    for (int b = b0 + wv; b < b1; b += n_waves * kReduceAhead) {
        float r[kReduceAhead][4];
#pragma unroll
        for (int i = 0; i < kReduceAhead; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int bi = b + n_waves * i, l = bi * 256 + lane + 64 * j;
                r[i][j] = (bi < b1 && l < n_rows) ? rq[l] : 0.0f;
            }
#pragma unroll
        for (int i = 0; i < kReduceAhead; ++i) {
            const int bi = b + n_waves * i;
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc += r[i][j];
            acc = wave_sum(acc);
            if (lane == 0 && bi < b1) {
                if (alone)
                    sums[bi] = acc;
                else
                    agent_store(&part[bi], acc);
            }
        }
    }
    if (alone) {
        __syncthreads();
    } else {
        // the workgroups of this output that hold blocks
        if (!arrive_last(&a.counter[q], (unsigned)((nb + per - 1) / per), &flag_sh)) return;
    }
    // one wave adds the block sums in order, eight loads in flight
    float total = 0.0f;
    for (int c0 = 0; c0 < nb; c0 += (int)blockDim.x) {
        const int nc = min((int)blockDim.x, nb - c0);
        if (!alone) {
            __syncthreads();  // the last part's sums are read
            if (tid < nc) sums[tid] = agent_load(&part[c0 + tid]);
            __syncthreads();
        }
        if (wv != 0) continue;
        int i = 0;
        for (; i + 8 <= nc; i += 8) {
            float t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) t[j] = sums[i + j];
#pragma unroll
            for (int j = 0; j < 8; ++j) total += t[j];
        }
        for (; i < nc; ++i) total += sums[i];
    }
    if (tid == 0) a.grad_out[q] = total;
}

__global__ void __launch_bounds__(256) k_update_grad(StepConst c, int G, int parts, const float* __restrict__ S,
                                                     const float* __restrict__ cvar, const float2* __restrict__ u,
                                                     float* __restrict__ S_tilde, float* part, unsigned* counter,
                                                     float* __restrict__ w_hat, GradOut go) {
    extern __shared__ float ush[];
    __shared__ float red[16];
    __shared__ int is_last;
    update_body(c, blockIdx.x, G, parts, S, cvar, u, S_tilde, part, counter, nullptr, nullptr, nullptr, w_hat, ush,
                red, &is_last, &go);
}

template <int kForm>
static hipError_t launch_grad_rollouts(const StepConst& c, const GradArgs& a, int grid, hipStream_t stream) {
    const GradLaunch g{c, a};
    if (c.noise_kind == 1)
        hipLaunchKernelGGL((k_grad_rollouts<1, kForm>), dim3(grid), dim3(256), 0, stream, g);
    else if (c.noise_kind == 2)
        hipLaunchKernelGGL((k_grad_rollouts<2, kForm>), dim3(grid), dim3(256), 0, stream, g);
    else
        hipLaunchKernelGGL((k_grad_rollouts<0, kForm>), dim3(grid), dim3(256), 0, stream, g);
    return hipGetLastError();
}

hipError_t launch_grad(const StepConst& c, const StepBuffers& b, const GradArgs& a, const GradOut& go, int block,
                       size_t lds_rollout, int G, size_t lds_update, int n_lane_blocks, hipStream_t stream) {
    const int n_dist_wg = (c.K + c.spb - 1) / c.spb;
    hipError_t e = launch_rollout(c, b, block, lds_rollout, n_dist_wg, stream, a.ranks_w, a.tail_w);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_update_grad, dim3(G), dim3(256), lds_update, stream, c, G, update_parts(c.T), b.S, b.cvar,
                       b.u, b.S_tilde, b.part, b.counter, b.w_hat, go);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t max_rows = (int64_t)c.K * a.R;
    const int n_time = (int)std::min<int64_t>(time_grid(c.T), (max_rows + kTimeRows - 1) / kTimeRows);
    e = n_time == 0 ? launch_grad_rollouts<kRowsByLane>(c, a, n_lane_blocks, stream)
        : max_rows <= (int64_t)kTimeRows * n_time
            ? launch_grad_rollouts<kRowsByTime>(c, a, n_time, stream)
            : launch_grad_rollouts<kRowsEither>(c, a, std::max(n_lane_blocks, n_time), stream);
    if (e != hipSuccess) return e;
    const int split = std::min(16, (n_lane_blocks + kReduceBlocks - 1) / kReduceBlocks);
    // enough waves for a workgroup's share of the most rows there can be
    const int share = (n_lane_blocks + split - 1) / split;
    const int waves = std::max(4, std::min(16, (share + kReduceAhead - 1) / kReduceAhead));
    hipLaunchKernelGGL(k_grad_reduce, dim3(2 * c.T, split), dim3(64 * waves), 0, stream, a);
    return hipGetLastError();
}

}  // namespace ramppi
