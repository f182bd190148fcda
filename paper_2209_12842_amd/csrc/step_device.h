// Device bodies of one RA-MPPI step, shared by the single-controller
// kernels and the batched (many-controller) kernels.
#pragma once

#include "device.h"

namespace ramppi {

// Outputs of the update in gradient mode (the free energy, the list of
// samples of non-zero weight and its length).
struct GradOut {
    float* J;
    int* act_list;
    int* n_act;
};

// Entry i of the obstacle table of a step, in the local frame centred on the
// start position (fx, fy), with cx, cy relative to it:
// (-2 cx, -2 cy, r^2 - cx^2 - cy^2, q), q = (1 + 2^-16) r^2 + 2^-15 (cx^2 + cy^2)
// the squared reach of the broad-phase test (obstacle_hits_culled); entries
// i >= n_obs are padding that no point can hit, (0, 0, -inf, -inf).
// The obstacles are three floats apart, as the caller of the step without a
// handle holds them: that step reads them where they are.
__device__ __forceinline__ float4 obstacle_entry(const float* __restrict__ obs, int n_obs, int i, float fx,
                                                 float fy) {
    if (i < n_obs) {
        const float cx = obs[3 * i] - fx;
        const float cy = obs[3 * i + 1] - fy;
        const float r = obs[3 * i + 2];
        const float c2 = __fmaf_rn(cx, cx, cy * cy);
        const float q = __fmaf_rn(1.0000152587890625f * r, r, 3.0517578125e-05f * c2);
        return make_float4(-2.0f * cx, -2.0f * cy, __fmaf_rn(r, r, -c2), q);
    }
    return make_float4(0.0f, 0.0f, -__builtin_inff(), -__builtin_inff());
}

// The group boxes of the broad phase's group skip: for each group g of 64
// table entries, the union of its discs' squares |x - cx|, |y - cy|
// <= sqrt(q), as (x0, x1, y0, y1) in gbox[g]; entries
// n_grp..63 get a box that meets nothing.  One whole wave computes them
// (lane j takes entry 64 g + j, computed as obstacle_entry computes it),
// before the barrier that precedes the rollouts.
__device__ __forceinline__ void group_bounds(const float* __restrict__ obs, int n_obs, int n_grp, float fx,
                                             float fy, float4* gbox) {
    const int lane = threadIdx.x & 63;
    const float inf = __builtin_inff();
    if (lane >= n_grp) gbox[lane] = make_float4(inf, -inf, inf, -inf);
    for (int g = 0; g < n_grp; ++g) {
        const int i = 64 * g + lane;
        const bool valid = i < n_obs;
        const float4 e = obstacle_entry(obs, n_obs, i, fx, fy);
        const float cx = -0.5f * e.x, cy = -0.5f * e.y;  // exact: e.x = -2 cx
        const float R = valid ? __builtin_amdgcn_sqrtf(e.w) : 0.0f;
        const float x0 = wave_min(valid ? cx - R : inf), x1 = wave_maxf(valid ? cx + R : -inf);
        const float y0 = wave_min(valid ? cy - R : inf), y1 = wave_maxf(valid ? cy + R : -inf);
        if (lane == 0) gbox[g] = make_float4(x0, x1, y0, y1);
    }
}

// Time steps whose points share one broad-phase box (obstacle_hits_culled):
// a longer run divides the box and group tests over more steps but widens
// the box by the distance travelled; 6 gave the shortest steps on the 50- and
// 200-obstacle tracks (horizons 50 and 100).
constexpr int kCullSteps = 6;
// CVaR of stored risk costs for tails of at most kWaveTail values, by
// workgroup wg of 256 threads: a wave per sample, or for M <= 32 a segment of
// P lanes of a wave (wave_tail_mean); the mean for the risk scaling from the
// sample's costs staged in LDS (wsh: cvar_lds_bytes).
__device__ __forceinline__ void cvar_pass(const float* __restrict__ L, int K, int M, int P, int n_tail,
                                          int scale_risk, float B, float* __restrict__ cvar_out, int wg, float* wsh) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, per = 64 / P;
    const int seg = lane / P;
    const int k = (wg * 4 + wv) * per + seg;
    const float* Lk = L + (size_t)min(k, K - 1) * M;
    float mu = 0.0f;
    if (scale_risk) {
        float* v = wsh + (size_t)(wv * per + seg) * M;
        for (int i = lane & (P - 1); i < M; i += P) v[i] = Lk[i];
        __syncthreads();
        mu = seq_sum(v, M) / (float)M;
    }
    const float cv = wave_tail_mean<true>(
        [&](int i) {
            const float x = Lk[i];
            return scale_risk ? __fmaf_rn(B, x - mu, mu) : x;
        },
        (uint32_t)lane, M, P, n_tail);
    if (k < K && (lane & (P - 1)) == 0) cvar_out[k] = cv;
}

// LDS floats of one run of sampled controls for 64 samples: (dt a, tan(delta)
// / wheelbase) and the control-cost term of each.  A nominal workgroup has a
// buffer for each of its groups of samples, or two for a single one
// (nominal_rollouts), before the obstacle table (aligned to 16 bytes).
constexpr int kNomBuf = 3 * 64 * kCullSteps;

// Arguments of a rollout kernel: one struct, the kernel's first parameter, so
// that a workgroup can read it again from the kernel-argument segment after
// its rollouts (RolloutLate).
struct RolloutArgs {
    StepConst c;
    const float* obs;
    const float* V;
    float2* u;
    float* S;
    float* cvar;
    float* L;
    int* ranks;
    int* tail_idx;
    unsigned long long* work;  // broad-phase counters, or null
    const struct FuseArgs* fa;  // the update's buffers (one-launch step)
    unsigned* clear;  // the update's counter, set to zero by a two-launch step
                      // whose workspace other steps use too, or null
};

// What a workgroup needs after its rollouts.  The compiler loads every kernel
// argument when the kernel begins and keeps in scalar registers, or spilled
// into vector-register lanes, whatever the end of the kernel uses; read again
// through a pointer it cannot see through (late_ptr), these values need no
// register while the rollouts run (with the nominal rollouts as they are now,
// scalar spills of the one-launch kernel 94 -> 57, of k_serve 164 -> 68).
struct RolloutLate {
    const StepConst* c;
    float* S;
    float* cvar;
    float* L;
    int* ranks;
    int* tail_idx;
    unsigned long long* work;
};

// p as a pointer into constant memory of unknown origin (the loads through it
// are scalar loads and stay after this point).
template <class T>
__device__ __forceinline__ const T* late_ptr(const void* p) {
    uint64_t v = (uint64_t)(uintptr_t)p;
    asm volatile("" : "+s"(v));
    return (const T*)(const __attribute__((address_space(4))) T*)(uintptr_t)v;
}

// The kernel's own arguments, read again.
__device__ __forceinline__ const RolloutArgs* late_args() {
    return late_ptr<RolloutArgs>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
}

__device__ __forceinline__ RolloutLate late_view(const RolloutArgs* a) {
    return RolloutLate{&a->c, a->S, a->cvar, a->L, a->ranks, a->tail_idx, a->work};
}

// LDS layout of k_rollout (dynamic shared memory, in this order):
//   float2 ctl[spb * T]   (dt a, tan(delta) / wheelbase) of the WG's samples
//   float  vals[spb * M]  risk costs of the WG's samples
//   float  tail[spb * M]  tail slots (descending)
//   float  means[spb]     mean risk cost per sample (risk scaling)
//   float4 otab[64 n_grp] the obstacle table, padded to groups of 64 entries
//                         (16-byte aligned; n_grp = ceil(n_obs / 64))
//   float4 gbox[64]       the groups' boxes for the group skip (group_bounds)
// Nominal workgroups keep their runs of sampled controls (kNomBuf floats each)
// before otab instead.  rollout_otab_offset gives the offset of otab in
// floats.  Every workgroup writes otab and gbox from the raw obstacles before
// its rollouts.
__host__ __device__ __forceinline__ int rollout_otab_offset(int spb, int T, int M, int nom_groups) {
    const int dist = (2 * spb * T + 2 * spb * M + spb + 3) & ~3;
    const int nom = (nom_groups > 1 ? nom_groups : 2) * kNomBuf;
    return dist > nom ? dist : nom;
}

__host__ __device__ __forceinline__ int rollout_n_grp(int n_obs) { return (n_obs + 63) >> 6; }

// Compile-time switches for the per-step lambdas of the rollouts.
struct BoolTrue {
    static constexpr bool value = true;
};
struct BoolFalse {
    static constexpr bool value = false;
};
constexpr BoolTrue kTrue{};
constexpr BoolFalse kFalse{};

// Slots of the broad-phase work counters (wave w of item i adds to slot
// (16 i + w) mod kWorkSlots, spreading the atomics): exact tests in
// work[0..kWorkSlots), group tests in work[kWorkSlots..2 kWorkSlots).
constexpr int kWorkSlots = 256;
// Scal, Max and Average of Algorithm 1 for the spb samples of a workgroup.
// vals holds the raw risk costs (thread tid owns slot tid for tid < spb * M);
// returns the CVaR in the m == 0 lane of each sample.  The descending order
// of a sample's M costs (equal costs by smaller draw index) comes from a
// bitonic sort in registers when M is a power of two and the workgroup is
// exactly spb * M lanes (stages within a wave through lane exchanges, wider
// ones through LDS), otherwise from counting each cost's rank in LDS.  Either
// way the n_tail largest land in tail[0..n_tail-1] in that order and are
// summed in it, so both give the same bits.  pos_out / id_out receive one
// (position, draw index) pair of the sorted order per lane; together the
// lanes of a sample cover every draw once.  tid is the thread's index in the
// workgroup (a caller may pass a copy the compiler cannot tie to values it
// derived from the index earlier).
// kNanFirst: see tail_rank_scatter (the sort leaves such values anywhere).
template <bool kNanFirst = false>
__device__ __forceinline__ float cvar_epilogue(float* vals, float* tail, float* means, int spb, int M,
                                               int n_tail, int scale_risk, float B, int* pos_out = nullptr,
                                               int* id_out = nullptr, int tid = (int)threadIdx.x) {
    const int sl = tid / M;
    const int m = tid - sl * M;
    const bool own = sl < spb;
    __syncthreads();  // vals and tail initialisation visible
    if (scale_risk) {
        if (own && m == 0) {
            float s = 0.0f;
            for (int j = 0; j < M; ++j) s += vals[sl * M + j];
            means[sl] = s / (float)M;
        }
        __syncthreads();
        if (own) {
            const float mu = means[sl];
            vals[tid] = __fmaf_rn(B, vals[tid] - mu, mu);
        }
        __syncthreads();
    }
    if ((M & (M - 1)) == 0 && (int)blockDim.x == spb * M) {
        float v = vals[tid];  // every lane owns a slot
        int id = m;
        for (int k = 2; k <= M; k <<= 1) {
            for (int j = k >> 1; j >= 64; j >>= 1) {  // partner in another wave
                int* ids = reinterpret_cast<int*>(tail);
                __syncthreads();
                vals[tid] = v;
                ids[tid] = id;
                __syncthreads();
                bitonic_cx(v, id, vals[tid ^ j], ids[tid ^ j], m, j, k);
            }
            bitonic_wave_stages(v, id, m, k);
        }
        __syncthreads();  // tail free again
        if (m < n_tail) tail[tid] = v;
        if (pos_out) *pos_out = m;
        if (id_out) *id_out = id;
    } else if (own) {
        const int rank = tail_rank_scatter<kNanFirst>(vals + sl * M, tail + sl * M, M, m, n_tail);
        if (pos_out) *pos_out = rank;
        if (id_out) *id_out = m;
    }
    __syncthreads();
    float cv = 0.0f;
    if (own && m == 0) cv = tail_sum(tail + sl * M, n_tail);
    return cv;
}

// The same CVaR for tails of at most kWaveTail values, when nothing but the
// mean is wanted (the gradient also records every draw's place): samples are
// sorted inside single waves (wave_tail_mean), values alone.  The raw costs
// are in vals (slot sl M + m, stored by the caller); sample sl is taken by
// the wave and segment it maps to, which for M a power of two up to 64 (and
// a workgroup of spb M lanes) is the one that stored it, so no barrier is
// needed.  store(sl, cvar) is called by one lane per sample.  Bound by the
// chain of exchanges: at K = 2048, M = 64 the epilogue takes 1.9 us instead
// of the 3.5 us of the sort with draw indices, and for M not a power of two
// it replaces M comparisons per lane (K = 8333, T = 20, M = 120: step 82.0 ->
// 73.1 us).  Taken where the waves hold all samples at once (wave_tails_pay).
template <class Store>
__device__ __forceinline__ void cvar_waves(const float* vals, int spb, int M, int n_tail, int scale_risk, float B,
                                           int tid, Store store) {
    const int P = tail_lanes(M);
    const int lane = tid & 63;
    if (P == M && (int)blockDim.x == spb * M)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    else
        __syncthreads();
    const int per = 64 / P, n_waves = (int)blockDim.x >> 6;
#pragma clang loop unroll(disable)
    for (int s0 = (tid >> 6) * per; s0 < spb; s0 += n_waves * per) {
        const int sl = min(s0 + lane / P, spb - 1);
        const float* v = vals + sl * M;
        float mu = 0.0f;
        if (scale_risk) mu = seq_sum(v, M) / (float)M;
        const float cv = wave_tail_mean<false>(
            [&](int i) {
                const float x = v[i];
                return scale_risk ? __fmaf_rn(B, x - mu, mu) : x;
            },
            (uint32_t)lane, M, P, n_tail);
        if ((lane & (P - 1)) == 0 && s0 + lane / P < spb) store(sl, cv);
    }
}

// The forms of a kernel's nominal workgroups.
constexpr int kNomSplit = 0;   // nominal_rollouts, one group of 64 samples
constexpr int kNomOwn = 1;     // nominal_rollouts with kOwn: any number of groups
constexpr int kNomDirect = 2;  // nominal_rollouts_packed: any number of groups

// The nominal rollouts of a workgroup, one sample per lane, in runs of
// kCullSteps steps whose sampled controls pass through LDS (lanes past K repeat
// the last sample, since the obstacle test works on whole waves, and write
// nothing).  Two forms:
//  - one group of 64 samples: the first wave rolls them out while the other
//    waves draw the controls of the next run, one barrier per run.  The
//    rollouts are a chain of T steps bound by latency and by the issue slots
//    that the disturbed waves leave, and drawing the controls (Philox,
//    Box-Muller, the steering tangent) is 60 % of a nominal step's
//    instructions: moved off the chain, the nominal rollouts of K = 2048,
//    T = 50, M = 64 end at 27 us of the launch instead of 35 us and no longer
//    finish last (step 37.2 -> 33.4 us with RolloutLate).
//  - nom_groups > 1 (kOwn): each of the first nom_groups waves draws the
//    controls of 64 samples of its own, a run at a time, and rolls them out.
//    For served steps whose grid would not be resident at once otherwise
//    (K = 3900, T = 50, M = 64: served step 64.1 us; the groups one after the
//    other in the first form 68.2).
template <bool kOwn, class Mean, class Late>
__device__ __forceinline__ void nominal_rollouts(const StepConst& c, const Mean& V,
                                                 float2* __restrict__ u_out, int item, float2* smem,
                                                 const float4* otab, const float4* gbox, int n_grp, int& n_cand,
                                                 int& n_gtest, Late late) {
    float* buf = reinterpret_cast<float*>(smem);
    const int T = c.T;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n_waves = (int)blockDim.x >> 6;  // at least 3 (spb M > 128)
    const int n_runs = (T + kCullSteps - 1) / kCullSteps;
    const bool own = kOwn && c.nom_groups > 1;
    const int k0 = (item * c.nom_groups + (own ? wave : 0)) * 64;
    const bool rolls = own ? wave < c.nom_groups && k0 < c.K : wave == 0;
    const int k = k0 + lane;
    const bool act = k < c.K;
    const int kc = act ? k : c.K - 1;
    if (own) buf += wave * kNomBuf;
    // the controls of run r, its steps shared out over `count` waves
    const auto produce = [&](int r, int first, int count) {
        float* b = buf + (own ? 0 : (r & 1) * kNomBuf);
        for (int i = first; i < kCullSteps; i += count) {
            const int t = r * kCullSteps + i;
            if (t >= T) break;  // uniform
            const float2 u = sample_control(c, V, kc, t);
            if (c.store_u && act) u_out[(size_t)t * c.K + k] = u;
            reinterpret_cast<float2*>(b)[i * 64 + lane] = make_float2(c.dt * u.x, tan_steer(u.y) * c.inv_wheelbase);
            b[2 * 64 * kCullSteps + i * 64 + lane] =
                __fmaf_rn(V[2 * t] * c.inv_var0, u.x, V[2 * t + 1] * c.inv_var1 * u.y);
        }
    };
    if (!own) produce(0, wave, n_waves);
    __syncthreads();  // the first run's controls, and the table, staged
    const float4 first = n_grp > 0 ? (n_grp == 1 ? otab : gbox)[lane] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    State s{0.0f, 0.0f, c.psi0, c.v0};
    float acc = 0.0f, ctrl = 0.0f;
    int cnt = 0;
    const StepConst cn = with_vector_constants(c);
    const float gamma = in_vgpr(c.gamma);
    for (int r = 0; r < n_runs; ++r) {
        if (own ? rolls : wave != 0 && r + 1 < n_runs) {
            produce(own ? r : r + 1, own ? 0 : wave - 1, own ? 1 : n_waves - 1);
            if (own) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // every lane reads what it wrote itself
        }
        if (rolls) {
            const float* b = buf + (own ? 0 : (r & 1) * kNomBuf);
            // one nominal state step: running and control costs at x_t (the
            // control cost is summed in every case and used when asked, so
            // that the step holds no branch), then x_{t+1}
            auto step = [&](auto bdry, int i, float& px, float& py) {
                acc = smooth_cost_acc<decltype(bdry)::value>(cn, s, acc);
                px = s.x;
                py = s.y;
                const float2 cu = reinterpret_cast<const float2*>(b)[i * 64 + lane];
                ctrl = __fmaf_rn(gamma, b[2 * 64 * kCullSteps + i * 64 + lane], ctrl);
                bicycle_step(s, cu.x, cu.y, cn.dt);
            };
            float px[kCullSteps], py[kCullSteps];
            if ((r + 1) * kCullSteps <= T) {  // a whole run of steps with no branch between them
                if (c.use_bdry) {
#pragma unroll
                    for (int i = 0; i < kCullSteps; ++i) step(kTrue, i, px[i], py[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < kCullSteps; ++i) step(kFalse, i, px[i], py[i]);
                }
                if (n_grp > 0)
                    cnt += obstacle_hits_culled<kCullSteps>(otab, n_grp, first, px, py, kCullSteps, n_cand, n_gtest);
            } else {
                const int n = T - r * kCullSteps;
#pragma unroll
                for (int i = 0; i < kCullSteps; ++i) {
                    if (i < n) {
                        if (c.use_bdry)
                            step(kTrue, i, px[i], py[i]);
                        else
                            step(kFalse, i, px[i], py[i]);
                    } else {
                        px[i] = px[i > 0 ? i - 1 : 0];
                        py[i] = py[i > 0 ? i - 1 : 0];
                    }
                }
                if (n_grp > 0) cnt += obstacle_hits_culled<kCullSteps>(otab, n_grp, first, px, py, n, n_cand, n_gtest);
            }
        }
        if (!own) __syncthreads();  // the next run's controls are in, this run's are read
    }
    if (!rolls) return;
    const RolloutLate e = late();
    float S = __fmaf_rn(e.c->c_obs, (float)cnt, acc);
    if (e.c->use_ctrl) S += ctrl;
    if (e.c->use_term) S += terminal_cost(c, s);
    if (act) agent_store(&e.S[k], S);
}

// The nominal rollouts of a two-launch step's packed workgroups: a wave for
// each 64 samples, every lane drawing its sample's controls as it rolls them
// out (lanes past K as above).  A workgroup takes the LDS that the disturbed
// ones need, so where these fill it a nominal workgroup costs the place of one
// of them, whether four of its waves roll out samples or one does
// (K = 60000, T = 76, M = 3, 65 obstacles: step 115.6 -> 98.9 us); and where
// nominal rollouts are a good part of the work, three waves of four that only
// draw ahead wait (K = 200000, T = 20, M = 1: 82.4 us).  Drawing a run ahead
// through LDS, as nominal_rollouts does, is slower (102.2 us; and K = 200000,
// T = 22, M = 1: 80.6, here 78.3 us).
template <class Late>
__device__ __forceinline__ void nominal_rollouts_packed(const StepConst& c, const float* V,
                                                        float2* __restrict__ u_out, int item, float2* smem,
                                                        const float4* otab, const float4* gbox, int n_grp,
                                                        int& n_cand, int& n_gtest, Late late) {
    const int T = c.T;
    float* vsh = reinterpret_cast<float*>(smem);  // the mean sequence: no step waits for a global load
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) vsh[i] = V[i];
    __syncthreads();  // the mean sequence and the table staged
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int k0 = (item * c.nom_groups + wave) * 64;
    const bool rolls = wave < c.nom_groups && k0 < c.K;
    const int lane = threadIdx.x & 63;
    const int k = k0 + lane;
    const bool act = k < c.K;
    const bool store = act && c.store_u;
    const int kc = act ? k : c.K - 1;
    const float4 first = n_grp > 0 ? (n_grp == 1 ? otab : gbox)[lane] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    State s{0.0f, 0.0f, c.psi0, c.v0};
    float acc = 0.0f, ctrl = 0.0f;
    int cnt = 0;
    const StepConst cn = with_vector_constants(c);
    auto step = [&](auto bdry, int t, float& px, float& py) {
        const float2 u = sample_control(c, vsh, kc, t);
        if (store) u_out[(size_t)t * c.K + k] = u;
        acc = smooth_cost_acc<decltype(bdry)::value>(cn, s, acc);
        px = s.x;
        py = s.y;
        const float term = __fmaf_rn(vsh[2 * t] * c.inv_var0, u.x, vsh[2 * t + 1] * c.inv_var1 * u.y);
        ctrl = __fmaf_rn(c.gamma, term, ctrl);
        bicycle_step(s, c.dt * u.x, tan_steer(u.y) * c.inv_wheelbase, cn.dt);
    };
    for (int t0 = 0; rolls && t0 < T; t0 += kCullSteps) {
        float px[kCullSteps], py[kCullSteps];
        const int n = min(kCullSteps, T - t0);
        if (n == kCullSteps) {  // a whole run of steps with no branch between them
            if (c.use_bdry) {
#pragma unroll
                for (int i = 0; i < kCullSteps; ++i) step(kTrue, t0 + i, px[i], py[i]);
            } else {
#pragma unroll
                for (int i = 0; i < kCullSteps; ++i) step(kFalse, t0 + i, px[i], py[i]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kCullSteps; ++i) {
                if (i < n) {
                    if (c.use_bdry)
                        step(kTrue, t0 + i, px[i], py[i]);
                    else
                        step(kFalse, t0 + i, px[i], py[i]);
                } else {
                    px[i] = px[i > 0 ? i - 1 : 0];
                    py[i] = py[i > 0 ? i - 1 : 0];
                }
            }
        }
        if (n_grp > 0) cnt += obstacle_hits_culled<kCullSteps>(otab, n_grp, first, px, py, n, n_cand, n_gtest);
    }
    if (!rolls) return;
    const RolloutLate e = late();
    float S = __fmaf_rn(e.c->c_obs, (float)cnt, acc);
    if (e.c->use_ctrl) S += ctrl;
    if (e.c->use_term) S += terminal_cost(c, s);
    if (act) agent_store(&e.S[k], S);
}

// Adds a wave's broad-phase work to its slot of the counters (timing mode).
__device__ __forceinline__ void count_work(unsigned long long* work, int item, int n_cand, int n_gtest) {
    if (work && (threadIdx.x & 63) == 0) {
        const int slot = (item * 16 + ((int)threadIdx.x >> 6)) & (kWorkSlots - 1);
        atomicAdd(&work[slot], (unsigned long long)n_cand);
        atomicAdd(&work[kWorkSlots + slot], (unsigned long long)n_gtest);
    }
}

// One workgroup's share of the rollouts of a step: item < n_nom_wg is a
// nominal workgroup (one lane per sample), otherwise a disturbed workgroup
// (spb samples of M lanes).  Ends with every lane past its last LDS access
// (the caller may reuse the LDS after a barrier).
template <int kNoise, int kForm, class Mean, class Late>
__device__ __forceinline__ void rollout_body(const StepConst& c, const float* __restrict__ obs, const Mean& V,
                                             float2* __restrict__ u_out, int item, float2* smem, Late late) {
    float2* ctl = smem;
    const int tid = threadIdx.x;
    const int spb = c.spb, M = c.M, T = c.T;
    const int n_grp = rollout_n_grp(c.n_obs);
    float4* otab = reinterpret_cast<float4*>(reinterpret_cast<float*>(smem) + rollout_otab_offset(spb, T, M, c.nom_groups));
    float4* gbox = otab + 64 * n_grp;
    for (int i = tid; i < n_grp * 64; i += blockDim.x) otab[i] = obstacle_entry(obs, c.n_obs, i, c.fx, c.fy);
    if (n_grp > 1 && tid < 64) group_bounds(obs, c.n_obs, n_grp, c.fx, c.fy, gbox);
    int n_cand = 0;   // exact obstacle tests (state step, obstacle) of this wave (wave-uniform)
    int n_gtest = 0;  // broad-phase group tests of this wave (wave-uniform)

    if (item < c.n_nom_wg) {
        if constexpr (kForm == kNomDirect)
            nominal_rollouts_packed(c, V, u_out, item, smem, otab, gbox, n_grp, n_cand, n_gtest, late);
        else
            nominal_rollouts<kForm == kNomOwn>(c, V, u_out, item, smem, otab, gbox, n_grp, n_cand, n_gtest, late);
        count_work(late().work, item, n_cand, n_gtest);
        return;
    }

    // ---- disturbed rollouts: one lane per (sample, draw) ----
    // Where nominal and disturbed waves share a SIMD, the disturbed ones take
    // the issue slots first: there are M of them per sample against one
    // nominal lane per sample.  On the receding-horizon workload (K = 2048,
    // M = 64) this order gave the shortest one-launch step of the three
    // (equal priorities and nominal first were 2.7 us slower).
    __builtin_amdgcn_s_setprio(2);
    const int wg = item - c.n_nom_wg;
    // The workgroup's samples: spb of them, or with c.flat the (at most spb)
    // samples of its blockDim consecutive (sample, draw) pairs, k_first the
    // first of them.
    // (K M < 2^31 is checked on the host, so the pair indices fit 32 bits)
    const uint32_t KM = (uint32_t)c.K * (uint32_t)M;
    const uint32_t g0 = (uint32_t)wg * blockDim.x;  // flat: the first pair
    const int k_first = c.flat ? (int)(g0 / (uint32_t)M) : wg * spb;
    const int n_smp = c.flat ? (int)((min(g0 + blockDim.x, KM) - 1u) / (uint32_t)M) - k_first + 1 : spb;
    for (int idx = tid; idx < n_smp * T; idx += blockDim.x) {
        const int sl = idx / T;
        const int t = idx - sl * T;
        const int kk = k_first + sl;
        float2 cu = make_float2(0.0f, 0.0f);
        if (kk < c.K) {
            const float2 u = sample_control(c, V, kk, t);
            cu = make_float2(c.dt * u.x, tan_steer(u.y) * c.inv_wheelbase);
        }
        ctl[idx] = cu;
    }
    __syncthreads();

    int sl, m, k;
    if (c.flat) {  // lanes past the last pair repeat it, their results dropped
        const uint32_t g = min(g0 + (uint32_t)tid, KM - 1u);
        k = (int)(g / (uint32_t)M);
        m = (int)(g - (uint32_t)k * (uint32_t)M);
        sl = k - k_first;
    } else {
        sl = tid / M;
        m = tid - sl * M;
        k = wg * spb + sl;
    }
    float L = 0.0f;
    int hits = 0;
    {
        const StepConst cv = with_vector_constants(c);
        const PhiloxVKeys vk = philox_vkeys(c.key0, c.key1);
        const uint32_t exp_word = in_vgpr_u(0x7Fu);
        // every lane runs a rollout (the obstacle test works on whole waves);
        // lanes past the workgroup's last sample repeat its controls, and the
        // results of inactive lanes are dropped
        const float2* ck = ctl + min(sl, n_smp - 1) * T;
        const float4 first = n_grp > 0 ? (n_grp == 1 ? otab : gbox)[tid & 63] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        State s{0.0f, 0.0f, c.psi0, c.v0};
        float acc = 0.0f;
        int cnt = 0;
        // one disturbed state step: running cost at x_t, then (t < T - 1; the
        // last draw cannot reach the risk cost) x_{t+1}
        auto step = [&](auto bdry, int t, bool advance, float& px, float& py) {
            acc = smooth_cost_acc<decltype(bdry)::value>(cv, s, acc);
            px = s.x;
            py = s.y;
            if (advance) {
                const uint4 r = philox4x32_10((uint32_t)t, (uint32_t)m, (uint32_t)k, c.step_idx, c.key0, c.key1, vk);
                const float2 cc = ck[t];
                bicycle_step(s, cc.x, cc.y, cv.dt);
                s = disturbed_successor<kNoise>(cv, r, s, exp_word);
            }
        };
        for (int t0 = 0; t0 < T; t0 += kCullSteps) {  // the obstacle test runs once per kCullSteps points
            float px[kCullSteps], py[kCullSteps];
            if (t0 + kCullSteps < T) {
                // a whole run of steps with no branch between them, so that
                // the noise of later steps can be computed beside the
                // dynamics of earlier ones
                if (c.use_bdry) {
#pragma unroll
                    for (int i = 0; i < kCullSteps; ++i) step(kTrue, t0 + i, true, px[i], py[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < kCullSteps; ++i) step(kFalse, t0 + i, true, px[i], py[i]);
                }
                if (n_grp > 0)
                    cnt += obstacle_hits_culled<kCullSteps>(otab, n_grp, first, px, py, kCullSteps, n_cand, n_gtest);
            } else {
                const int n = T - t0;
#pragma unroll
                for (int i = 0; i < kCullSteps; ++i) {
                    if (i < n) {
                        if (c.use_bdry)
                            step(kTrue, t0 + i, i + 1 < n, px[i], py[i]);
                        else
                            step(kFalse, t0 + i, i + 1 < n, px[i], py[i]);
                    } else {
                        px[i] = px[i > 0 ? i - 1 : 0];
                        py[i] = py[i > 0 ? i - 1 : 0];
                    }
                }
                if (n_grp > 0) cnt += obstacle_hits_culled<kCullSteps>(otab, n_grp, first, px, py, n, n_cand, n_gtest);
            }
        }
        L = acc;
        hits = cnt;
    }
    // From here on the arguments are read again (RolloutLate), and the lane's
    // sample and draw are derived again from a copy of the thread index that
    // the compiler cannot tie to the one above, so that nothing but the cost
    // needs a register through the rollout (the kernel runs at its register
    // limit).
    const RolloutLate e = late();
    const StepConst& ce = *e.c;
    int tid_e = tid;
    asm volatile("" : "+v"(tid_e));
    L = __fmaf_rn(ce.c_obs, (float)hits, L);
    if (ce.flat) {
        // the risk costs go to memory; a separate pass forms each sample's
        // CVaR from them (k_cvar_wave, k_cvar_sorted: the same order)
        const uint32_t g = (uint32_t)wg * blockDim.x + (uint32_t)tid_e;
        if (g < (uint32_t)ce.K * (uint32_t)ce.M) e.L[g] = L;
        count_work(e.work, item, n_cand, n_gtest);
        return;
    }
    const int M_e = ce.M, spb_e = ce.spb;
    const int sl_e = tid_e / M_e;
    const int m_e = tid_e - sl_e * M_e;
    const int k_e = wg * spb_e + sl_e;
    const bool active_e = (sl_e < spb_e) && (k_e < ce.K);
    if (active_e && ce.debug) e.L[(size_t)k_e * M_e + m_e] = L;
    float* vals = reinterpret_cast<float*>(smem + (size_t)spb_e * ce.T);
    float* tail = vals + spb_e * M_e;
    float* means = tail + spb_e * M_e;
    if (!ce.grad && ce.wave_tails) {
        if (sl_e < spb_e) vals[tid_e] = active_e ? L : 0.0f;
        cvar_waves(vals, spb_e, M_e, ce.n_tail, ce.scale_risk, ce.B, tid_e, [&](int q, float cv) {
            const int ks = wg * spb_e + q;
            if (ks < ce.K) agent_store(&e.cvar[ks], cv);
        });
    } else {
        if (sl_e < spb_e) {
            vals[tid_e] = active_e ? L : 0.0f;
            tail[tid_e] = __builtin_nanf("");
        }
        int pos = M_e, id = m_e;
        const float cv =
            cvar_epilogue(vals, tail, means, spb_e, M_e, ce.n_tail, ce.scale_risk, ce.B, &pos, &id, tid_e);
        if (active_e && m_e == 0) agent_store(&e.cvar[k_e], cv);
        if (ce.grad && active_e) {  // tail membership for the gradient
            e.ranks[(size_t)k_e * M_e + id] = pos;
            if (pos < ce.n_tail) e.tail_idx[(size_t)k_e * ce.n_tail + pos] = id;
        }
    }
    count_work(e.work, item, n_cand, n_gtest);
}

// Sum and minimum of 256 values held in LDS (v[0..255]) in a fixed order that
// does not depend on the workgroup size: wave-sized segments of 64 values are
// reduced by the butterflies of wave_sum / wave_min, the four segment results
// combined as (s0 + s1) + (s2 + s3).  Every thread of the workgroup (a
// multiple of 64 threads) must call them; the result is returned to all.
// red holds at least 16 floats of LDS.
__device__ __forceinline__ float seg_sum_256(const float* v, float* red) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();  // v written
    for (int sg = wv; sg < 4; sg += nw) {
        const float x = wave_sum(v[64 * sg + lane]);
        if (lane == 0) red[sg] = x;
    }
    __syncthreads();
    const float r = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();  // red and v free again
    return r;
}

__device__ __forceinline__ float seg_min_256(const float* v, float* red) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    for (int sg = wv; sg < 4; sg += nw) {
        const float x = wave_min(v[64 * sg + lane]);
        if (lane == 0) red[sg] = x;
    }
    __syncthreads();
    const float r = fminf(fminf(red[0], red[1]), fminf(red[2], red[3]));
    __syncthreads();
    return r;
}

// Weights and update (Eq. 14-17 and Eq. 4), in chunks of 256 samples; any
// workgroup size that is a multiple of 64 gives the same bits.
//  1. (update_chunk) S~ = S + J_C per sample of chunk b; the chunk's minimum
//     beta_b, its weights exp(-(S~ - beta_b)/lambda) and their sum Z_b;
//  2. (update_chunk) the chunk's weighted control sums N_b[t] = sum_k w_k
//     u_{k,t}, item (t, part) summing a contiguous slice of the chunk, the
//     slices then added in order; (beta_b, Z_b, N_b) go to part[b], or, when
//     the chunk is the only one (`single`), to red[0], red[1] and the LDS
//     array that the call returns;
//  3. (update_merge, run by whoever finishes the last chunk) beta = min
//     beta_b, scale_b = exp(-(beta_b - beta)/lambda), V+ = sum_b scale_b N_b /
//     sum_b scale_b Z_b; then V (shifted when asked), the first command and,
//     in debug mode, w_hat; in gradient mode J, every w_hat and the list of
//     samples of non-zero weight instead, V unchanged.
// LDS (dynamic, ush): w[256] | slice sums [parts][2T] | nzpos[257] |
// nzlist[256] | mean sequence [2T], then for the merge v[256] | scale[G] |
// zb[G] | vp[2T] (update_lds_bytes).
//
// With kRegen the chunk draws the controls of its samples of non-zero
// weight again from the same Philox counters and the same V (which the merge
// rewrites only after every chunk is in) instead of reading stored ones:
// sample_control is the function that drew them, so the values are the same
// bits.  Stored controls would have been written by workgroups on other
// XCDs, and each round of loads waits about 1.4 us for memory, while a
// redrawn control costs a few tens of instructions; so a step stores no
// controls unless the debug view or the gradient asks for them, and even a
// chunk whose every weight is non-zero is summed sooner than by loading.
// Where the controls are stored, the two-launch update reads them (the
// one-launch update still draws them), so the bit-exact comparison of the
// two forms in debug mode also checks that the drawn controls are the stored
// ones.
template <int kB, bool kRegen = false, bool kServe = false>
__device__ __forceinline__ float* update_chunk(const StepConst& c, int b, int parts, const float* S,
                                               const float* cvar, const float2* __restrict__ u, float* S_tilde,
                                               float* part, float* ush, float* red, bool single,
                                               const float* __restrict__ V = nullptr) {
    const int T = c.T, K = c.K;
    const int tid = threadIdx.x, nt = blockDim.x;
    float* wsh = ush;
    float* psh = wsh + 256;
    int* nzpos = reinterpret_cast<int*>(psh + (size_t)parts * 2 * T);  // 257
    int* nzlist = nzpos + 257;                                          // 256
    float* vsh = reinterpret_cast<float*>(nzlist + 256);                // 2T
    const int k0 = b * 256;
    const int n = min(256, K - k0);
    const int stride = 2 + 2 * T;
    const int slice = (n + parts - 1) / parts;
    // V (for the redrawn controls) is staged into LDS after the first step
    // below, but the thread's first value is loaded now, so that its load and
    // the first wave's loads of S and CVaR wait on memory together
    const bool has_v = kRegen && tid < 2 * T;
    const float v_first = has_v ? mean_load<kServe>(&V[tid]) : 0.0f;

    // 1. modified costs, the chunk's minimum beta_b, its weights and their
    // sum Z_b, and the samples of non-zero weight, all by the first wave:
    // lane l holds samples l, l + 64, l + 128 and l + 192 (the four 64-value
    // segments of seg_min_256 / seg_sum_256, reduced by the same butterflies
    // and combined in the same order, so the bits are theirs), and no
    // barrier separates the steps.  The samples of non-zero weight go to
    // nzlist in index order (exp underflows to an exact zero once a cost
    // exceeds the chunk's minimum by about 104 lambda), nzpos[k] counting
    // how many come before sample k.  A zero weight adds 0 * u, which leaves
    // a sum exactly as it is, so the sums below skip those samples and still
    // give the bits of the full sums.
    float beta_b = 0.0f, Z_b = 0.0f;
    if (tid < 64) {
        // the eight loads first (a lane past the chunk's end reads its last
        // sample and drops it), so that they wait on memory once, not once
        // per segment
        float cvl[4], sl[4];
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
            const int i = min(64 * sg + tid, n - 1);
            cvl[sg] = agent_load(&cvar[k0 + i]);
            sl[sg] = agent_load(&S[k0 + i]);
        }
        float w[4];
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
            const int i = 64 * sg + tid;
            float st = __builtin_inff();
            if (i < n) {
                const float cv = cvl[sg];
                const float jc = (cv > c.C_u) ? c.A * cv : 0.0f;  // Eq. 14-15
                st = sl[sg] + jc;                                  // Eq. 16
                agent_store(&S_tilde[k0 + i], st);
            }
            w[sg] = st;
        }
        beta_b = wave_min(fminf(fminf(w[0], w[1]), fminf(w[2], w[3])));  // a minimum: exact in any order
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) w[sg] = (64 * sg + tid < n) ? expf(-(w[sg] - beta_b) / c.lambda) : 0.0f;
        Z_b = (wave_sum(w[0]) + wave_sum(w[1])) + (wave_sum(w[2]) + wave_sum(w[3]));
        int off = 0;
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
            const int k = 64 * sg + tid;
            const uint64_t bal = __builtin_amdgcn_ballot_w64(w[sg] != 0.0f);
            const int q = off + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            nzpos[k] = q;
            if (w[sg] != 0.0f) nzlist[q] = k;
            wsh[k] = w[sg];
            off += __builtin_popcountll(bal);
        }
        if (tid == 0) nzpos[256] = off;
    }
    if (kRegen) {
        if (has_v) vsh[tid] = v_first;
        for (int i = tid + nt; i < 2 * T; i += nt) vsh[i] = mean_load<kServe>(&V[i]);
    }
    __syncthreads();  // wsh, nzpos, nzlist and V published

    // 2. weighted control sums over slices of the chunk, in index order
    for (int idx = tid; idx < T * parts; idx += nt) {
        const int t = idx / parts;  // neighbouring lanes read the slices of one row
        const int pr = idx % parts;
        const int ka = pr * slice, kb = min(n, ka + slice);
        float ax = 0.0f, ay = 0.0f;
        int q = ka < kb ? nzpos[ka] : 0;
        const int qb = ka < kb ? nzpos[kb] : 0;
        if constexpr (kRegen) {
            for (; q < qb; ++q) {
                const int k = nzlist[q];
                const float ww = wsh[k];
                const float2 uu = sample_control(c, vsh, k0 + k, t);
                ax = __fmaf_rn(ww, uu.x, ax);
                ay = __fmaf_rn(ww, uu.y, ay);
            }
        } else {
            const float2* ut = u + (size_t)t * K + k0;
            for (; q + kB <= qb; q += kB) {  // kB loads in flight, then the sums in order
                float2 uu[kB];
                float ww[kB];
#pragma unroll
                for (int i = 0; i < kB; ++i) {
                    const int k = nzlist[q + i];
                    ww[i] = wsh[k];
                    uu[i] = ut[k];
                }
#pragma unroll
                for (int i = 0; i < kB; ++i) {
                    ax = __fmaf_rn(ww[i], uu[i].x, ax);
                    ay = __fmaf_rn(ww[i], uu[i].y, ay);
                }
            }
            if (q < qb) {  // the rest in one more round
                float2 uu[kB];
                float ww[kB];
#pragma unroll
                for (int i = 0; i < kB; ++i) {
                    const bool in = q + i < qb;
                    const int k = in ? nzlist[q + i] : 0;
                    ww[i] = in ? wsh[k] : 0.0f;
                    uu[i] = in ? ut[k] : make_float2(0.0f, 0.0f);
                }
#pragma unroll
                for (int i = 0; i < kB; ++i) {
                    if (q + i < qb) {
                        ax = __fmaf_rn(ww[i], uu[i].x, ax);
                        ay = __fmaf_rn(ww[i], uu[i].y, ay);
                    }
                }
            }
        }
        psh[(size_t)pr * 2 * T + 2 * t] = ax;
        psh[(size_t)pr * 2 * T + 2 * t + 1] = ay;
    }
    __syncthreads();
    if (single) {  // the only chunk: its sums stay in LDS (in vsh, read for the last time above) for the merge
        for (int j = tid; j < 2 * T; j += nt) {
            float acc = 0.0f;
            for (int pr = 0; pr < parts; ++pr) acc += psh[(size_t)pr * 2 * T + j];
            vsh[j] = acc;
        }
        if (tid == 0) {
            red[0] = beta_b;
            red[1] = Z_b;
        }
        __syncthreads();
        return vsh;
    }
    float* pb = part + (size_t)b * stride;
    for (int j = tid; j < 2 * T; j += nt) {
        float acc = 0.0f;
        for (int pr = 0; pr < parts; ++pr) acc += psh[(size_t)pr * 2 * T + j];
        agent_store(&pb[2 + j], acc);
    }
    if (tid == 0) {
        agent_store(&pb[0], beta_b);
        agent_store(&pb[1], Z_b);
    }
    return nullptr;
}

// The merge's last part, once vp (2T) holds V+ in LDS and beta, Z (and
// invZ = 1 / Z) are known: V (shifted when asked), the first command and the
// completion word, w_hat in debug mode; in gradient mode J, every w_hat and
// the samples of non-zero weight instead, V unchanged.
__device__ __forceinline__ void merge_finish(const StepConst& c, float beta, float Z, float invZ, const float* vp,
                                             const float* S_tilde, float* __restrict__ V, float* __restrict__ u0,
                                             float* __restrict__ u0_host, float* __restrict__ w_hat,
                                             float* ush, const float* w_only, const GradOut* go) {
    const int T = c.T, K = c.K;
    const int tid = threadIdx.x, nt = blockDim.x;
    __syncthreads();
    if (go) {
        // gradient mode: V stays as it is; write J = beta - lambda log(Z/K),
        // every w_hat, and the samples of non-zero weight in increasing order
        if (tid == 0) *go->J = beta - c.lambda * logf(Z / (float)K);
        // (gradient mode runs in workgroups of 256 threads).  Tiles of 16 x
        // 256 samples, sample k of a tile in thread k mod 256, so that the
        // loads and stores are whole lines with 16 in flight; a wave counts
        // its non-zero weights of each 64 by ballot, one wave adds the counts
        // up in sample order, and every non-zero sample goes to its place.
        // (A contiguous run of samples per thread waits on memory for each
        // of them, twice: K = 4096, the whole update 15.2 us, now 11.0.)
        // The only chunk's weights are still in LDS (w_only): they are those
        // of the merge, its minimum being beta.
        constexpr int kTile = 16;
        int* cnt_sh = reinterpret_cast<int*>(ush + 256);  // 4 kTile counts, then their exclusive sums
        const int lane = tid & 63, wv = tid >> 6;
        int total = 0;
        for (int base = 0; base < K; base += 256 * kTile) {
            const int nj = min(kTile, (K - base + 255) >> 8);  // rows of the tile that hold samples
            float st[kTile];
            if (!w_only) {
#pragma unroll
                for (int j = 0; j < kTile; ++j) {
                    const int k = base + 256 * j + tid;
                    st[j] = k < K ? agent_load(&S_tilde[k]) : __builtin_inff();  // no weight past the end
                }
            }
            uint32_t nz = 0;
            int before[kTile];
#pragma unroll
            for (int j = 0; j < kTile; ++j) {
                if (j >= nj) break;  // uniform
                const int k = base + 256 * j + tid;
                const float wk = (w_only ? w_only[tid] : expf(-(st[j] - beta) / c.lambda)) * invZ;
                const bool on = k < K && wk > 0.0f;
                if (k < K) w_hat[k] = wk;
                const uint64_t bal = __builtin_amdgcn_ballot_w64(on);
                nz |= on ? 1u << j : 0u;
                before[j] = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                if (lane == 0) cnt_sh[4 * j + wv] = __builtin_popcountll(bal);
            }
            __syncthreads();
            if (tid < 64) {  // up to 4 kTile = 64 counts in sample order
                const int own = lane < 4 * nj ? cnt_sh[lane] : 0;
                int incl = own;
                for (int d = 1; d < 64; d <<= 1) {
                    const int o = __shfl_up(incl, d);
                    if (lane >= d) incl += o;
                }
                cnt_sh[lane] = incl - own;
                if (lane == 63) cnt_sh[64] = incl;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kTile; ++j) {
                if (j >= nj) break;
                if (nz & (1u << j)) go->act_list[total + cnt_sh[4 * j + wv] + before[j]] = base + 256 * j + tid;
            }
            total += cnt_sh[64];
            __syncthreads();  // cnt_sh is refilled
        }
        if (tid == 0) *go->n_act = total;
        return;
    }
    const int shift = (c.flags & 2u) != 0;
    for (int j = tid; j < 2 * T; j += nt) {
        int src = j;
        if (shift) src = min(j + 2, 2 * T - 2 + (j & 1));
        agent_store(&V[j], vp[src]);
    }
    // The workgroup that merges differs from step to step, and where one launch
    // serves many, an XCD's L2 could still hold an earlier step's command or
    // weights and write them back over later ones: both are written through.
    if (tid < 2) agent_store(&u0[tid], vp[tid]);
    if (c.debug) {
        // (before the completion word, after which the next served step may
        // rewrite S~)
        for (int k = tid; k < K; k += nt)
            agent_store(&w_hat[k], expf(-(agent_load(&S_tilde[k]) - beta) / c.lambda) * invZ);
    }
    if (u0_host) {
        // mapped pinned host memory: the command first, then the completion
        // word, each at system scope.  The word may release the next served
        // step, whose workgroups read V: every wave waits for its stores of V
        // (written through to the memory that the XCDs share, from which the
        // next step's readers load: mean_load), and the workgroup meets at a
        // barrier before the word is stored.
        if (tid < 2) __hip_atomic_store(&u0_host[tid], vp[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        stores_done();
        __syncthreads();
        if (tid == 0 && c.u0_seq)
            __hip_atomic_store(reinterpret_cast<unsigned*>(u0_host + 2), c.u0_seq, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <int kB>
__device__ __forceinline__ void update_merge(const StepConst& c, int G, const float* part, const float* S_tilde,
                                             float* __restrict__ V,
                                             float* __restrict__ u0, float* __restrict__ u0_host,
                                             float* __restrict__ w_hat, float* ush, float* red,
                                             const GradOut* go = nullptr) {
    const int T = c.T;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int stride = 2 + 2 * T;
    float* vsh = ush;  // 256 per-virtual-thread values
    float* scale = vsh + 256;
    float* zb = scale + G;
    float* vp = zb + G;
    // rows of the weighted sums loaded before beta and Z are known
    constexpr int kP = kB > 8 ? kB : 8;

    // The first kP rows of the weighted sums (thread j < 2T) do not depend
    // on beta or Z: their loads are issued first.
    float pre[kP];
    const int n_pre = G < kP ? G : kP;
    const bool has_pre = tid < 2 * T;
    if (has_pre) {
#pragma unroll
        for (int i = 0; i < kP; ++i) pre[i] = i < n_pre ? agent_load(&part[(size_t)i * stride + 2 + tid]) : 0.0f;
    }
    float beta, Z;
    if (G <= 64) {
        // one wave, chunk b in lane b: the minimum (exact in any order), the
        // scales, and Z by the butterfly of seg_sum_256's first segment (its
        // other three segments hold zeros, whose sums add nothing to a
        // positive Z, so the bits are the same); one barrier publishes them
        if (tid < 64) {
            const bool in = tid < G;
            const float be = in ? agent_load(&part[(size_t)tid * stride]) : __builtin_inff();
            const float z0 = in ? agent_load(&part[(size_t)tid * stride + 1]) : 0.0f;
            const float bmin = wave_min(be);
            const float sc = in ? expf(-(be - bmin) / c.lambda) : 0.0f;
            const float zs = wave_sum(__fmaf_rn(z0, sc, 0.0f));
            if (in) scale[tid] = sc;
            if (tid == 0) {
                red[0] = bmin;
                red[1] = zs;
            }
        }
        __syncthreads();
        beta = red[0];
        Z = red[1];
    } else {
        // virtual thread i (of 256) takes chunks i, i + 256, ...; beta_b and
        // Z_b are read once and kept in LDS
        for (int i = tid; i < 256; i += nt) {
            float m = __builtin_inff();
            for (int bb = i; bb < G; bb += 256) {
                const float be = agent_load(&part[(size_t)bb * stride]);
                scale[bb] = be;
                zb[bb] = agent_load(&part[(size_t)bb * stride + 1]);
                m = fminf(m, be);
            }
            vsh[i] = m;
        }
        beta = seg_min_256(vsh, red);  // also publishes scale (beta_b) and zb
        for (int i = tid; i < 256; i += nt) {
            float z = 0.0f;
            for (int bb = i; bb < G; bb += 256) {
                const float sc = expf(-(scale[bb] - beta) / c.lambda);
                scale[bb] = sc;
                z = __fmaf_rn(zb[bb], sc, z);
            }
            vsh[i] = z;
        }
        Z = seg_sum_256(vsh, red);  // also publishes scale
    }
    const float invZ = 1.0f / Z;
    for (int j = tid; j < 2 * T; j += nt) {
        float acc = 0.0f;
        int bb = 0;
        if (j == tid && has_pre) {  // the prefetched rows, summed in the same order
#pragma unroll
            for (int i = 0; i < kP; ++i)
                if (i < n_pre) acc = __fmaf_rn(pre[i], scale[i], acc);
            bb = n_pre;
        }
        for (; bb + kB <= G; bb += kB) {  // kB loads in flight, then the sums in order
            float pv[kB];
#pragma unroll
            for (int i = 0; i < kB; ++i) pv[i] = agent_load(&part[(size_t)(bb + i) * stride + 2 + j]);
#pragma unroll
            for (int i = 0; i < kB; ++i) acc = __fmaf_rn(pv[i], scale[bb + i], acc);
        }
        if (bb < G) {  // the rest in one more round (padding terms 0 * 0)
            float pv[kB], sv[kB];
#pragma unroll
            for (int i = 0; i < kB; ++i) {
                const bool in = bb + i < G;
                pv[i] = in ? agent_load(&part[(size_t)(bb + i) * stride + 2 + j]) : 0.0f;
                sv[i] = in ? scale[bb + i] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < kB; ++i) acc = __fmaf_rn(pv[i], sv[i], acc);
        }
        vp[j] = acc * invZ;
    }
    merge_finish(c, beta, Z, invZ, vp, S_tilde, V, u0, u0_host, w_hat, ush, nullptr, go);
}

// The merge when there is one chunk (K <= 256), run by the workgroup that
// has just formed it (nb: its sums, in LDS; beta and Z in red): beta =
// beta_0, every scale is exp(0) = 1 and Z = Z_0, so V+ = N_0 / Z_0 -- the
// bits of update_merge with G = 1, without the counter, the reductions or a
// trip through memory.
__device__ __forceinline__ void update_merge_single(const StepConst& c, float* nb, const float* S_tilde,
                                                    float* __restrict__ V, float* __restrict__ u0,
                                                    float* __restrict__ u0_host, float* __restrict__ w_hat,
                                                    float* ush, float* red, const GradOut* go = nullptr) {
    const float beta = red[0];
    const float Z = red[1];
    const float invZ = 1.0f / Z;
    for (int j = threadIdx.x; j < 2 * c.T; j += blockDim.x) nb[j] *= invZ;
    if (c.debug) stores_done();  // S~, read back below by other waves of this workgroup
    merge_finish(c, beta, Z, invZ, nb, S_tilde, V, u0, u0_host, w_hat, ush, ush, go);
}

// Counts the workgroup in at a device-scope counter, after every wave's
// stores (see agent_store); returns to every thread whether this made it
// reach `target`, in which case the counter is reset to zero and whatever the
// other workgroups stored before counting in may be loaded by agent_load.
__device__ __forceinline__ bool arrive_last(unsigned* counter, unsigned target, int* flag_sh) {
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned done = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag_sh = (done == target - 1u);
        if (*flag_sh) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return *flag_sh != 0;
}

// Loads in flight per thread in the update run inside the rollout launch,
// whose register budget is the rollout's (the separate update launch uses 16).
constexpr int kFuseBatch = 4;

// Buffers of the update run inside the rollout launch (one step in one
// kernel), held in device memory so that they occupy no registers during the
// rollouts.
struct FuseArgs {
    unsigned* chunk_ctr;  // G counters of finished contributors (zero between launches)
    unsigned* counter;    // chunks finished (zero between launches)
    float* S_tilde;
    float* part;
    float* u0;
    float* u0_host;       // mapped host buffer, written when the step asks for the first command
    float* w_hat;
    int G, parts;
};

// FuseArgs as read from device memory, its pointers in the global address
// space (as_global).
__device__ __forceinline__ FuseArgs global_view(const FuseArgs& f) {
    FuseArgs g = f;
    g.chunk_ctr = as_global(f.chunk_ctr);
    g.counter = as_global(f.counter);
    g.S_tilde = as_global(f.S_tilde);
    g.part = as_global(f.part);
    g.u0 = as_global(f.u0);
    g.u0_host = as_global(f.u0_host);
    g.w_hat = as_global(f.w_hat);
    return g;
}

// ---- persistent serving: one resident launch runs step after step ----

// One served step's request: the per-step constants the host derives from
// the measured state (the same arithmetic as for a launched step), each in
// the upper half of an eight-byte word whose lower half is the request's
// number (1, 2, ... within a session), in one line of mapped host memory and
// again of device memory.  A word is stored and loaded whole, so whoever sees
// the number in all eight has the request, whatever order they came in.
enum ServeField {
    kServeIdx, kServeFx, kServeFy, kServeTox, kServeToy, kServeTheta, kServePsi, kServeV,
    kServeFields
};
struct ServeReq {
    uint64_t w[kServeFields];
};

__host__ __device__ __forceinline__ uint64_t serve_word(uint32_t seq, uint32_t value) {
    return (uint64_t)value << 32 | seq;
}

struct ServeArgs {
    const ServeReq* req_host;  // mapped host memory (device address)
    ServeReq* req_dev;         // device copy read by the other workgroups
    uint32_t naps;             // sleeps of 640 clocks added between two reads of either
    uint64_t idle_ticks;       // longest wait for a request (s_memrealtime ticks, 100 MHz)
};

__device__ __forceinline__ ServeArgs global_view(const ServeArgs& a) {
    ServeArgs g = a;
    g.req_host = as_global(a.req_host);
    g.req_dev = as_global(a.req_dev);
    return g;
}

constexpr unsigned kServeExit = 0xFFFFFFFFu;  // a request number: leave

// The first wave of a workgroup: waits for request seq and leaves its values
// in words (LDS, published by the caller's barrier).  Workgroup 0 waits on
// host memory and copies the request to device memory, on which the others
// wait.  Returns whether to leave: when kServeExit comes, or without a
// request within idle_ticks (workgroup 0, which then passes kServeExit on) or
// twice that.  Lane l takes word l mod 8, so a request is there as soon as
// it is seen, one trip across PCIe and one through device memory after the
// host has posted it.  No cache is written back or invalidated: what changes
// between requests (the request, V, the values of agent_store) is stored and
// loaded at device scope, and the rest stays in the caches.  (32 served steps
// of K = 2048, T = 50, M = 64: 1376 us when every workgroup invalidated its
// XCD's L2 as it started, 1308 without, 1197 with the numbers in the words
// instead of in words of their own, stored after the others.)
__device__ __forceinline__ bool serve_wait(const ServeArgs& sa, unsigned seq, bool leader, uint32_t* words) {
    const int i = threadIdx.x & (kServeFields - 1);
    const uint64_t limit = leader ? sa.idle_ticks : 2 * sa.idle_ticks;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    uint64_t w;
    bool leave = false;
    for (;;) {
        w = leader ? __hip_atomic_load(&sa.req_host->w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)
                   : __hip_atomic_load(&sa.req_dev->w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        leave = __builtin_amdgcn_ballot_w64((uint32_t)w == kServeExit) != 0;
        if (leave || __builtin_amdgcn_ballot_w64((uint32_t)w != seq) == 0) break;
        leave = __builtin_amdgcn_s_memrealtime() - t0 > limit;
        if (leave) break;
        __builtin_amdgcn_s_sleep(1);
        for (uint32_t n = sa.naps; n > 0u; --n) __builtin_amdgcn_s_sleep(10);
    }
    if (threadIdx.x < kServeFields) {
        if (leader)
            __hip_atomic_store(&sa.req_dev->w[i], leave ? serve_word(kServeExit, 0u) : w, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        words[i] = (uint32_t)(w >> 32);
    }
    return leave;
}

// A value of the request being served, after that barrier (the same in every lane).
__device__ __forceinline__ uint32_t serve_value(const uint32_t* words, ServeField f) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)words[f]);
}

// Workgroups of a rollout launch whose samples fall in chunk b: the nominal
// workgroups (64 nom_groups samples each) and the disturbed ones (spb each).
__device__ __forceinline__ unsigned chunk_contributors(const StepConst& c, int b) {
    const int klo = 256 * b, khi = min(c.K, klo + 256) - 1;
    const int nom = 64 * c.nom_groups;
    return (unsigned)((khi / nom - klo / nom + 1) + (khi / c.spb - klo / c.spb + 1));
}

// After a rollout workgroup has stored its results: it counts itself in the
// chunks its samples fall in, and for every chunk it completes runs that
// chunk's update (its inputs S, CVaR and u are then all stored, written
// through by agent_store); the workgroup that completes the last chunk merges
// them.  No workgroup waits for another.
template <bool kServe = false>
__device__ __forceinline__ void fused_update(const StepConst& c, const FuseArgs& f, int item, const float* S,
                                             const float* cvar, const float2* u, float* V, float* ush, float* red,
                                             int* flag_sh, int* fin_sh) {
    int lo, hi;
    if (item < c.n_nom_wg) {
        lo = item * 64 * c.nom_groups;
        hi = min(c.K, lo + 64 * c.nom_groups);
    } else {
        lo = (item - c.n_nom_wg) * c.spb;
        hi = min(c.K, lo + c.spb);
    }
    stores_done();
    __syncthreads();  // every wave's stores of S and CVaR are done; LDS free
    if (threadIdx.x == 0) {
        int nf = 0;
        for (int b = lo >> 8; b <= (hi - 1) >> 8; ++b) {
            const unsigned target = chunk_contributors(c, b);
            const unsigned done =
                __hip_atomic_fetch_add(&f.chunk_ctr[b], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (done == target - 1u) {
                __hip_atomic_store(&f.chunk_ctr[b], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                fin_sh[nf++] = b;
            }
        }
        fin_sh[7] = nf;
    }
    __syncthreads();
    const int nf = fin_sh[7];
    if (nf == 0) return;
    for (int i = 0; i < nf; ++i) {
        float* nb = update_chunk<kFuseBatch, true, kServe>(c, fin_sh[i], f.parts, S, cvar, u, f.S_tilde, f.part, ush, red,
                                                   f.G == 1, V);
        if (f.G == 1)
            update_merge_single(c, nb, f.S_tilde, V, f.u0, c.u0_seq ? f.u0_host : nullptr, f.w_hat, ush, red);
        else if (arrive_last(f.counter, (unsigned)f.G, flag_sh))
            update_merge<kFuseBatch>(c, f.G, f.part, f.S_tilde, V, f.u0, c.u0_seq ? f.u0_host : nullptr, f.w_hat,
                                     ush, red);
    }
}

// One chunk of the update, and the merge when it is the last chunk to finish
// (a separate launch of G workgroups, one chunk each).  No workgroup waits
// for another, and every sum runs in a fixed order.
__device__ __forceinline__ void update_body(const StepConst& c, int b, int G, int parts, const float* S,
                                            const float* cvar, const float2* __restrict__ u, float* S_tilde,
                                            float* part, unsigned* counter,
                                            float* __restrict__ V, float* __restrict__ u0,
                                            float* __restrict__ u0_host, float* __restrict__ w_hat, float* ush,
                                            float* red, int* flag_sh, const GradOut* go = nullptr) {
    // the stored controls when the rollouts stored them (debug and
    // gradient modes), else the same controls drawn again
    float* nb = c.store_u ? update_chunk<16>(c, b, parts, S, cvar, u, S_tilde, part, ush, red, G == 1)
                          : update_chunk<16, true>(c, b, parts, S, cvar, u, S_tilde, part, ush, red, G == 1, V);
    if (G == 1) {
        update_merge_single(c, nb, S_tilde, V, u0, u0_host, w_hat, ush, red, go);
        return;
    }
    if (!arrive_last(counter, (unsigned)G, flag_sh)) return;
    update_merge<16>(c, G, part, S_tilde, V, u0, u0_host, w_hat, ush, red, go);
}

}  // namespace ramppi
