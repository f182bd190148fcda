// Batched serving: one step of many independent controllers (uneven K, T, M
// and obstacle counts) in three or four launches that a HIP graph can hold:
//   k_batch_prep     one thread per controller: reads the controller's
//                    measured state and call index from mapped host memory
//                    and completes its per-step constants;
//   k_batch_rollout  one workgroup per (controller, workgroup) item of a list
//                    that the host orders (by default longest first; the
//                    hardware starts workgroups in list order), running the
//                    same rollout body as the single-controller kernel;
//   k_batch_cvar     where the batch has controllers in the flattened layout:
//                    the CVaR of their samples from the stored risk costs;
//   k_batch_update   one workgroup per (controller, chunk) item, the same
//                    update body as the single-controller kernel, merged per
//                    controller by its last chunk.
// Nothing waits for another workgroup, so every wave reaches its exit.
#include <algorithm>

#include "launch.h"
#include "step_device.h"

namespace ramppi {

// Per-step constants that depend on the measured state (the same arithmetic
// as the host-side fill for a single controller).
__device__ __forceinline__ void set_dynamic(StepConst& c, const BatchCtl& b, const BatchInput& in) {
    c.fx = in.x0[0];
    c.fy = in.x0[1];
    c.tox = in.x0[0] - b.track[0];
    c.toy = in.x0[1] - b.track[1];
    c.theta0 = (float)atan2(((double)in.x0[1] - (double)b.track[1]) / (double)b.track[3],
                            ((double)in.x0[0] - (double)b.track[0]) / (double)b.track[2]);
    c.psi0 = start_heading(in.x0[2]);
    c.v0 = in.x0[3];
    c.step_idx = in.step_idx;
}

__global__ void __launch_bounds__(64) k_batch_prep(BatchCtl* __restrict__ ctls, const BatchInput* __restrict__ inputs,
                                                   int n_ctl) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i < n_ctl) set_dynamic(ctls[i].c, ctls[i], inputs[i]);
}

// One item of the batch's rollouts: kNoise >= 0 is the one disturbance form
// of every controller of the batch; -1 picks it per item.  A workgroup runs
// one item and leaves: a persistent grid that takes items from a queue paid
// two device atomics per item and kept what it derives from the thread index
// in registers across items (18 VGPRs spilled), and the hardware's own
// dispatch of waiting workgroups balances the list as well (8 controllers of
// K <= 1024, T <= 40: step 91 -> 66 us; 48 of K <= 8192, T <= 100: 2.62 ->
// 2.57 ms).
template <int kNoise>
__device__ __forceinline__ void batch_rollout_item(const BatchCtl* __restrict__ ctls, const int2* __restrict__ items,
                                                   unsigned long long* __restrict__ work) {
    extern __shared__ float2 bsmem[];
    const int2 cw = items[blockIdx.x];
    const BatchCtl& b = ctls[__builtin_amdgcn_readfirstlane(cw.x)];
    const int w = __builtin_amdgcn_readfirstlane(cw.y);
    const StepConst c = b.c;
    // the controller's buffers, read from device memory: in the global
    // address space (as_global)
    const float* obs = as_global(b.obs);
    const float* V = as_global(b.V);
    float2* u = as_global(b.u);
    const auto late = [&] {
        const BatchCtl* e = late_ptr<BatchCtl>(&b);
        return RolloutLate{&e->c, as_global(e->S), as_global(e->cvar), as_global(e->L), nullptr, nullptr, work};
    };
    if constexpr (kNoise >= 0) {
        rollout_body<kNoise, false>(c, obs, V, u, w, bsmem, late);
    } else {
        if (c.noise_kind == 1)
            rollout_body<1, false>(c, obs, V, u, w, bsmem, late);
        else if (c.noise_kind == 2)
            rollout_body<2, false>(c, obs, V, u, w, bsmem, late);
        else
            rollout_body<0, false>(c, obs, V, u, w, bsmem, late);
    }
}

// Controllers of several disturbance forms.  Like the two-launch rollout kernel
// compiled for five waves per SIMD.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
    k_batch_rollout(const BatchCtl* __restrict__ ctls, const int2* __restrict__ items,
                    unsigned long long* __restrict__ work) {
    batch_rollout_item<-1>(ctls, items, work);
}

// One disturbance form for the whole batch: a third of the code.
template <int kNoise>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
    k_batch_rollout_one(const BatchCtl* __restrict__ ctls, const int2* __restrict__ items,
                        unsigned long long* __restrict__ work) {
    batch_rollout_item<kNoise>(ctls, items, work);
}

// The CVaR pass of the controllers in the flattened layout: one workgroup per
// (controller, workgroup) item.
__global__ void __launch_bounds__(256) k_batch_cvar(const BatchCtl* __restrict__ ctls,
                                                    const int2* __restrict__ citems) {
    extern __shared__ float bush[];
    const int2 cw = citems[blockIdx.x];
    const BatchCtl& b = ctls[__builtin_amdgcn_readfirstlane(cw.x)];
    const StepConst& c = b.c;
    cvar_pass(as_global(b.L), c.K, c.M, tail_lanes(c.M), c.n_tail, c.scale_risk, c.B, as_global(b.cvar),
              __builtin_amdgcn_readfirstlane(cw.y), bush);
}

__global__ void __launch_bounds__(256) k_batch_update(const BatchCtl* __restrict__ ctls,
                                                      const int2* __restrict__ uitems) {
    extern __shared__ float bush[];
    __shared__ float red[16];
    __shared__ int is_last;
    const int2 cb = uitems[blockIdx.x];
    const BatchCtl& b = ctls[cb.x];
    const StepConst c = b.c;
    update_body(c, cb.y, b.G, b.parts, as_global(b.S), as_global(b.cvar), as_global(b.u), as_global(b.S_tilde),
                as_global(b.part), as_global(b.counter), as_global(b.V), as_global(b.u0), as_global(b.u0_host),
                as_global(b.w_hat), bush, red, &is_last);
}

// Items of one rollout launch: a grid holds fewer than 2^32 threads.
constexpr int kMaxItemsPerLaunch = 1 << 23;

// (As in a single step, no launch follows one that failed.)
hipError_t launch_batch(const BatchLaunch& L, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_mid) {
    hipLaunchKernelGGL(k_batch_prep, dim3((L.n_ctl + 63) / 64), dim3(64), 0, stream, L.ctls, L.inputs, L.n_ctl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ev_start) (void)hipEventRecord(ev_start, stream);
    for (int i0 = 0; i0 < L.n_items; i0 += kMaxItemsPerLaunch) {  // one launch unless the batch is enormous
        const dim3 grid(std::min(L.n_items - i0, kMaxItemsPerLaunch));
        const int2* items = L.items + i0;
        if (L.noise_kind == 0)
            hipLaunchKernelGGL(k_batch_rollout_one<0>, grid, dim3(256), L.lds_rollout, stream, L.ctls, items, L.work);
        else if (L.noise_kind == 1)
            hipLaunchKernelGGL(k_batch_rollout_one<1>, grid, dim3(256), L.lds_rollout, stream, L.ctls, items, L.work);
        else if (L.noise_kind == 2)
            hipLaunchKernelGGL(k_batch_rollout_one<2>, grid, dim3(256), L.lds_rollout, stream, L.ctls, items, L.work);
        else
            hipLaunchKernelGGL(k_batch_rollout, grid, dim3(256), L.lds_rollout, stream, L.ctls, items, L.work);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    for (int i0 = 0; i0 < L.n_citems; i0 += kMaxItemsPerLaunch) {
        hipLaunchKernelGGL(k_batch_cvar, dim3(std::min(L.n_citems - i0, kMaxItemsPerLaunch)), dim3(256), L.lds_cvar,
                           stream, L.ctls, L.citems + i0);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (ev_mid) (void)hipEventRecord(ev_mid, stream);
    hipLaunchKernelGGL(k_batch_update, dim3(L.n_uitems), dim3(256), L.lds_update, stream, L.ctls, L.uitems);
    return hipGetLastError();
}

hipError_t batch_rollout_occupancy(int* wg_per_cu, size_t lds_rollout, int noise_kind) {
    if (noise_kind == 0)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(wg_per_cu, k_batch_rollout_one<0>, 256, lds_rollout);
    if (noise_kind == 1)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(wg_per_cu, k_batch_rollout_one<1>, 256, lds_rollout);
    if (noise_kind == 2)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(wg_per_cu, k_batch_rollout_one<2>, 256, lds_rollout);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(wg_per_cu, k_batch_rollout, 256, lds_rollout);
}

}  // namespace ramppi
