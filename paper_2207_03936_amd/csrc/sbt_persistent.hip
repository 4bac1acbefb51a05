// Batched form: a persistent work-stealing kernel that runs every stage of an
// event inside one workgroup and then takes the next event (largest first)
// from a device counter.  Built once per workgroup width (SBT_TPE).
#include <hip/hip_runtime.h>

#include "sbt.h"
#include "sbt_device.h"
#include "sbt_kernels.h"

#ifndef SBT_TPE
#error "SBT_TPE (workgroup width) must be defined"
#endif

using namespace sbt;

// The next event of a group, or -1 (on one lane; see kTakeOwnThenQueue).  Own
// events are taken by exchanging their entry of the order for -1, the others
// are met once.
template <int B>
__device__ __forceinline__ int take_event(const Work &W, int E, int group, int take)
{
    int32_t *order = ws_orderp(W);
    if (take == kTakeQueue) {
        const int idx = (int)atomicAdd(ws_counterp(W), 1u);
        return idx < E ? order[idx] : -1;
    }
    const int own = min((int)(gridDim.x * (B == 64 ? blockDim.x >> 6 : 1u)), E);
    int e = group >= 0 && group < E ? atomicExch(&order[group], -1) : -1;
    while (e < 0) {
        const int idx = (int)atomicAdd(ws_counterp(W), 1u);
        if (idx >= E + own) break;
        e = idx < E ? order[idx] : atomicExch(&order[idx - E], -1);
    }
    return e;
}

// One event per group of B lanes.  For B > 64 the group is the workgroup and
// its static LDS holds the event's Shared block.  For B = 64 a workgroup of
// any number of waves runs one event per wave, each with its own region of
// the dynamic LDS (the Shared block, then the layout of lds_bytes(CAP,
// own_cap) bytes), and no wave ever waits for another.  take: kTakeQueue,
// kTakeOwn or kTakeOwnThenQueue.
template <int B, int CAP>
__global__ __launch_bounds__((max_block_lanes<B, CAP>())) __attribute__((amdgpu_waves_per_eu(
    simd_waves<B, CAP>()))) void k_persistent(sbt_params P, HitsArgs H, Work W0, int own_cap, int sortcap, int take)
{
    uint32_t lo = 0;
    Shared<B> *sp;
    if constexpr (B == 64) {
        const uint32_t region = event_region_bytes<B>(CAP, own_cap);
        const uint32_t r0 = (uint32_t)uni((int)(threadIdx.x >> 6)) * region;
        sp = reinterpret_cast<Shared<B> *>(g_lds + r0);
        lo = r0 + shared_block_bytes<B>();
    } else {
        __shared__ Shared<B> S_wg;
        sp = &S_wg;
    }
    Shared<B> &S = *sp;
    int e = (int)blockIdx.x;
    if (B == 64) e = e * (int)(blockDim.x >> 6) + uni((int)(threadIdx.x >> 6));
    if (take == kTakeOwn) {
        e = e < H.n_events ? e : -1;
    } else {
        if (tid<B>() == 0) S.e = take_event<B>(W0, H.n_events, e, take);
        ev_sync<B>();
        e = uni(S.e);
    }
    while (e >= 0) {
        // the workspace base is hidden from the optimiser per event, so the
        // pointers derived from it are not hoisted out of this loop
        Work W = W0;
        W.base = opq_global(W0.base);
        W.H = opq(W0.H);
        W.E = opq(W0.E);
        int hb, N;
        const int st = load_event<B>(P, H, e, S, &hb, &N);
        if (tid<B>() == 0) ws_evinfo(W)[e].st = st;
        if (st == 0) {
            const Ev v = event_view(W, e, hb, N, lo);
            stage_sort<B>(P, H, v, S, sortcap);
            const bool in_lds = stage_track<B, CAP>(P, v, S, own_cap, false);
            const int n_fin = uni(S.cnt[3]);
            if (CAP > 0 && in_lds) {
                stage_filter_lds<B>(P, v, n_fin, lay_own(CAP));
                // (the LDS of 1,024-hit slots holds everything of events of up
                // to 22,300 hits, more than flags for 16,384 let in; the one
                // event that the rule runs there took 1.2 % longer with the
                // form for larger ones)
                stage_compact<B, true, CAP != 1024>(v, S.scan, (int)lds_sort_head() + 4 * sortcap);
            } else {
                stage_filter<B>(P, v, n_fin, v.own());
                stage_compact<B, false>(v, S.scan, (int)lds_sort_head() + 4 * sortcap);
            }
        } else if (tid<B>() == 0) {
            ws_evinfo(W)[e].nt = 0;
            ws_evinfo(W)[e].nh = 0;
        }
        if (take == kTakeOwn) break;
        ev_sync<B>();
        if (tid<B>() == 0) S.e = take_event<B>(W, H.n_events, -1, take);
        ev_sync<B>();
        e = uni(S.e);
    }
}

#if SBT_TPE == 512
// The 512-lane kernel held to six waves per SIMD (at most 80 VGPRs), so that
// three workgroups with 448- or 480-hit slots (49.5 or 52.7 KB of LDS each)
// share a compute unit: more events in flight for long batches.  With defer, events whose
// busiest module or flag count does not fit the LDS form are not run from
// memory but listed for a second pass.  The body is otherwise k_persistent's
// for B = 512, written out again: routing both kernels through one inlined
// function changes the default kernel's generated code, which is kept as it
// was measured.
template <int CAP>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6))) void k_persistent_dense(
    sbt_params P, HitsArgs H, Work W0, int own_cap, int sortcap, int defer)
{
    constexpr int B = 512;
    constexpr uint32_t lo = 0;
    __shared__ Shared<B> S;
    for (;;) {
        // the workspace base is hidden from the optimiser per event, so the
        // pointers derived from it are not hoisted out of this loop
        Work W = W0;
        W.base = opq_global(W0.base);
        W.H = opq(W0.H);
        W.E = opq(W0.E);
        if (tid<B>() == 0) {
            const int idx = (int)atomicAdd(ws_counterp(W), 1u);
            S.e = idx < H.n_events ? ws_orderp(W)[idx] : -1;
        }
        ev_sync<B>();
        const int e = uni(S.e);
        if (e < 0) break;
        int hb, N;
        const int st = load_event<B>(P, H, e, S, &hb, &N);
        if (defer && st == 0 && !event_fits_lds<B, CAP>(S, N, own_cap)) {
            // with defer, an event that does not fit the LDS slots is set
            // aside for a second pass with larger slots
            if (tid<B>() == 0) ws_deferp(W)[atomicAdd(ws_defer_countp(W), 1u)] = e;
        } else {
            if (tid<B>() == 0) ws_evinfo(W)[e].st = st;
            if (st == 0) {
                const Ev v = event_view(W, e, hb, N, lo);
                stage_sort<B>(P, H, v, S, sortcap);
                const bool in_lds = stage_track<B, CAP>(P, v, S, own_cap, false);
                const int n_fin = uni(S.cnt[3]);
                if (CAP > 0 && in_lds) {
                    stage_filter_lds<B>(P, v, n_fin, lay_own(CAP));
                    stage_compact<B, true>(v, S.scan, (int)lds_sort_head() + 4 * sortcap);
                } else {
                    stage_filter<B>(P, v, n_fin, v.own());
                    stage_compact<B, false>(v, S.scan, (int)lds_sort_head() + 4 * sortcap);
                }
            } else if (tid<B>() == 0) {
                ws_evinfo(W)[e].nt = 0;
                ws_evinfo(W)[e].nh = 0;
            }
        }
        ev_sync<B>();
    }
}

#endif

#define SBT_CAT2(a, b) a##b
#define SBT_CAT(a, b) SBT_CAT2(a, b)

namespace sbt {

const void *SBT_CAT(persistent_kernel_, SBT_TPE)(int cap)
{
    switch (cap) {
    case 0: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 0>);
    case 256: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 256>);
    case 448: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 448>);
    case 672: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 672>);
    case 768: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 768>);
    case 1024: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 1024>);
    case 1536: return reinterpret_cast<const void *>(k_persistent<SBT_TPE, 1536>);
    default: return nullptr;
    }
}

#if SBT_TPE == 512
const void *persistent_kernel_512_dense(int cap)
{
    switch (cap) {
    case 448: return reinterpret_cast<const void *>(k_persistent_dense<448>);
    case 480: return reinterpret_cast<const void *>(k_persistent_dense<480>);
    default: return nullptr;
    }
}
#endif

}  // namespace sbt
